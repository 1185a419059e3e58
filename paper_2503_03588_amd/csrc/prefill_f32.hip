// fp32 prefill (Equation 1 over the listed key blocks): fp32 inputs, fp32 products and sums, on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32 (its products and sums are those of an fp32 fused multiply-add).
//
// Decomposition.  A workgroup owns MQ tiles of 16 query rows of one head; its NW wavefronts share the KEYS: each walks
// a contiguous part of the row's 16-key tiles for all of the workgroup's queries with an online softmax of its own,
// and the (max, sum, O) of the wavefronts meet in LDS once, at the end.  No tile is staged in LDS and there is no
// barrier in the loop: a wavefront loads its K and V rows straight into operand registers, each used by MQ tiles.
//
// In the transposed form S^T = K Q^T (A = K rows, B = Q^T) a lane owns one query column, and its four scores of a
// 16-key tile are the keys 4*(lane/16) + r, which is what O^T += V^T P^T takes as its B operand when step r contracts
// over the keys 4*(lane/16) + r, lane/16 = 0..3.  The contraction index of S^T is permuted so that one 16-byte load
// of a K row feeds four steps, and the rows of O^T so that one 16-byte load of a V row feeds four tiles of it.
//
// Bound by the fp32 matrix rate (153 TFLOP/s in a large matrix product on the same card): 84 TFLOP/s at 8 heads,
// head_dim 64, N = 8192, blocks of 64 keys, 80 at head_dim 128; a kernel of plain multiply-adds with K/V staged in LDS,
// which this replaced, 4.  Short prompts are bound by latency (2 heads, N = 1024: 74 us before, 10.5 now).
//
// Loads run LA tiles ahead of the products (the K tiles of a step of TS tiles, then its V tiles, then the next step's).
#include <math.h>
#include "common.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int N> struct f32_vec { typedef f32x4 type; };
template <> struct f32_vec<2> { typedef f32x2 type; };

struct f32_params {
  const float* q; const float* k; const float* v; float* o; float* lse;
  const int32_t* kv_cnt; const int32_t* kv_idx;
  int32_t max_k, nb, B, hq, hkv, G, dense;
  int32_t q_tiles;               // workgroups per head and part of the head dimension: nb * per_block
  uint32_t per_block_magic, tpb_magic, G_magic;   // reciprocals of B / query rows of a workgroup, B / 16 and G (see quot)
  int64_t N;
  float c2;   // softmax scale * log2(e)
};

constexpr int NW = 4;              // wavefronts per workgroup (eight share the compute unit's matrix cores no better and
                                   // have twice the partials to merge: 10-40 % slower at every size measured)
constexpr float RAISE_BY = 8.0f;   // the exponentials' reference point is raised when exceeded by 2^8: any reference
                                   // gives the same result, and raising it costs a multiplication of all of O

constexpr int o_stride(int DV) { return DV + 4; }   // floats per query row of a wavefront's partial output in LDS
template <int DV, int MQ>
constexpr size_t merge_lds() { return sizeof(float) * NW * 16 * MQ * (o_stride(DV) + 2); }

// x / y through ceil(2^32 / y), which the host passes where it is exact for every x (else 0): divisions stand in front of the
// first load, forty instructions each in 32 bits and a hundred in 64.
__device__ __forceinline__ int quot(int x, int y, uint32_t magic) {
  return y == 1 ? x : magic ? (int)__umulhi((uint32_t)x, magic) : x / y;
}

// DS: the output's columns are dealt to DS workgroups, which all form the scores (launches that leave compute units idle)
template <int D, int MQ, int DS>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void pa_prefill_f32_kernel(f32_params p) {
  constexpr int NK = D / 16;                // 16-byte pieces of a K row per lane; each feeds four steps
  constexpr int DV = D / DS;                // columns of V and O of this workgroup
  constexpr int VW = DV >= 64 ? 4 : 2;      // floats in a lane's piece of a V row; each feeds a tile of O^T
  constexpr int NV = DV / (16 * VW);        // pieces per lane
  typedef typename f32_vec<VW>::type v_piece;
  constexpr int QR = 16 * MQ;               // query rows of the workgroup
  constexpr int TS = MQ * D <= 128 ? 4 : 2; // 16-key tiles per step (scores held at a time)
  // Sums a score is formed in (one for every CH-th head element), added up at the end.  With a single sum of D products the
  // outputs were up to 1.6 times as far from 64 bits (2-norm; 2.3 times, largest difference) as those of four short ones
  // per lane in plain multiply-adds; with these 0.44 .. 0.88 times (0.42 .. 0.94).  Four 16-row tiles at head_dim 64 have no
  // registers for more than two (four spill 40: 52.8 -> 57.3 us at 8 heads, N = 4096), and reach long sequences only.
  constexpr int CH = MQ == 4 ? 2 : 4;
  constexpr int LA = MQ * D <= 64 ? 4 : MQ * D <= 128 ? 2 : 1;   // tiles loaded ahead
  extern __shared__ __attribute__((aligned(16))) float s_o[];   // [NW][QR][DV + 4], then the maxima and sums [NW][QR]
  float* s_m = s_o + NW * QR * o_stride(DV);
  float* s_l = s_m + NW * QR;
  __shared__ int s_some[NW];                // whether the wavefront's part held any key

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 15, kg = lane >> 4;
  int dpart = 0;                                               // (a quotient below four: a compare each)
#pragma unroll
  for (int x = 1; x < DS; ++x) dpart += (int)blockIdx.x >= x * p.q_tiles;
  const int qx = (int)blockIdx.x - dpart * p.q_tiles, qblk = quot(qx, p.B / QR, p.per_block_magic);
  const int qb = p.nb - 1 - qblk;                              // longest rows first
  const int q_in_blk = (qx - qblk * (p.B / QR)) * QR;
  const int h = blockIdx.y, b = blockIdx.z;
  const int kvh = quot(h, p.G, p.G_magic);
  const int64_t q0 = (int64_t)qb * p.B + q_in_blk;
  if (q0 >= p.N) return;                                       // uniform over the workgroup

  const float* qbase = p.q + ((int64_t)b * p.hq + h) * p.N * D;
  const float* kbase = p.k + ((int64_t)b * p.hkv + kvh) * p.N * D;
  const float* vbase = p.v + ((int64_t)b * p.hkv + kvh) * p.N * D + dpart * DV;

  // ---- the row's list, 64 entries at a time: lane e keeps entry list_base + e ----
  const int32_t* list = p.kv_idx + (int64_t)qb * p.max_k;
  auto list_lanes = [&](int base) -> int {
    if (p.dense) return base + lane;
    const int e = base + lane;
    return list[e < p.max_k ? e : p.max_k - 1];
  };
  int row_e = list_lanes(0);                                   // requested beside the count, not after it
  int n_list = qb + 1;
  if (!p.dense) {
    n_list = p.kv_cnt[qb];
    if (n_list > p.max_k) n_list = p.max_k;
  }
  f32x4 qf[MQ][NK];
#pragma unroll
  for (int m = 0; m < MQ; ++m) {
    const int64_t row = q0 + 16 * m + ln;
#pragma unroll
    for (int c = 0; c < NK; ++c)
      qf[m][c] = row < p.N ? *reinterpret_cast<const f32x4*>(qbase + row * D + 16 * c + 4 * kg) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  n_list = __builtin_amdgcn_readfirstlane(n_list);

  // ---- this wavefront's 16-key tiles: tile tau is piece tau % tpb of list entry tau / tpb ----
  const int tpb = p.B / 16;
  const int diag_tiles = q_in_blk / 16 + MQ;                   // tiles of the diagonal block that any query reaches
  int tiles = n_list * tpb;                                    // (fewer than 2^27: positions are 32-bit numbers)
  int last_row = row_e;
  if (n_list > 64) last_row = list_lanes((n_list - 1) & ~63);
  if (n_list > 0 && __builtin_amdgcn_readlane(last_row, (n_list - 1) & 63) == qb) tiles -= tpb - diag_tiles;
  static_assert(NW == 4, "the parts of the row are formed with shifts");
  const int lo = (tiles >> 2) * wave + (((tiles & 3) * wave) >> 2), hi = (tiles >> 2) * (wave + 1) + (((tiles & 3) * (wave + 1)) >> 2);
  const int n_steps = (hi - lo + TS - 1) / TS;
  int ct = quot(lo, tpb, p.tpb_magic), cs = lo - ct * tpb;     // cursor of the loads: list entry, piece
  int left = hi - lo;
  if (ct >= 64) row_e = list_lanes(ct & ~63);
  const int last = (int)(p.N - 1);
  bool any = false;                                            // a tile to attend: a block's first one holds a key of every query
  auto next_key0 = [&]() -> int {                              // first key of the next tile, or -1: nothing to attend
    const int j = __builtin_amdgcn_readlane(row_e, ct & 63);
    const bool some = left > 0 && j >= 0 && (j < qb || (j == qb && cs < diag_tiles));
    int key0 = some ? j * p.B + 16 * cs : -1;
    if (key0 > last) key0 = -1;                                // (later query tiles of a last block that is not full)
    any = any || key0 >= 0;
    --left;
    if (++cs == tpb) {
      cs = 0;
      if ((++ct & 63) == 0) row_e = list_lanes(ct);
    }
    return key0;
  };

  f32x4 kf[TS][NK];
  v_piece vf[TS][4][NV];
  // A tile's address is scalar, a lane adds its row and piece; rows beyond the sequence repeat its last one (masked).
  // "No tile" reads the start of the slab and its products are left out, so that nothing unattended reaches the sums.
  auto load_k = [&](int i, int key0) {
    const int k0 = key0 < 0 ? 0 : key0, lim = last - k0;
    const float* src = kbase + (int64_t)k0 * D;
    const uint32_t off = (uint32_t)(ln < lim ? ln : lim) * D + 4 * kg;
#pragma unroll
    for (int c = 0; c < NK; ++c) kf[i][c] = *reinterpret_cast<const f32x4*>(src + off + 16 * c);
  };
  auto load_v = [&](int i, int key0) {
    const int k0 = key0 < 0 ? 0 : key0, lim = last - k0;
    const float* src = vbase + (int64_t)k0 * D;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * kg + r;
      const uint32_t off = (uint32_t)(row < lim ? row : lim) * D + VW * ln;
#pragma unroll
      for (int x = 0; x < NV; ++x) vf[i][r][x] = *reinterpret_cast<const v_piece*>(src + off + 16 * VW * x);
    }
  };

  f32x4 O[MQ][VW * NV];
  float m_run[MQ], l_run[MQ];
#pragma unroll
  for (int m = 0; m < MQ; ++m) {
    m_run[m] = -INFINITY; l_run[m] = 0.f;
#pragma unroll
    for (int j = 0; j < VW * NV; ++j) O[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  int key0[TS], nkey0[TS];
#pragma unroll
  for (int i = 0; i < TS; ++i) key0[i] = next_key0();
#pragma unroll
  for (int i = 0; i < LA; ++i) load_k(i, key0[i]);

  for (int s = 0; s < n_steps; ++s) {
#pragma unroll
    for (int i = 0; i < TS; ++i) nkey0[i] = next_key0();
    auto load_ahead = [&](int at) {                            // number at + LA of: the step's K tiles, its V tiles, the next K tiles
      const int x = at + LA;
      if (x < TS) load_k(x, key0[x % TS]);
      else if (x < 2 * TS) load_v(x % TS, key0[x % TS]);
      else load_k(x % TS, nkey0[x % TS]);
    };
    // ---- S^T = K Q^T ----
    f32x4 S[MQ][TS];
#pragma unroll
    for (int i = 0; i < TS; ++i) {
      load_ahead(i);
      __builtin_amdgcn_sched_barrier(0);
      if (key0[i] < 0) {
#pragma unroll
        for (int m = 0; m < MQ; ++m) S[m][i] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      } else {
        f32x4 part[CH][MQ];
#pragma unroll
        for (int x = 0; x < CH * MQ; ++x) part[x / MQ][x % MQ] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NK; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int m = 0; m < MQ; ++m)
              part[e % CH][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][c][e], qf[m][c][e], part[e % CH][m], 0, 0, 0);
#pragma unroll
        for (int m = 0; m < MQ; ++m)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            S[m][i][r] = CH == 4 ? (part[0][m][r] + part[1][m][r]) + (part[2 % CH][m][r] + part[3 % CH][m][r])
                                 : part[0][m][r] + part[1][m][r];
        if ((int64_t)key0[i] + 15 > q0) {                      // causality: a tile that reaches the workgroup's queries
#pragma unroll
          for (int m = 0; m < MQ; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if ((int64_t)key0[i] + 4 * kg + r > q0 + 16 * m + ln) S[m][i][r] = -INFINITY;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- online softmax ----
#pragma unroll
    for (int m = 0; m < MQ; ++m) {
      float mx = S[m][0][0];
#pragma unroll
      for (int x = 1; x < 4 * TS; ++x) mx = fmaxf(mx, S[m][x >> 2][x & 3]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * p.c2;
      const bool raise = mx > m_run[m] + RAISE_BY;             // (a first score raises -inf)
      if (__builtin_amdgcn_ballot_w64(raise) != 0) {
        const float m_new = raise ? mx : m_run[m];
        const float alpha = raise ? __builtin_amdgcn_exp2f(m_run[m] - m_new) : 1.f;
        m_run[m] = m_new;
        l_run[m] *= alpha;
#pragma unroll
        for (int j = 0; j < VW * NV; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) O[m][j][r] *= alpha;
      }
      const float ref = m_run[m] == -INFINITY ? 0.f : m_run[m];   // nothing attended yet: every exponential is 0
      float sum = 0.f;
#pragma unroll
      for (int x = 0; x < 4 * TS; ++x) {
        const float pe = __builtin_amdgcn_exp2f(fmaf(S[m][x >> 2][x & 3], p.c2, -ref));
        S[m][x >> 2][x & 3] = pe;
        sum += pe;
      }
      l_run[m] += sum;
    }
    // ---- O^T += V^T P^T: row R of tile VW x + j is column VW (16x + R) + j of the workgroup's ----
#pragma unroll
    for (int i = 0; i < TS; ++i) {
      load_ahead(TS + i);
      __builtin_amdgcn_sched_barrier(0);
      if (key0[i] >= 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int x = 0; x < NV; ++x)
#pragma unroll
            for (int j = 0; j < VW; ++j)
#pragma unroll
              for (int m = 0; m < MQ; ++m)
                O[m][VW * x + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i][r][x][j], S[m][i][r], O[m][VW * x + j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < TS; ++i) key0[i] = nkey0[i];
  }

  // ---- the wavefronts' partials meet in LDS ----
  if (lane == 0) s_some[wave] = any;
#pragma unroll
  for (int m = 0; m < MQ; ++m) {
    const int row = wave * QR + 16 * m + ln;
    float l = l_run[m] + __shfl_xor(l_run[m], 16);
    l += __shfl_xor(l, 32);
    if (kg == 0) { s_m[row] = m_run[m]; s_l[row] = l; }
#pragma unroll
    for (int x = 0; x < NV; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v_piece piece;
#pragma unroll
        for (int j = 0; j < VW; ++j) piece[j] = O[m][VW * x + j][r];
        *reinterpret_cast<v_piece*>(s_o + row * o_stride(DV) + VW * (16 * x + 4 * kg + r)) = piece;
      }
  }
  __syncthreads();
  int some = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) some |= s_some[w];
  for (int e = tid; e < QR * (DV / 4); e += 64 * NW) {
    const int row = e / (DV / 4), d4 = e % (DV / 4);
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w * QR + row]);
    float L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float lw = s_l[w * QR + row];
      const float wt = lw > 0.f ? __builtin_amdgcn_exp2f(s_m[w * QR + row] - M) : 0.f;   // (0 times a sum that is NaN is NaN)
      L = fmaf(wt, lw, L);
      const f32x4 ow = *reinterpret_cast<const f32x4*>(s_o + (w * QR + row) * o_stride(DV) + 4 * d4);
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] = fmaf(wt, ow[x], acc[x]);
    }
    const int64_t tok = q0 + row;
    if (tok >= p.N) continue;
    // a row whose list is empty: o = 0, lse = -inf; one whose scores are all -inf: 0 * (1 / 0), no number, as softmax has it
    const float inv = some ? 1.0f / L : 0.f;
    const int64_t at = ((int64_t)b * p.hq + h) * p.N + tok;
    *reinterpret_cast<f32x4*>(p.o + at * D + dpart * DV + 4 * d4) = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
    if (p.lse && d4 == 0 && dpart == 0) p.lse[at] = (M + log2f(L)) * 0.69314718055994530942f;
  }
}

template <int D, int MQ, int DS>
int launch(f32_params p, int32_t batch, hipStream_t stream) {
  constexpr size_t lds = merge_lds<D / DS, MQ>();
  static std::atomic<unsigned long long> done{0};
  if (int st = pa_allow_dynamic_lds(reinterpret_cast<const void*>(&pa_prefill_f32_kernel<D, MQ, DS>), lds, done)) return st;
  const int per_block = p.B / (16 * MQ), tpb = p.B / 16;
  // exact for x < n if n * y <= 2^32
  auto magic = [](int64_t n, int64_t y) -> uint32_t { return y > 1 && n * y <= 0xffffffffLL ? (uint32_t)(((1ull << 32) + y - 1) / y) : 0u; };
  p.q_tiles = p.nb * per_block;
  p.per_block_magic = magic((int64_t)p.nb * per_block, per_block);
  p.tpb_magic = magic((int64_t)(p.max_k > p.nb ? p.max_k : p.nb) * tpb, tpb);
  p.G_magic = magic(p.hq, p.G);
  dim3 grid((uint32_t)p.q_tiles * DS, (uint32_t)p.hq, (uint32_t)batch);
  hipLaunchKernelGGL((pa_prefill_f32_kernel<D, MQ, DS>), grid, dim3(64 * NW), lds, stream, p);
  return pa_note_hip(hipGetLastError());
}

// Query tiles per workgroup.  A K/V row loaded once serves MQ tiles, so larger is better (8 heads, head_dim 64,
// N = 8192: 59 / 70 / 84 TFLOP/s at 1 / 2 / 4) as long as every compute unit gets a workgroup: at 8 heads and N = 1024
// 1 / 2 / 4 tiles (512 / 256 / 128 workgroups) take 19.8 / 16.3 / 26.1 us, at 2 heads 11.6 / 15.1 / 25.4.
// At most 64 queries at head_dim 64 and 32 at 128, which is what the 256 registers of a wavefront hold.
// Where even workgroups of 16 queries leave half of the compute units idle, the output's columns are dealt to two or four
// workgroups: half of a workgroup's products are those of the output, and the scores are
// formed anew.  us with the list, one / more workgroups: head_dim 128, 2 heads, N = 1000 17.8 / 16.0, N = 130 (four) 12.1 / 11.0.
// Without it, head_dim 64: 2 heads, N = 1024 10.46 / 10.13, 512 10.10 / 9.81, 130 7.06 / 6.72; 4 heads, N = 500 8.28 / 7.81; 8, N = 200
// 7.55 / 7.15.  (With the list: steps of six or eight key tiles instead of four at head_dim 64: 12.5, 13.2 where four take 12.1.)
template <int D>
int launch_d(const f32_params& p, int32_t batch, hipStream_t stream) {
  constexpr int MQ_MAX = 256 / D;
  int n_cu = 1;
  pa_current_device(nullptr, &n_cu);
  const int64_t tiles = (int64_t)p.nb * (p.B / 16) * p.hq * batch;
  int mq = 1;
  while (mq < MQ_MAX && p.B % (32 * mq) == 0 && tiles / (2 * mq) >= n_cu) mq *= 2;
  if constexpr (MQ_MAX == 4)
    if (mq == 4) return launch<D, 4, 1>(p, batch, stream);
  if (mq == 2) return launch<D, 2, 1>(p, batch, stream);
  if constexpr (D == 128)
    if (4 * tiles <= n_cu) return launch<D, 1, 4>(p, batch, stream);
  return 2 * tiles <= n_cu ? launch<D, 1, 2>(p, batch, stream) : launch<D, 1, 1>(p, batch, stream);
}

}  // namespace

int pa_launch_prefill_f32(const pa_prefill_args& a) {
  f32_params p;
  p.q = (const float*)a.q; p.k = (const float*)a.k; p.v = (const float*)a.v; p.o = (float*)a.o; p.lse = a.lse;
  p.kv_cnt = a.kv_cnt; p.kv_idx = a.kv_idx; p.max_k = a.max_k; p.nb = a.nb; p.B = a.pat.block;
  p.hq = a.hq; p.hkv = a.hkv; p.G = a.hq / a.hkv; p.dense = (a.pat.flags & POWATTN_DENSE) ? 1 : 0;
  p.N = a.seq_len;
  p.c2 = a.scale * 1.44269504088896340736f;
  if (a.hq > 65535 || a.batch > 65535) return POWATTN_UNSUPPORTED;
  if (a.seq_len > 0x7fffffffLL - 1024) return POWATTN_UNSUPPORTED;   // key positions are kept in 32 bits
  return a.head_dim == 64 ? launch_d<64>(p, a.batch, a.stream) : launch_d<128>(p, a.batch, a.stream);
}
