// Gradients of Equation 1 (Section 3.1) under the block pattern of Algorithm 1, bf16 inputs, fp32 accumulation.
// The paper trains with the sparse pattern in place (Section 4.1), which needs dQ, dK and dV of
//   O = softmax(mask(scale Q K^T)) V.
// With P the softmax (recomputed from the saved log-sum-exp), dP = dO V^T, Delta_i = sum_d dO_id O_id and
// dS = P * (dP - Delta):   dQ = scale dS K,   dK = scale dS^T Q,   dV = P^T dO.
//
// Two kernels:
//   dq    : a workgroup per (batch, KV head, query block, group of query-head slices) walks the row's key blocks
//           (the lists powattn_mask_build writes), as the forward pass does; wavefront = 32 queries of one head,
//           lane = one query.  S^T = K Q^T and dP^T = V dO^T share the K/V tiles in LDS; dQ^T += K^T dS^T.
//           It also forms Delta = rowsum(dO * O) of its rows (dO is in its registers anyway) and leaves it, with
//           the log-sum-exp in base-2 units, in the workspace for the kernel below.
//   dkv   : a workgroup per (batch, KV head, slab of 32, 64 or 128 keys of a block) walks the COLUMN of the block mask: the
//           query blocks j .. j+W-1 and j + 2^k (closed form), all of them for a sink block; lane = one key.
//           Q and dO tiles go through LDS; dV^T += dO^T P, dK^T += Q^T dS.  A sink block's column is
//           as long as the sequence: it is cut into parts that add into an fp32 buffer, converted at the end.
//           The two halves of this work sit on different wavefronts.
// Both products of a pair reuse the forward kernel's operand trick: in the transposed form the accumulator layout
// of the first product is the B-operand layout of the second (the permutation of the contraction index inside a
// 16-step is applied to both operands).  Tiles use the forward kernel's LDS layout (chunk-major kilobytes, padded),
// copied asynchronously global -> LDS, one barrier per tile.
#include <math.h>
#include <type_traits>
#include "common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;

constexpr int KT = 64;            // rows per staged tile
constexpr int TILE_CAP = 2048;    // tiles per query block in the dq kernel
constexpr int PFD = 2;            // matrix instructions per group of LDS fragment reads
constexpr float LOG2E = 1.44269504088896340736f;
constexpr int dq_stages(int) { return 2; }   // LDS stages of the dQ kernel's tile stream (see there)

struct bwd_params {
  const __bf16* q; const __bf16* k; const __bf16* v; const __bf16* o; const __bf16* dout; const float* lse;
  __bf16* dq; __bf16* dk; __bf16* dv;
  float* delta;          // [batch, hq, N]: -Delta
  float* lse2;           // [batch, hq, N]: the log-sum-exp in base-2 units (lse * log2 e)
  float* dk_sink;        // [batch, hkv, sink_rows, D] fp32 sums of the sink blocks' parts
  float* dv_sink;
  const int32_t* kv_cnt; const int32_t* kv_idx;
  int32_t max_k, nb, B, W, S; uint32_t flags;
  int32_t hq, hkv, G, subs, tasks, chunks;
  int32_t sink_blocks;   // min(S, nb) (0 when the column of no block is cut)
  int32_t part;          // query blocks per part of a sink block's column
  int32_t max_parts;     // parts of the longest column
  int64_t N;
  int64_t sink_floats;   // from dk_sink on: both sums, cleared by the dQ kernel (a multiple of 64)
  float scale, c2;
};

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
// 16 bytes per lane: lane l's land at lds_base + OFF + 16*l
template <int OFF>
__device__ __forceinline__ void async_copy16_at(const void* sbase, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_add_u32 m0, %2, %3\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_base), "n"(OFF) : "memory", "scc", "m0");
}
// one dword per lane: lane l's value lands at lds_off + 4*l
__device__ __forceinline__ void async_copy4(const void* addr, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dword %0, off" ::"v"(addr), "s"(lds_off) : "memory", "m0");
}
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* ptr) {
  const uint64_t u = (uint64_t)(uintptr_t)ptr;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const T*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ uint32_t pack2(float x, float y) {
  const f32x2 v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Geometry of a staged tile of 64 rows x D bf16 (the forward kernel's layout).
template <int D>
struct tile_geo {
  static constexpr int ROWB = 2 * D;
  static constexpr int CPR = D / 8;
  static constexpr int RPI = 64 / CPR;          // rows per wavefront-wide copy instruction
  static constexpr int IPT = KT / RPI;          // copy instructions per tile
  static constexpr int SRB = 1024 + 16 * RPI;   // LDS distance between consecutive copy instructions' kilobytes
  static constexpr int TILEB = IPT * SRB;
  static constexpr int NC = D / 16;             // 16-wide steps of the head dimension
  static constexpr int ND = D / 32;             // 32-row tiles of a transposed accumulator
  static constexpr int K_C = 32 * RPI, K_RT = (32 / RPI) * SRB;
  static constexpr int V_KK = (16 / RPI) * SRB, V_DT = 4 * RPI * 16, V_HI = (8 / RPI) * SRB;
};

// copy instruction X of a wavefront's share of a tile, and the ones after it (instruction number wave + X * NWV)
template <int D, int NWV, int X>
__device__ __forceinline__ void copy_tile_unrolled(const __bf16* sb, int row0w, int lim, uint32_t chunk_off, uint32_t wdst) {
  using G = tile_geo<D>;
  if constexpr (X < G::IPT / NWV) {
    int row = row0w + G::RPI * NWV * X;
    row = row < lim ? row : lim;
    async_copy16_at<X * NWV * G::SRB>(sb, (uint32_t)row * G::ROWB + chunk_off, wdst);
    copy_tile_unrolled<D, NWV, X + 1>(sb, row0w, lim, chunk_off, wdst);
  }
}
// Copies rows row0 .. row0+63 of a row-major [rows, D] array (rows beyond `last_row` repeat it) into the LDS tile
// at `dst`; the NWV wavefronts of the workgroup share the tile's copy instructions.
template <int D, int NWV>
__device__ __forceinline__ void copy_tile(const __bf16* base, int64_t row0, int64_t last_row, uint32_t dst, int wave, int lane) {
  using G = tile_geo<D>;
  const int cp_row = lane % G::RPI, cp_chunk = lane / G::RPI;
  int64_t r0 = row0 < last_row ? row0 : last_row;
  const int lim = (int)(last_row - r0);
  const __bf16* sb = uniform_ptr(base + r0 * D);
  static_assert(G::IPT % NWV == 0, "tile copies must divide over the wavefronts");
  const uint32_t wdst = __builtin_amdgcn_readfirstlane(dst + wave * G::SRB);
  copy_tile_unrolled<D, NWV, 0>(sb, G::RPI * wave + cp_row, lim, (uint32_t)(cp_chunk << 4), wdst);
}
// A operand "rows of the tile": rows 32rt + (lane%32), elements 16c + 8(lane/32) .. +7
template <int D>
__device__ __forceinline__ bf16x8 row_frag(uint32_t tile, int c, int rt, int lane) {
  using G = tile_geo<D>;
  const int ln = lane & 31, hh = lane >> 5;
  const uint32_t a = tile + (ln / G::RPI) * G::SRB + ((hh * G::RPI + ln % G::RPI) << 4) + c * G::K_C + rt * G::K_RT;
  return *reinterpret_cast<const lds_bf16x8*>((uintptr_t)a);
}
// A operand "transposed tile": row = element 32dt + lane%32 of the head dimension, contraction over the tile's rows
// 16kk .. 16kk+15 in the order {0..3, 8..11} + 4(lane/32), {4..7, 12..15} for the other half-wave
template <int D>
__device__ __forceinline__ bf16x8 tr_frag(uint32_t tile, int kk, int dt, int lane) {
  using G = tile_geo<D>;
  const int hh = lane >> 5;
  const int r4 = 4 * hh + ((lane & 15) >> 2);
  const int x = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  const uint32_t a = tile + (r4 / G::RPI) * G::SRB + ((x * G::RPI + r4 % G::RPI) << 4) + 8 * (lane & 1) + kk * G::V_KK + dt * G::V_DT;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)a);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(a + G::V_HI));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// B operand "rows held in registers": lane = row (lane%32), elements 16c + 8(lane/32) .. +7; zero when !ok
template <int D>
__device__ __forceinline__ void reg_rows(const __bf16* row, bool ok, int lane, bf16x8 (&f)[D / 16]) {
  const int hh = lane >> 5;
#pragma unroll
  for (int c = 0; c < D / 16; ++c) {
    const bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    f[c] = ok ? *reinterpret_cast<const bf16x8*>(row + 16 * c + 8 * hh) : z;
  }
}
// N matrix instructions whose A operands come from LDS, software-pipelined with scheduling barriers (left alone,
// the compiler reads each fragment right before its use into the same registers, and a wavefront that is alone on
// its SIMD waits out every LDS latency).
template <int N, int GRP, class LoadF, class MmaF>
__device__ __forceinline__ void pipelined_mfma(LoadF load, MmaF mma) {
  // groups of GRP instructions: the reads of the next group go out together before the current group's matrix
  // instructions, so that one wait serves a whole group
  static_assert(N % GRP == 0, "instructions must come in whole groups");
  bf16x8 fr[N];
#pragma unroll
  for (int m = 0; m < GRP; ++m) fr[m] = load(m);
#pragma unroll
  for (int g = 0; g < N / GRP; ++g) {
    if (g + 1 < N / GRP) {
#pragma unroll
      for (int j = 0; j < GRP; ++j) fr[(g + 1) * GRP + j] = load((g + 1) * GRP + j);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = GRP - 1; j >= 0; --j) mma(g * GRP + j, fr[g * GRP + j]);   // the last one first: LDS answers in order, so its wait covers the group
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Element rg (0..15) of a 32x32 accumulator is row 8(rg/4) + 4(lane/32) + rg%4, column lane%32.
__device__ __forceinline__ int acc_row(int rg, int hh) { return 8 * (rg >> 2) + 4 * hh + (rg & 3); }

// ---------------------------------------------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------------------------------------------
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void pa_bwd_dq_kernel(bwd_params p) {
  using G = tile_geo<D>;
  constexpr int NC = G::NC, ND = G::ND;
  constexpr int STAGEB = 2 * G::TILEB;           // K tile then V tile
  // LDS stages of the tile stream: the copies run NST-1 tiles ahead of the products.  Two: four stages for the
  // workgroups of eight wavefronts (which have their compute unit to themselves anyway) were measured 5 % slower
  // at the 128K workload, three halve the workgroups per compute unit at blocks of 64 keys.
  constexpr int NST = dq_stages(NW);
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  __shared__ int s_tile[TILE_CAP];
  __shared__ int s_ntiles;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, hh = lane >> 5;
  const int slice_bits = __builtin_ctz((unsigned)p.B / 32);      // blocks are 64, 128 or 256 keys

  // item: ((b*hkv + kvh)*nb + i)*chunks + chunk (in 32 bits: the divisions stand in front of every workgroup's first load)
  uint32_t L = blockIdx.x, rest = L / (uint32_t)p.chunks;
  const int chunk = (int)(L - rest * (uint32_t)p.chunks);
  L = rest; rest = L / (uint32_t)p.nb;
  const int i = (int)(L - rest * (uint32_t)p.nb);
  L = rest; rest = L / (uint32_t)p.hkv;
  const int kvh = (int)(L - rest * (uint32_t)p.hkv);
  const int b = (int)rest;

  // ---- the row's tiles: every 64-key tile of every listed block up to the diagonal one ----
  // The first wavefront reads 64 list entries at a time, one per lane (a single thread walking the list pays a
  // trip to memory per entry, at the start of every workgroup); the rank of a valid entry is a prefix count.
  if (wave == 0) {
    // (the first entries are requested beside the row's length, not after it)
    int ahead = p.kv_idx[(int64_t)i * p.max_k + (lane < p.max_k ? lane : p.max_k - 1)];
    int n = p.kv_cnt[i];
    if (n > p.max_k) n = p.max_k;
    n = __builtin_amdgcn_readfirstlane(n);
    int blocks = 0;
    for (int base = 0; base < n; base += 64) {
      const int e = base + lane;
      if (base > 0) ahead = e < n ? p.kv_idx[(int64_t)i * p.max_k + e] : -1;
      const int j = e < n ? ahead : -1;
      const bool valid = j >= 0 && j <= i;
      const uint64_t vm = __builtin_amdgcn_ballot_w64(valid);
      const int rank = blocks + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(vm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)vm, 0));
      if (valid)
        for (int u = 0; u < p.subs; ++u)
          if (rank * p.subs + u < TILE_CAP) s_tile[rank * p.subs + u] = j * p.B + u * KT;
      blocks += __builtin_popcountll(vm);
    }
    if (lane == 0) s_ntiles = blocks * p.subs < TILE_CAP ? blocks * p.subs : TILE_CAP;
  }
  __syncthreads();
  const int n_tiles = s_ntiles;

  const int task = chunk * NW + wave;
  const bool active = task < p.tasks;
  const int g = active ? task >> slice_bits : 0, sl = active ? task & ((1 << slice_bits) - 1) : 0;
  const int h = kvh * p.G + g;
  const int64_t tok = (int64_t)i * p.B + sl * 32 + ln;          // this lane's query
  const bool ok = active && tok < p.N;
  const int64_t qrow = ((int64_t)b * p.hq + h) * p.N + (ok ? tok : 0);

  const __bf16* kslab = p.k + ((int64_t)b * p.hkv + kvh) * p.N * D;
  const __bf16* vslab = p.v + ((int64_t)b * p.hkv + kvh) * p.N * D;
  static_assert(G::IPT % NW == 0, "tile copies must divide over the wavefronts");
  constexpr int CPF = 2 * G::IPT / NW;     // copies per wavefront and fill (K and V)
  auto fill = [&](int t) {
    const int key0 = s_tile[t];
    const uint32_t dst = lds0 + (t % NST) * STAGEB;
    copy_tile<D, NW>(kslab, key0, p.N - 1, dst, wave, lane);
    copy_tile<D, NW>(vslab, key0, p.N - 1, dst + G::TILEB, wave, lane);
  };
  // the first tiles are requested before this wavefront's own rows: their copies would queue behind those loads
  for (int s0 = 0; s0 < NST - 1; ++s0)
    if (s0 < n_tiles) fill(s0);

  bf16x8 qf[NC], dof[NC];
  reg_rows<D>(p.q + qrow * D, ok, lane, qf);
  reg_rows<D>(p.dout + qrow * D, ok, lane, dof);
  // Delta = rowsum(dO * O) of this lane's row and its log-sum-exp in base-2 units: formed here, where the row of dO
  // is in registers anyway (the two halves of the wavefront hold the two halves of the row), and left in the
  // workspace for the dK/dV kernel, which follows on the stream.  Every row belongs to exactly one task.
  float lse2 = INFINITY, dl = 0.f;                               // exp2(s - inf) = 0: idle lanes contribute nothing
  {
    bf16x8 of[NC];
    reg_rows<D>(p.o + qrow * D, ok, lane, of);
    float part = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) part = fmaf((float)of[c][e], (float)dof[c][e], part);
    part += __shfl_xor(part, 32);
    if (ok) {
      dl = part;
      lse2 = p.lse[qrow] * LOG2E;
      if (hh == 0) { p.delta[qrow] = -dl; p.lse2[qrow] = lse2; }
    }
  }
  const int tok32 = (int)tok, n32 = (int)p.N;                    // positions fit 32 bits (checked by the host)
  // the sums of dP start at -Delta (every element of a lane belongs to its one query): no subtraction per element
  f32x16 minus_delta;
#pragma unroll
  for (int r = 0; r < 16; ++r) minus_delta[r] = -dl;

  f32x16 acc[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;
  // Tile t has landed when only the fills of tiles t+1 .. t+NST-2 are outstanding (the counter retires in
  // order).  Near the end, where fewer fills follow, wait for all.  (The loads of Q and dO above are younger than
  // the first fills; the compiler waits for them before their first use, which covers everything older.)
  for (int t = 0; t < n_tiles; ++t) {
    if (t + NST - 1 <= n_tiles) wait_vmcnt<(NST - 2) * CPF>(); else wait_vmcnt<0>();
    __syncthreads();                       // tile t has landed for everybody; everybody is done with tile t-1
    if (t + NST - 1 < n_tiles) fill(t + NST - 1);        // into the stage tile t-1 has just left
    const int key0 = s_tile[t];
    // tiles that start beyond this wavefront's last query are masked out entirely for it
    if (!active || (int64_t)key0 > (int64_t)i * p.B + sl * 32 + 31) continue;
    const uint32_t kt = lds0 + (t % NST) * STAGEB, vt = kt + G::TILEB;
    f32x16 S[2], dP[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) S[rt][r] = 0.f;
    // instruction m: d-step c = m/4, key half rt = (m/2)%2, S (K tile) or dP (V tile) = m%2: four independent chains
    pipelined_mfma<4 * NC, PFD>(
        [&](int m) { return row_frag<D>((m & 1) ? vt : kt, m >> 2, (m >> 1) & 1, lane); },
        [&](int m, bf16x8 a) {
          const int c = m >> 2, rt = (m >> 1) & 1;
          if (m & 1) dP[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, dof[c], c == 0 ? minus_delta : dP[rt], 0, 0, 0);
          else S[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[c], S[rt], 0, 0, 0);
        });
    // dS^T = P^T * (dP^T - Delta), the difference formed by the sums above, packed to bf16 in the B-operand order of the next product
    u32x4 ds[4];
    // Only tiles that reach the diagonal or the end of the sequence need the mask (wavefront-uniform test); the
    // others skip the compares and selects.  Idle lanes (query beyond the sequence) carry lse = inf: P = 0.
    auto elements = [&](auto masked) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          float x[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            // computed for every element and selected afterwards: a conditional exponential becomes a branch
            const float pr = __builtin_amdgcn_exp2f(fmaf(S[rt][r + e], p.c2, -lse2));
            x[e] = pr * dP[rt][r + e];
            if (decltype(masked)::value) {
              const int key = key0 + 32 * rt + acc_row(r + e, hh);
              x[e] = (key <= tok32 && key < n32) ? x[e] : 0.f;
            }
          }
          const int rg = 16 * rt + r;
          ds[rg >> 3][(rg & 7) >> 1] = pack2(x[0], x[1]);
        }
    };
    if ((int64_t)key0 + KT - 1 > (int64_t)i * p.B + sl * 32 || (int64_t)key0 + KT > p.N) elements(std::true_type{});
    else elements(std::false_type{});
    pipelined_mfma<4 * ND, PFD>(
        [&](int m) { return tr_frag<D>(kt, m / ND, m % ND, lane); },
        [&](int m, bf16x8 a) {
          acc[m % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, ds[m / ND]), acc[m % ND], 0, 0, 0);
        });
  }
  wait_vmcnt<0>();

  // The sums that the dK/dV kernel, next on the stream, adds to with atomics start at zero: cleared here, a share per
  // workgroup.  (A kernel of its own for it, and items found with 64-bit divisions, gradients in us: 32 heads on 8, block 128,
  // N = 574 92.1 / 90.0, N = 131072 11456 / 11375; head_dim 64, block 64, N = 1000 47.1 / 45.4.)
  for (int64_t e = 4 * ((int64_t)blockIdx.x * (64 * NW) + tid); e < p.sink_floats; e += 4 * (int64_t)gridDim.x * (64 * NW))
    *reinterpret_cast<f32x4*>(p.dk_sink + e) = f32x4{0.f, 0.f, 0.f, 0.f};

  // element r of tile dt is d = 32dt + 8(r/4) + 4hh + r%4 of this lane's query row: 8-byte pieces
  if (ok) {
    __bf16* out = p.dq + qrow * D;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const u32x2 w = {pack2(acc[dt][4 * r4] * p.scale, acc[dt][4 * r4 + 1] * p.scale),
                         pack2(acc[dt][4 * r4 + 2] * p.scale, acc[dt][4 * r4 + 3] * p.scale)};
        *reinterpret_cast<u32x2*>(out + 32 * dt + 8 * r4 + 4 * hh) = w;
      }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// dK, dV
// ---------------------------------------------------------------------------------------------------------------
// The two halves of the work sit on different wavefronts: every 32-key slice has a wavefront that forms S and P and
// accumulates dV^T, and one that forms dP and dS and accumulates dK^T.  P travels through LDS, lane to same lane
// (both hold the same element layout), and the second wavefront runs one tile behind the first, so that the step's
// one barrier orders the exchange.  Each needs about 170 registers: two per SIMD, one of each kind.  (With both
// accumulators in one wavefront a lane needs 356 registers: one wavefront per SIMD, or spills.)
//
// A workgroup owns NSL slices (a slab of 32 NSL keys; a block of B keys is B / (32 NSL) slabs) and stages tiles of
// 32 QW QI queries: QW groups of wavefronts share a tile's 32-query pieces, QI pieces each, and add their sums up in
// LDS at the end.
//
// Bound: instruction issue (a SIMD issues about one instruction per 4 to 5 cycles, a matrix instruction lasts 32).  Per
// matrix instruction the kernel executes 7.9 instructions at blocks of 128 keys and head_dim 128, 8.7 at 256, 9.5 at 64
// (counters; 10.0 at 128 with a cursor each for copies and products, Delta subtracted element by element and a wait per
// matrix instruction).  Training steps with
// 32 query heads on 8 (28 on 4 at block 256), N = 32768: block 64 2.19 -> 1.98 ms, block 256 6.29 -> 4.65 ms (of which
// the kernel 3.9 -> 2.3); N = 2000, block 64: 232 -> 144 us, block 256: 766 -> 254 us.
template <int NSL, int QW, int QI, bool P32, int NST_>
struct dkv_geo {
  static constexpr int NW = 2 * NSL * QW;        // wavefronts
  static constexpr int TR = 32 * QW * QI;        // queries per tile
  static constexpr int PPIECE = P32 ? 4096 : 2048;       // P of a 32 x 32 piece, fp32 or bf16
  static constexpr int PBUF = NSL * QW * QI * PPIECE;    // P of one tile
  template <int D> static constexpr int tileb() { return TR / tile_geo<D>::RPI * tile_geo<D>::SRB; }
  template <int D> static constexpr int stageb() { return 2 * tileb<D>() + 8 * TR; }   // Q, dO, log-sum-exps, Deltas
  static constexpr int NST = NST_;               // tiles it+1 .. it+NST-2 arriving, tile it (P side), tile it-1 (dS side)
  template <int D> static constexpr size_t lds() { return NST * (size_t)stageb<D>() + 2 * (size_t)PBUF; }
};
// copy instruction x of a wavefront's share of a tile and, if BOTH, of the tile behind it
template <int D, int NW, int TILEB, bool BOTH>
__device__ __forceinline__ void dkv_copy(const __bf16* qb, const __bf16* ob, uint32_t voff, uint32_t dst, int x) {
  constexpr int STEP = NW * tile_geo<D>::SRB;
  static_assert(tile_geo<D>::IPT / NW <= 4, "the switch lists the copies");
  switch (x) {                                   // x is a constant wherever this is called (unrolled loops)
    case 0: async_copy16_at<0>(qb, voff, dst); if (BOTH) async_copy16_at<TILEB>(ob, voff, dst); break;
    case 1: async_copy16_at<STEP>(qb, voff, dst); if (BOTH) async_copy16_at<TILEB + STEP>(ob, voff, dst); break;
    case 2: async_copy16_at<2 * STEP>(qb, voff, dst); if (BOTH) async_copy16_at<TILEB + 2 * STEP>(ob, voff, dst); break;
    default: async_copy16_at<3 * STEP>(qb, voff, dst); if (BOTH) async_copy16_at<TILEB + 3 * STEP>(ob, voff, dst); break;
  }
}
template <int D, int NSL, int QW, int QI, bool P32, int NST_>
__global__ __launch_bounds__(128 * NSL * QW) __attribute__((amdgpu_waves_per_eu(2)))
void pa_bwd_dkv_kernel(bwd_params p) {
  using G = tile_geo<D>;
  using W = dkv_geo<NSL, QW, QI, P32, NST_>;
  constexpr int NW = W::NW, TR = W::TR, PBUF = W::PBUF, NST = W::NST;
  constexpr int NC = G::NC, ND = G::ND;
  constexpr int TILEB = W::template tileb<D>(), STAGEB = W::template stageb<D>();
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, hh = lane >> 5;
  const int kvh = blockIdx.y, b = blockIdx.z;
  const int slice = wave % NSL;
  const int qg = QW == 1 ? 0 : (wave / NSL) % QW;
  const bool krole = wave >= NSL * QW;           // false: S, P, dV^T; true: dP, dS, dK^T

  // ---- which slab of which key block, which part of its column ----
  int j, part;
  // the parts of the sink blocks' columns come first in the launch: they are the longest workgroups,
  // and the last ones to start should be the shortest
  const int slabs = p.B / (32 * NSL);
  const int slab = (int)blockIdx.x % slabs, e0 = (int)blockIdx.x / slabs;
  const int n_extra = p.sink_blocks * (p.max_parts - 1);
  if (e0 >= n_extra) { j = e0 - n_extra; part = 0; }
  else {
    j = e0 / (p.max_parts - 1);
    part = 1 + e0 % (p.max_parts - 1);
  }
  const bool whole_column = j < p.sink_blocks;                    // a sink block: every later query block
  const int parts = whole_column ? (p.nb - j + p.part - 1) / p.part : 1;
  if (part >= parts) return;                                      // uniform over the workgroup
  const int64_t slab0 = (int64_t)j * p.B + slab * (32 * NSL);     // its first key
  if (slab0 >= p.N) return;
  // entries of the column: query blocks j .. j+n_win-1, then j + 2^k for 2^k >= the window
  const int weff = (p.flags & POWATTN_POWER) ? (p.W > 1 ? p.W : 1) : p.W;
  int n_win, n_ent, first_pow = 1;
  if (whole_column) {
    n_win = p.nb - j - part * p.part;
    if (n_win > p.part) n_win = p.part;
    n_ent = n_win;
  } else {
    n_win = weff < p.nb - j ? weff : p.nb - j;
    n_ent = n_win;
    if (p.flags & POWATTN_POWER) {
      while (first_pow < weff && first_pow < p.nb) first_pow <<= 1;      // (a window above 2^30 has no power of two in 32 bits)
      for (int64_t pw = first_pow; j + pw < p.nb; pw <<= 1) ++n_ent;
    }
  }
  auto entry = [&](int e) -> int {
    if (whole_column) return j + part * p.part + e;
    if (e < n_win) return j + e;
    return j + (first_pow << (e - n_win));
  };

  // this lane's key; its K row (P side) or V row (dS side) as B operand
  const int64_t key = slab0 + 32 * slice + ln;
  const bool kok = key < p.N;
  const int key32 = (int)key, n32 = (int)p.N;          // positions fit 32 bits (checked by the host)
  const int64_t krow = ((int64_t)b * p.hkv + kvh) * p.N + (kok ? key : 0);
  bf16x8 xf[NC];

  f32x16 acc[ND];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[dt][r] = 0.f;

  // The tiles of the column in order: the tiles of a query block (those of the diagonal block that end before the
  // slab's first key are masked out entirely and left out), for each head of the group, for each entry of the column.
  // A SIMD issues about one instruction of any kind every 4 to 5 cycles, so the walk has to be short: one cursor, run
  // by the copies, moved on by additions; the products get a tile's first query handed on from the copies.
  const int tpb = p.B / TR;                                       // tiles per query block
  const int u_diag = slab * (32 * NSL) / TR;                      // first tile of the diagonal block
  const int n_tiles = n_ent * p.G * tpb - (part == 0 ? p.G * u_diag : 0);   // (the diagonal is the first entry of part 0)
  int c_e = 0, c_gg = 0, c_left = 0;             // entry, head of the group, tiles left of that head's
  int c_q0 = 0, c_first = 0, c_cnt = 0;          // first query of the tile; of the entry's first tile; tiles per head
  int64_t c_row = 0;                             // the tile's first row in [batch, hq, N]
  uint32_t c_stage = 0;
  auto enter = [&]() {                           // the first tile of the first head of entry c_e
    const int i = entry(c_e);
    const int u = i == j ? u_diag : 0;
    c_gg = 0;
    c_cnt = tpb - u;
    c_left = c_cnt;
    c_q0 = c_first = i * p.B + u * TR;
    c_row = ((int64_t)b * p.hq + (int64_t)kvh * p.G) * p.N + c_q0;
  };
  auto advance = [&]() {
    c_stage = c_stage == (NST - 1) * STAGEB ? 0u : c_stage + STAGEB;
    if (--c_left > 0) { c_q0 += TR; c_row += TR; return; }
    if (++c_gg < p.G) {
      c_row += n32 - (c_q0 - c_first);
      c_q0 = c_first;
      c_left = c_cnt;
    } else if (++c_e < n_ent) {
      enter();
    }
  };
  enter();
  // this lane's part of a tile copy that lies inside the sequence: byte offsets of its copy instructions, X apart
  // (copy instructions per wavefront and tile; with twice as many wavefronts as instructions the lower half of them
  // copies the Q tile and the upper half the dO tile)
  constexpr bool EITHER = 2 * (TR / G::RPI) == NW;
  constexpr int CPT = EITHER ? 1 : TR / G::RPI / NW;
  const int cw = EITHER ? wave % (NW / 2) : wave;
  uint32_t voff[CPT];
#pragma unroll
  for (int x = 0; x < CPT; ++x)
    voff[x] = (uint32_t)(G::RPI * (cw + NW * x) + lane % G::RPI) * G::ROWB + (uint32_t)((lane / G::RPI) << 4);
  const uint32_t w_dst = __builtin_amdgcn_readfirstlane(lds0 + cw * G::SRB + (EITHER && wave >= NW / 2 ? TILEB : 0));
  // The copies of the next tile; returns its first query.
  auto fill = [&]() -> int {
    const int q0 = c_q0;
    const __bf16* qb = uniform_ptr((EITHER && wave >= NW / 2 ? p.dout : p.q) + c_row * D);
    const __bf16* ob = uniform_ptr(p.dout + c_row * D);
    const uint32_t dst = w_dst + c_stage;
    const bool inside = q0 + TR <= n32;
    const int last = n32 - 1 - q0;               // rows beyond the sequence repeat its last row (masked where used)
    if (inside) {
#pragma unroll
      for (int x = 0; x < CPT; ++x) dkv_copy<D, NW, TILEB, !EITHER>(qb, ob, voff[x], dst, x);
    } else {
#pragma unroll
      for (int x = 0; x < CPT; ++x) {
        int row = G::RPI * (cw + NW * x) + lane % G::RPI;
        row = row < last ? row : last;           // (last may be negative: a tile that starts behind the sequence)
        const int64_t back = last < 0 ? last : 0;
        dkv_copy<D, NW, TILEB, !EITHER>(uniform_ptr(qb + back * D), uniform_ptr(ob + back * D),
                               (uint32_t)(row - (int)back) * G::ROWB + (uint32_t)((lane / G::RPI) << 4), dst, x);
      }
    }
    if (wave == 0) {
      // the tile's log-sum-exps and Deltas, copied asynchronously like the tiles (a load through registers would make
      // this wavefront wait for memory in every iteration)
      const uint32_t vdst = __builtin_amdgcn_readfirstlane(lds0 + c_stage + 2 * TILEB);
      int r = lane % TR;
      r = r < last ? r : last;
      if (TR == 32) {
        async_copy4((hh ? p.delta : p.lse2) + c_row + r, vdst);
      } else {
        async_copy4(p.lse2 + c_row + r, vdst);
        async_copy4(p.delta + c_row + r, vdst + 4 * TR);
      }
    }
    advance();
    return q0;
  };
  static_assert(TR == 32 || TR == 64, "a tile's vectors are one or two copy instructions");
  static_assert((TR / G::RPI) % NW == 0 || EITHER, "tile copies must divide over the wavefronts");
  // The mask matters where queries lie before the slab's last key, and where queries or keys run past the sequence: tiles
  // whose first query lies outside [m_lo, m_lo + m_span].
  int m_lo = (int)(slab0 + 32 * NSL < n32 ? slab0 + 32 * NSL : n32);
  uint32_t m_span = n32 - TR - m_lo > 0 ? (uint32_t)(n32 - TR - m_lo) : 0u;
  if (n32 - TR < m_lo || slab0 + 32 * NSL > p.N) { m_lo = 0x7fffffff; m_span = 0; }     // every tile
  const uint32_t pbase = lds0 + NST * STAGEB + (slice * QW + qg) * (QI * W::PPIECE) + lane * 16;

  // First queries of the tiles behind the one the P side works on; the copies run AHEAD tiles in front of it.
  constexpr int AHEAD = NST - 2;
  static_assert(AHEAD == 1 || AHEAD == 2, "one or two tiles on their way");
  int q_next = fill(), q_after = 0;
  if (AHEAD == 2 && n_tiles > 1) q_after = fill();
  // (after the first tile's copies: they would queue behind these row-per-lane loads)
  reg_rows<D>((krole ? p.v : p.k) + krow * D, kok, lane, xf);
  if (AHEAD > 1) {
    // Touched here, the compiler waits for them here, once.  Left to their first use, inside the loop, it puts a wait for
    // everything outstanding there, the copies just issued included.
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(xf[c]));
  }

  // in a tile with a mask: whether query qi attends this lane's key (key32 <= qi < n32, in one comparison)
  const uint32_t q_span = kok ? (uint32_t)(n32 - key32) : 0u;
  auto attended = [&](int qi) -> bool { return (uint32_t)(qi - key32) < q_span; };
  // One tile's products: piece by piece, S or dP, the elements, dV^T or dK^T.
  auto products = [&](auto role, auto masked_side, int q0, uint32_t stage, uint32_t pbuf) {
    constexpr bool KR = decltype(role)::value;
    const uint32_t qt = lds0 + stage, dot = qt + TILEB;
    const uint32_t vec = qt + 2 * TILEB;
#pragma unroll
    for (int x_ = 0; x_ < QI; ++x_) {
      const int half = QI * qg + x_;              // the 32-query piece of the tile
      f32x16 X;           // S on the P side, dP - Delta on the dS side
      u32x4 w[2];         // packed P (P side) or dS (dS side): the B operand of the second product
      const uint32_t vrow = vec + 4 * (32 * half + 4 * hh);          // this lane's rows of the vectors: +32 r4 bytes
      lds_u32x4* slot = (lds_u32x4*)(uintptr_t)(pbuf + x_ * W::PPIECE);
      u32x4 pr[P32 ? 4 : 2];
      if (KR) {
        // the accumulators start at -Delta of their rows
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 d4 = *(const lds_f32x4*)(uintptr_t)(vrow + 4 * TR + 32 * r4);
#pragma unroll
          for (int e = 0; e < 4; ++e) X[4 * r4 + e] = d4[e];
        }
#pragma unroll
        for (int x = 0; x < (P32 ? 4 : 2); ++x) pr[x] = slot[64 * x];      // P of the same elements, masked by its producer
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) X[r] = 0.f;
      }
      const uint32_t rows_from = KR ? dot : qt;
      if constexpr (NSL == 1) {
        // (one wavefront per SIMD: two sums of half the products each, or every product waits for the one before it)
        f32x16 X2;
#pragma unroll
        for (int r = 0; r < 16; ++r) X2[r] = 0.f;
        pipelined_mfma<NC, PFD>(
            [&](int m) { return row_frag<D>(rows_from, m, half, lane); },
            [&](int m, bf16x8 a) {
              if (m & 1) X2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf[m], X2, 0, 0, 0);
              else X = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf[m], X, 0, 0, 0);
            });
#pragma unroll
        for (int r = 0; r < 16; ++r) X[r] += X2[r];
      } else {
        pipelined_mfma<NC, PFD>(
            [&](int m) { return row_frag<D>(rows_from, m, half, lane); },
            [&](int m, bf16x8 a) { X = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf[m], X, 0, 0, 0); });
      }
      if (!KR) {
        auto elements = [&](auto masked) {
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 l4 = *(const lds_f32x4*)(uintptr_t)(vrow + 32 * r4);
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              // computed for every element and selected afterwards: a conditional exponential becomes a branch
              x[e] = __builtin_amdgcn_exp2f(fmaf(X[4 * r4 + e], p.c2, -l4[e]));
              if (decltype(masked)::value) x[e] = attended(q0 + 32 * half + 8 * r4 + 4 * hh + e) ? x[e] : 0.f;
            }
            const int r = 4 * r4;
            w[r >> 3][(r & 7) >> 1] = pack2(x[0], x[1]);
            w[r >> 3][((r & 7) >> 1) + 1] = pack2(x[2], x[3]);
            if (P32) slot[64 * r4] = __builtin_bit_cast(u32x4, f32x4{x[0], x[1], x[2], x[3]});
          }
        };
        if ((uint32_t)(q0 - m_lo) > m_span) elements(std::true_type{}); else elements(std::false_type{});
        if (!P32) {                                // lane l's 16-byte pieces at l*16, 1024 + l*16
          slot[0] = w[0];
          slot[64] = w[1];
        }
      } else {
        // (P is masked by its producer; 0 times a dP that is no number, where a query's row of O or dO is none, would not be 0)
        if (decltype(masked_side)::value) {
#pragma unroll
          for (int r = 0; r < 16; ++r) X[r] = attended(q0 + 32 * half + acc_row(r, hh)) ? X[r] : 0.f;
        }
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = 4 * r4 + e;
            uint32_t pk;
            if (P32) pk = pr[r >> 2][r & 3];
            else pk = (r & 1) ? (pr[r >> 3][(r & 7) >> 1] & 0xffff0000u) : (pr[r >> 3][(r & 7) >> 1] << 16);
            y[e] = __builtin_bit_cast(float, pk) * X[r];
          }
          const int r = 4 * r4;
          w[r >> 3][(r & 7) >> 1] = pack2(y[0], y[1]);
          w[r >> 3][((r & 7) >> 1) + 1] = pack2(y[2], y[3]);
        }
      }
      const uint32_t cols_from = KR ? qt : dot;
      pipelined_mfma<2 * ND, PFD>(
          [&](int m) { return tr_frag<D>(cols_from, 2 * half + m / ND, m % ND, lane); },
          [&](int m, bf16x8 a) {
            acc[m % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, w[m / ND]), acc[m % ND], 0, 0, 0);
          });
    }
  };
  // Iteration it: the P side works on tile it, the dS side on tile it-1 while the copies of tile it+1 are under way.
  // A loop per side with the same number of barriers.
  constexpr int CPF = CPT * (EITHER ? 1 : 2);      // copies of a fill; the first wavefront's vectors come on top
  auto top = [&](int it) {
    if (AHEAD == 1 || it + 1 >= n_tiles) wait_vmcnt<0>();
    else if (wave == 0) wait_vmcnt<CPF + (TR == 32 ? 1 : 2)>();    // (tile it+1 may still be on its way)
    else wait_vmcnt<CPF>();
    __syncthreads();      // tile it has landed; P of tile it-1 is in LDS; everybody is done with tile it-2
    if (AHEAD == 1) {
      if (it + 1 < n_tiles) q_next = fill();
    } else {
      q_next = q_after;
      if (it + 2 < n_tiles) q_after = fill();
    }
  };
  uint32_t stage = 0, pbuf = pbase;
  auto moved_on = [&]() {
    stage = stage == (NST - 1) * STAGEB ? 0u : stage + STAGEB;
    pbuf = pbuf == pbase ? pbase + PBUF : pbase;
  };
  if (!krole) {
    for (int it = 0; it < n_tiles; ++it) {
      const int q0 = q_next;
      top(it);
      products(std::false_type{}, std::false_type{}, q0, stage, pbuf);
      moved_on();
    }
    top(n_tiles);
  } else {
    // The tiles that need the mask are among those of the diagonal block, which comes first, and of the sequence's last
    // block; each range has a loop of its own (a test in every tile: +2 % at the 128K workload).
    int n_diag = part == 0 ? p.G * (tpb - u_diag) : 0;
    int n_last = n32 % p.B != 0 && entry(n_ent - 1) == p.nb - 1 ? p.G * tpb : 0;
    if (n_diag + n_last > n_tiles || slab0 + 32 * NSL > p.N) { n_diag = n_tiles; n_last = 0; }
    int q0 = q_next, it = 1;
    top(0);
    auto run = [&](auto masked_side, int to) {
      for (; it <= to; ++it) {
        const int q1 = q_next;
        top(it);
        products(std::true_type{}, masked_side, q0, stage, pbuf);
        q0 = q1;
        moved_on();
      }
    };
    int stop = n_diag;
    while (it <= n_tiles) {                      // (one copy of either loop, left at one place only: the sums stay in their registers)
      run(std::true_type{}, stop);
      run(std::false_type{}, n_tiles - n_last);
      stop = n_tiles;
    }
  }
  wait_vmcnt<0>();

  // the query groups' sums meet in LDS (the tiles are no longer needed), in a fixed order
  if constexpr (QW > 1) {
    static_assert(QW == 2 && (size_t)2 * NSL * ND * 4096 <= W::template lds<D>(), "one group hands its sums over");
    f32x16* sums = reinterpret_cast<f32x16*>(smem) + ((krole ? NSL : 0) + slice) * (ND * 64);
    __syncthreads();
    if (qg == 1) {
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)               // lane-contiguous 16-byte pieces
          reinterpret_cast<f32x4*>(sums)[(4 * dt + r4) * 64 + lane] = f32x4{acc[dt][4 * r4], acc[dt][4 * r4 + 1], acc[dt][4 * r4 + 2], acc[dt][4 * r4 + 3]};
    }
    __syncthreads();
    if (qg == 1) return;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 s4 = reinterpret_cast<const f32x4*>(sums)[(4 * dt + r4) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[dt][4 * r4 + e] += s4[e];
      }
  }

  if (!kok) return;
  const float f = krole ? p.scale : 1.0f;
  if (!whole_column) {
    __bf16* out = (krole ? p.dk : p.dv) + krow * D;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const u32x2 wv = {pack2(acc[dt][4 * r4] * f, acc[dt][4 * r4 + 1] * f), pack2(acc[dt][4 * r4 + 2] * f, acc[dt][4 * r4 + 3] * f)};
        *reinterpret_cast<u32x2*>(out + 32 * dt + 8 * r4 + 4 * hh) = wv;
      }
  } else {
    const int64_t srow = ((int64_t)b * p.hkv + kvh) * ((int64_t)p.sink_blocks * p.B) + key;
    float* sums = (krole ? p.dk_sink : p.dv_sink) + srow * D;
#pragma unroll
    for (int dt = 0; dt < ND; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) atomicAdd(sums + 32 * dt + acc_row(r, hh), acc[dt][r] * f);
  }
}

// the sink blocks' fp32 sums -> bf16 rows of dK and dV
template <int D>
__global__ __launch_bounds__(256) void pa_bwd_sink_store_kernel(bwd_params p, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;      // over [batch*hkv, sink_rows, D]
  if (e >= total) return;
  const int64_t sink_rows = (int64_t)p.sink_blocks * p.B;
  const int d = (int)(e % D);
  const int64_t key = (e / D) % sink_rows, bh = e / (D * sink_rows);
  if (key >= p.N) return;
  p.dk[(bh * p.N + key) * D + d] = (__bf16)p.dk_sink[e];
  p.dv[(bh * p.N + key) * D + d] = (__bf16)p.dv_sink[e];
}

template <int D, int NW>
int launch_dq(const bwd_params& p, int64_t items, hipStream_t stream) {
  constexpr size_t lds = dq_stages(NW) * 2 * (size_t)tile_geo<D>::TILEB;
  static std::atomic<unsigned long long> done{0};
  if (int st = pa_allow_dynamic_lds(reinterpret_cast<const void*>(&pa_bwd_dq_kernel<D, NW>), lds, done)) return st;
  hipLaunchKernelGGL((pa_bwd_dq_kernel<D, NW>), dim3((uint32_t)items), dim3(64 * NW), lds, stream, p);
  return pa_note_hip(hipGetLastError());
}
template <int D, int NSL, int QW, int QI, bool P32, int NST = 3>
int launch_dkv(const bwd_params& p, int batch, hipStream_t stream) {
  constexpr size_t lds = dkv_geo<NSL, QW, QI, P32, NST>::template lds<D>();
  static_assert(lds <= 160 * 1024, "LDS of a compute unit");
  const int64_t gx = ((int64_t)p.nb + (int64_t)p.sink_blocks * (p.max_parts - 1)) * (p.B / (32 * NSL));
  if (gx > 0x7fffffffLL) return POWATTN_UNSUPPORTED;
  const void* fn = reinterpret_cast<const void*>(&pa_bwd_dkv_kernel<D, NSL, QW, QI, P32, NST>);
  static std::atomic<unsigned long long> done{0};
  if (int st = pa_allow_dynamic_lds(fn, lds, done)) return st;
  hipLaunchKernelGGL((pa_bwd_dkv_kernel<D, NSL, QW, QI, P32, NST>), dim3((uint32_t)gx, (uint32_t)p.hkv, (uint32_t)batch),
                     dim3(128 * NSL * QW), lds, stream, p);
  return pa_note_hip(hipGetLastError());
}
// Which form of the kernel.  Training steps (forward and backward, 32 query heads on 8), MI355X:
//  * Where every 32-key slab has a compute unit: those, one wavefront per SIMD, and at head_dim 128 two tiles on their way
//    (there is LDS for four stages).  Gradients in us, 64-key slabs / these: head_dim 128, 32 heads on 8, block 128, N = 574
//    89.8 / 79.9, block 64, N = 1000 55.5 / 51.9; 16 on 2, N = 2000 107 / 92; head_dim 64, block 128, N = 600 58.9 / 54.8, but
//    block 64, N = 1000 (256 slabs) 45.7 / 48.2; with more workgroups than compute units (16 on 2, N = 4000) 129 / 143.
//  * Up to one 64-key slab per compute unit the length of a column decides: 64-key slabs, two query groups.  Against
//    one group: head_dim 128, N = 2000: block 64 0.139 / 0.149 ms, block 256 0.247 / 0.291; head_dim 64, N = 1000:
//    block 64 0.063 / 0.078, block 128 0.089 / 0.115, block 256 0.117 / 0.158.
//  * Blocks of 64 keys beyond that: one group, tiles of 32 queries, two or three workgroups per compute unit that are
//    not in step with each other.  Against two groups: head_dim 128, N = 32768: 2.03 / 2.13 ms; head_dim 64: 1.21 / 1.26.
//  * head_dim 128, larger blocks: 128-key slabs, which read the query tiles half as often (64-key slabs: block 128,
//    N = 131072 15.4 ms against 14.5).  At blocks of 128 keys P goes from wavefront to wavefront in bf16 and the tiles are
//    64 queries; at 256 it goes in fp32, which leaves room for tiles of 32 (block 256, N = 32768: 4.85 ms; block 128,
//    N = 131072: 14.8 ms).
//  * head_dim 64, larger blocks: 128-key slabs and two groups, sixteen wavefronts.  Against one group with tiles of 64
//    and 64-key slabs: block 256, N = 32768 3.13 / 3.34 / 3.36 ms, N = 4000 0.317 / 0.345 / 0.351.
template <int D>
int launch_dkv_any(const bwd_params& p, int batch, hipStream_t stream) {
  int n_cu = 1;
  pa_current_device(nullptr, &n_cu);
  const int64_t slabs64 = (int64_t)p.nb * (p.B / 64) * p.hkv * batch;
  const int64_t parts = p.sink_blocks > 0 ? (p.nb + p.part - 1) / p.part : 1;       // of the longest sink column
  const int64_t wgs32 = (p.nb + p.sink_blocks * (parts - 1)) * (p.B / 32) * p.hkv * batch;
  if (D == 128 && wgs32 <= n_cu) return launch_dkv<D, 1, 2, 1, true, 4>(p, batch, stream);
  if (D == 64 && 4 * wgs32 <= 3 * n_cu) return launch_dkv<D, 1, 2, 1, true, 3>(p, batch, stream);
  if (slabs64 <= n_cu) return launch_dkv<D, 2, 2, 1, true>(p, batch, stream);
  if (p.B == 64) return launch_dkv<D, 2, 1, 1, true>(p, batch, stream);
  if constexpr (D == 64) return launch_dkv<D, 4, 2, 1, true>(p, batch, stream);
  else return p.B == 128 ? launch_dkv<D, 4, 1, 2, false>(p, batch, stream) : launch_dkv<D, 4, 1, 1, true>(p, batch, stream);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t pa_backward_workspace_bytes(const powattn_pattern& pat, int32_t batch, int32_t hq, int32_t hkv, int64_t seq_len, int32_t head_dim) {
  const int64_t nb = (seq_len + pat.block - 1) / pat.block;
  const int64_t sink_rows = (pat.sink < nb ? pat.sink : nb) * (int64_t)pat.block;
  return 2 * align256((size_t)batch * hq * seq_len * sizeof(float)) +
         2 * align256((size_t)batch * hkv * sink_rows * head_dim * sizeof(float));
}

int pa_launch_backward_bf16(const pa_backward_args& a) {
  bwd_params p;
  p.q = (const __bf16*)a.q; p.k = (const __bf16*)a.k; p.v = (const __bf16*)a.v; p.o = (const __bf16*)a.o;
  p.dout = (const __bf16*)a.dout; p.lse = a.lse;
  p.dq = (__bf16*)a.dq; p.dk = (__bf16*)a.dk; p.dv = (__bf16*)a.dv;
  p.kv_cnt = a.kv_cnt; p.kv_idx = a.kv_idx; p.max_k = a.max_k; p.nb = a.nb;
  p.B = a.pat.block; p.W = a.pat.window; p.S = a.pat.sink; p.flags = a.pat.flags;
  p.hq = a.hq; p.hkv = a.hkv; p.G = a.hq / a.hkv; p.subs = p.B / KT;
  p.N = a.seq_len; p.scale = a.scale; p.c2 = a.scale * LOG2E;
  if ((int64_t)a.max_k * p.subs > TILE_CAP) return POWATTN_UNSUPPORTED;
  if (a.seq_len > 0x7fffffffLL - 1024) return POWATTN_UNSUPPORTED;
  if (p.B > 256) return POWATTN_UNSUPPORTED;                       // a wavefront per 32 keys of the block, at most 8
  if (a.batch > 65535 || a.hkv > 65535) return POWATTN_UNSUPPORTED;
  const int64_t tasks = (int64_t)p.G * p.B / 32;
  if (tasks > (1 << 20)) return POWATTN_UNSUPPORTED;
  p.tasks = (int32_t)tasks;
  // eight wavefronts per workgroup when a query block has that many tasks and blocks of 128 keys or more; at
  // blocks of 64 keys four (two workgroups per compute unit that are not in step with each other: 4-7 % faster
  // at configuration 2's shape than one workgroup of eight)
  // ... and where there is a compute unit for every workgroup of four (gradients of one sequence, eight / four, us:
  // block 128, 32 heads on 8, N = 500 88.0 / 79.9, N = 1000 105.2 / 95.9; block 256, 8 on 8, N = 2000 114.9 / 99.8)
  int n_cu = 1;
  pa_current_device(nullptr, &n_cu);
  const bool few = (int64_t)a.batch * a.hkv * a.nb * ((p.tasks + 3) / 4) <= n_cu;
  const int nwq = (p.tasks > 4 && p.B >= 128 && !few) ? 8 : 4;
  p.chunks = (p.tasks + nwq - 1) / nwq;
  p.sink_blocks = a.pat.sink < a.nb ? a.pat.sink : a.nb;
  p.part = pa_sink_part(a.nb, p.sink_blocks, p.W, p.flags, (int64_t)a.hkv * a.batch, p.G, p.B);
  p.max_parts = p.sink_blocks > 0 ? (a.nb + p.part - 1) / p.part : 1;
  if (p.max_parts < 2) p.max_parts = 2;                            // keeps the part arithmetic of the kernel defined

  // workspace: Delta, the log-sum-exp in base 2, then the sink blocks' sums
  unsigned char* ws = (unsigned char*)a.workspace;
  p.delta = (float*)ws;
  ws += align256((size_t)a.batch * a.hq * a.seq_len * sizeof(float));
  p.lse2 = (float*)ws;
  ws += align256((size_t)a.batch * a.hq * a.seq_len * sizeof(float));
  const int64_t sink_elems = (int64_t)a.batch * a.hkv * p.sink_blocks * p.B * a.head_dim;
  p.dk_sink = (float*)ws;
  ws += align256((size_t)sink_elems * sizeof(float));
  p.dv_sink = (float*)ws;

  int st = POWATTN_OK;
  p.sink_floats = sink_elems > 0 ? 2 * (int64_t)(align256((size_t)sink_elems * sizeof(float)) / sizeof(float)) : 0;

  const int64_t items = (int64_t)a.batch * a.hkv * a.nb * p.chunks;
  if (items > 0x7fffffffLL) return POWATTN_UNSUPPORTED;
  if (a.head_dim == 128) st = nwq == 8 ? launch_dq<128, 8>(p, items, a.stream) : launch_dq<128, 4>(p, items, a.stream);
  else st = nwq == 8 ? launch_dq<64, 8>(p, items, a.stream) : launch_dq<64, 4>(p, items, a.stream);
  if (st != POWATTN_OK) return st;

  st = a.head_dim == 128 ? launch_dkv_any<128>(p, a.batch, a.stream) : launch_dkv_any<64>(p, a.batch, a.stream);
  if (st != POWATTN_OK) return st;

  if (sink_elems > 0) {
    const int64_t sb = (sink_elems + 255) / 256;
    if (a.head_dim == 128)
      hipLaunchKernelGGL((pa_bwd_sink_store_kernel<128>), dim3((uint32_t)sb), dim3(256), 0, a.stream, p, sink_elems);
    else
      hipLaunchKernelGGL((pa_bwd_sink_store_kernel<64>), dim3((uint32_t)sb), dim3(256), 0, a.stream, p, sink_elems);
    st = pa_note_hip(hipGetLastError());
  }
  return st;
}
