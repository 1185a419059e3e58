// Split-K decode: one query token per sequence attends its KV cache under the
// prefill pattern (Section 4.1: the same pattern in both phases).  The query
// sits at t = kv_len-1; the attended block list of row floor(t/B) comes from
// the closed form of Algorithm 1, inside the kernel.
//
// The step reads 2*D*2 bytes per attended token and does a handful of flops
// with them: it is bound by HBM bandwidth and latency, so the kernel is built
// around having every byte in flight at once and keeping the dependent chain
// after the loads short.
//
//  * A workgroup of 8 wavefronts owns one (sequence, KV head[, split]).  The
//    attended tokens are cut into 64-token chunks, dealt round-robin to the
//    splits and their wavefronts; a wavefront issues all K and V loads of a
//    chunk before touching any.  What stands between the sequence length and the first of them is scalar and 32 bits
//    wide, and the loads are buffer loads, which answer zeros beyond the last attended token: no address or comparison per
//    load.  (One sequence, 32 query heads on 8, 32001 tokens: 9.8 us -> 8.1 with the two changes below; 128 of 1000 .. 16384
//    tokens over pages, persistent workgroups: 66.9 -> 64.4.)
//  * Everything stays in registers.  K rows are loaded straight into the
//    A-operand layout of v_mfma_f32_16x16x32_bf16 (S^T = K q^T, the G query
//    heads of the group are the 16 columns, unused ones zero).  V is loaded
//    fully coalesced as 8 tokens x 8 d per lane and transposed inside the lane
//    (32 byte-permutes per 8x8 block) into the A operand of O^T += V^T P^T.
//    The K rows are fetched in a permuted token order chosen so that the
//    accumulator layout of S^T is the B-operand layout of the second product.
//  * Each wavefront keeps a running (max, sum, O) over its chunks; the eight
//    partials meet in LDS.  With one workgroup per (sequence, KV head) that is
//    the result; with several, every workgroup leaves its unnormalised partial
//    in the workspace as tagged 8-byte packets, waits until memory has taken
//    them, and then reads the packets of the other workgroups: the one whose
//    packets landed last finds all of them in place and writes the output
//    (with many splits a merge kernel does that instead).  The wavefronts' partials are read for the wavefronts that have
//    a chunk, and the weights of the splits do not wait for one another.  There are no
//    counters and nothing in the workspace has to be initialised: a packet
//    is valid when its tag matches the generation number that the (sequence,
//    KV head) keeps in the workspace and that the finishing workgroup advances.
//    Packet stores and loads act at device scope by themselves; no fence is
//    used, because a device-scope fence writes back and invalidates a whole L2
//    on this chip.
//  * With several work items per compute unit (large batches) persistent
//    workgroups take over (pa_decode_stream_kernel): the loads of the next item
//    are in flight while the current one is merged.
#include <math.h>
#include <type_traits>
#include "common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int CH = 64;         // tokens per chunk
constexpr int NW = 8;          // wavefronts per workgroup
constexpr int MAXG = 16;       // query heads per KV head (columns of the MFMA tile)

struct dec_params {
  const __bf16* q; const __bf16* k; const __bf16* v; const int32_t* kv_len;
  __bf16* o; float* lse;
  float* partials;      // [batch, hq, splits, D + 2] floats when splits > 1 and a merge kernel follows
  uint64_t* packets;    // the same shape as (value, tag) packets when the workgroups merge among themselves
  uint32_t* gen;        // [batch, hkv] generation numbers of the packets (any initial value)
  int64_t capacity;
  int32_t len_max;      // the capacity, or the largest sequence length that there is
  int32_t B, W, S; uint32_t flags;
  int32_t hq, hkv, G, splits, subs;
  uint32_t subs_magic;  // ceil(2^32 / subs) for subs > 1: slot / subs = umulhi(slot, subs_magic) for every slot of a row
  uint32_t per_b_magic; // persistent workgroups: ceil(2^32 / items of a sequence) where that replaces the division of any item's number (else 0)
  int32_t kvh_first;    // 1: the KV head is the fastest digit of a workgroup's number, 0: the split
  int32_t through;      // 1: packets are taken back with stores that go through to memory
  int32_t fused;        // 1: the workgroups of a (sequence, KV head) merge their partials among themselves
  float c2;
  const int32_t* block_table;   // paged cache: page of block j of sequence b at [b * table_stride + j]; else null
  int32_t table_stride;
  int32_t last_page;            // the pool's last page (that an entry of the table can name)
};

// ---- merging the workgroups of a (sequence, KV head) without a second kernel ----
// Every value of a partial result travels as one 8-byte packet (value, tag), written and read with single 8-byte
// device-scope accesses, so a reader sees a value together with its tag or not at all.  The tag is derived from the
// generation number g that the (sequence, KV head) keeps in the workspace, read at the start of the kernel, and from
// the split.  Protocol of a workgroup: store its packets; wait until memory has acknowledged every one of them
// (s_waitcnt, then the workgroup's barrier); load the packets of the other splits; if every tag is the expected one,
// combine all partials in split order, write the output and store g + 1 as the new generation.
//  * Some workgroup finishes: order the workgroups by the time at which the last of their stores was acknowledged;
//    the latest one loads after that, when every other workgroup's packets are in memory.
//  * Several may finish: they combine the same values in the same order and write the same bits.  (Each thread decides for
//    the outputs it owns: a vote of the workgroup took another 0.6 us.)
//  * Nothing stale is taken for valid.  An output's packet is taken back by the thread that used it (its tag becomes 0, and
//    a valid one is odd): no call leaves one behind, whatever the memory is used for before it is a workspace again, its
//    words g put back to old ones included, and also where a graph replays the launch.  Maxima and sums are shared by the
//    threads of a head and stay; those of the call before carry generation g - 1 (the finisher advanced it only after every
//    workgroup of the pair had stored packets, hence all of its wavefronts had read g, before the barrier in front of its
//    stores), and older ones whose generation is back do not fit the output's packet, whose tag is formed with the bits of
//    the maximum and the sum that go with it.  The very first call on a workspace meets whatever the memory held: a word
//    there passes for the tag of a maximum only if it equals ~g ^ ((split + 1) << 24) for the word g found in the same
//    memory (never for a memory filled with one byte value, zeros included).
//  * No workgroup waits for another one: whoever finds a packet missing simply leaves.  (A look before the acknowledgement
//    may find everything in place already; only the one after it has to be there.)
// Calls that may run at the same time must not share a workspace (they would share generation numbers).
// With more splits than this a merge kernel follows: what a workgroup reads grows with their number.  us, merged among
// themselves / by the kernel, 32 query heads on 8: 7 splits, batch 2 10.35 / 8.9, 5 19.8 / 15.2 (batch 1 level); 8 splits, batch 4,
// 29 chunks 12.3 / 10.9, 62 chunks 18.2 / 15.7, batch 8 37.8 / 32.5, 128 heads on 8 24.2 / 13.5.  Up to 6 the kernel's time on the
// GPU is no longer either (6 splits, batch 1 8.7 / 7.85), but its launch takes the host longer than the step takes the GPU:
// launched from Python, one after another, such steps were paced at 8.7 to 9.1 us on some hosts.
constexpr int MAX_FUSED_SPLITS = 6;
__device__ __forceinline__ uint32_t dec_tag(uint32_t gen, int split) { return ~gen ^ ((uint32_t)(split + 1) << 24); }
// ... of an output: with the maximum and the sum of its head; odd
__device__ __forceinline__ uint32_t dec_tag_of_output(uint32_t tag, uint32_t m_bits, uint32_t l_bits) {
  return (tag ^ m_bits ^ (l_bits << 16 | l_bits >> 16)) | 1u;
}
__device__ __forceinline__ void dec_put(uint64_t* slot, float x, uint32_t tag) {
  __hip_atomic_store(slot, ((uint64_t)tag << 32) | __builtin_bit_cast(uint32_t, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The launch that has to see it is a later one, so an ordinary store is enough; where the launch fills the chip, it is better
// written through at once than left for the end of the kernel (us, 32 query heads on 8, not taken back / ordinary / through:
// batch 1 7.9 / 8.0 / 8.4, batch 4 9.05 / 9.05 / 9.32, batch 16 12.15 / 12.75 / 12.21; 28 on 4, ordinary: batch 2 9.4 / 9.9, 4
// 10.15 / 10.6; all of them at the end of the kernel instead: 0 to 0.5 more).
template <int SCOPE>
__device__ __forceinline__ void dec_take_back(uint64_t* first, int splits, int stride) {
#pragma unroll
  for (int y = 0; y < MAX_FUSED_SPLITS; ++y)
    if (y < splits) __hip_atomic_store(first + (int64_t)y * stride, (uint64_t)0, __ATOMIC_RELAXED, SCOPE);
}
__device__ __forceinline__ uint64_t dec_get(const uint64_t* slot) {
  return __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// LDS layout of the wavefronts' partial outputs: the 32 values a lane holds (d = 32*q4 + x) form a row of 36 floats,
// so that the 16 lanes of a store (4 heads x 4 groups) start 36 floats apart and cover all banks between them.
constexpr int OROW = 36;
template <int D>
__device__ __forceinline__ int dec_o_at(int wave, int G, int g, int d) { return (((wave * G + g) * (D / 32) + (d >> 5)) * OROW) + (d & 31); }
template <int D>
constexpr size_t dec_o_bytes(int G) { return (size_t)NW * G * (D / 32) * OROW * sizeof(float); }

// The query's row of the pattern in closed form: [0, sink_end) ++ {i - 2^k inside [pow_lo, win_start), k
// descending} ++ [win_start, i].  Uniform over a workgroup, so all of it runs on the scalar unit, and it stands between
// the sequence length and the first load: positions are 32-bit numbers (as the lengths are), half the instructions.
struct dec_row {
  pa_row_shape_t<int32_t> rs;
  int32_t t, i;          // position of the query, its block
  int n_pow, k_max;      // isolated blocks i - 2^k for k = k_max, k_max-1, ...: n_pow of them
  int n_slots;           // 64-token chunks of the attended blocks
};
__device__ __forceinline__ dec_row dec_row_of(const dec_params& p, int32_t len) {
  dec_row r;
  if (len < 1) len = 1;
  if (len > p.len_max) len = p.len_max;
  r.t = len - 1;
  // t / B = (t / 64) / subs: exact through the multiply-high, because t / 64 stays below 2^25
  static_assert(CH == 64, "the block index is formed from 64-token chunks");
  const unsigned chunk_of_t = (unsigned)r.t >> 6;
  r.i = p.subs == 1 ? (int)chunk_of_t : (int)__umulhi(chunk_of_t, p.subs_magic);
  r.rs = pa_shape_of_row<int32_t>(p.W, p.S, p.flags, r.i);
  const pa_row_powers pw = pa_powers_of_row<int32_t>(r.rs, p.flags, r.i);
  r.n_pow = pw.n_pow; r.k_max = pw.k_max;
  const int n_blocks = r.rs.sink_end + r.n_pow + (r.i - r.rs.win_start + 1);
  r.n_slots = n_blocks * p.subs;
  return r;
}
__device__ __forceinline__ int32_t dec_block_at(const dec_row& r, int lp) {   // lp-th attended block, ascending
  if (lp < r.rs.sink_end) return lp;
  lp -= r.rs.sink_end;
  if (lp >= r.n_pow) return r.rs.win_start + (lp - r.n_pow);
  return r.i - (1 << (r.k_max - lp));
}
// Chunk `slot` of the row: its block, the chunk inside the block, the tokens of it the query attends (<= 0: none)
struct dec_place { int32_t blk; int sub; int n_tok; };
__device__ __forceinline__ dec_place dec_place_of(const dec_params& p, const dec_row& r, int slot) {
  // (no division in the kernel: a 64-bit one costs more than the rest of the address arithmetic)
  dec_place c;
  const int lp = p.subs == 1 ? slot : (int)__umulhi((unsigned)slot, p.subs_magic);
  c.sub = slot - lp * p.subs;
  c.blk = dec_block_at(r, lp);
  const int left = (r.t - c.blk * p.B) - c.sub * CH + 1;      // causal: tokens tok0..t are attended
  c.n_tok = left >= CH ? CH : left;
  return c;
}
// First K and V row of a chunk: in the contiguous cache, or in its page (page numbers outside the pool are clamped
// into it: a bad table gives wrong numbers, never an access outside the pool)
__device__ __forceinline__ int64_t dec_chunk_offset(const dec_params& p, int b, int kvh, const dec_place& c, int page, int D) {
  if (!p.block_table) return (((int64_t)b * p.hkv + kvh) * p.capacity + (int64_t)(c.blk * p.B + c.sub * CH)) * D;
  page = page < 0 ? 0 : (page > p.last_page ? p.last_page : page);
  return (((int64_t)page * p.hkv + kvh) * p.B + c.sub * CH) * D;
}
// the table's entry for block `blk`, through the scalar unit (the table does not change while a kernel runs)
__device__ __forceinline__ int dec_page(const dec_params& p, int b, int blk) {
  typedef const __attribute__((address_space(4))) int32_t scalar_int;
  return *(scalar_int*)(uintptr_t)(p.block_table + (int64_t)b * p.table_stride + blk);
}

// The registers of one 64-token chunk: every load of it is issued before any is used.
template <int D>
struct dec_chunk {
  u32x4 kraw[CH / 16][D / 32];
  u32x4 vraw[CH / 32][8];
};
// A buffer of `bytes` bytes from `base` on (uniform): loads beyond its end return zeros, so the rows behind the last
// attended token and the heads behind the group's last one need no comparison, no branch and no register of their own.
typedef __amdgpu_buffer_rsrc_t dec_buf;
__device__ __forceinline__ dec_buf dec_buffer(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 dec_load16(dec_buf buf, int lane_offset, int offset) {
  return __builtin_amdgcn_raw_buffer_load_b128(buf, lane_offset + offset, 0, 0);
}
// K tile 2x+y, row rho = lane%16 holds token 32x + 8(rho/4) + 4y + rho%4: with this order the S^T
// accumulator of lane (g, q4) holds tokens 32x + 8*q4 + (0..7), which is what P^T must supply below.
// V: lane (dg = lane%16, tg = lane/16) takes tokens 32x + 8tg + (0..7), d = 8dg .. 8dg+7.
// A lane's address is one register and an immediate offset below 4096 bytes: a buffer per 32 tokens.
template <int D>
__device__ __forceinline__ void dec_issue(dec_chunk<D>& c, const __bf16* kb, const __bf16* vb, int n_tok, int g, int q4) {
  constexpr int NC = D / 32, CPR = D / 8, ROW = 2 * D;
  const int k_lane = (8 * (g >> 2) + (g & 3)) * ROW + 16 * q4;
  const int v_lane = g < CPR ? 8 * q4 * ROW + 16 * g : 32 * ROW;      // (head_dim 64: half the lanes have no piece of a row)
#pragma unroll
  for (int x = 0; x < CH / 32; ++x) {
    const int left = n_tok - 32 * x;
    const dec_buf buf = dec_buffer(kb + 32 * x * D, (left < 0 ? 0 : left > 32 ? 32 : left) * ROW);
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) c.kraw[2 * x + y][cc] = dec_load16(buf, k_lane, 4 * y * ROW + 64 * cc);
  }
#pragma unroll
  for (int x = 0; x < CH / 32; ++x) {
    const int left = n_tok - 32 * x;
    const dec_buf buf = dec_buffer(vb + 32 * x * D, (left < 0 ? 0 : left > 32 ? 32 : left) * ROW);
#pragma unroll
    for (int r = 0; r < 8; ++r) c.vraw[x][r] = dec_load16(buf, v_lane, r * ROW);
  }
  __builtin_amdgcn_sched_barrier(0);                   // every load is under way before the first product
}
// One online-softmax update with the chunk: S^T = K q^T, then O^T += V^T P^T.  FIRST: nothing has been accumulated yet.
template <int D, bool FIRST>
__device__ __forceinline__ void dec_consume(const dec_chunk<D>& c, const bf16x8 (&qf)[D / 32], int n_tok, float c2, int q4,
                                            float& m_run, float& l_run, f32x4 (&O)[8]) {
  constexpr int NC = D / 32, NT = CH / 16;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 S[NT];
#pragma unroll
  for (int tau = 0; tau < NT; ++tau) {
    S[tau] = zero;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc)
      S[tau] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, c.kraw[tau][cc]), qf[cc], S[tau], 0, 0, 0);
  }
  // ---- online softmax; S[2x+y][r] is token 32x + 8*q4 + 4y + r of head g ----
  if (n_tok < CH) {                                   // uniform: the sequence's last chunk
#pragma unroll
    for (int tau = 0; tau < NT; ++tau)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int tk = 32 * (tau >> 1) + 8 * q4 + 4 * (tau & 1) + r;
        S[tau][r] = tk < n_tok ? S[tau][r] : -INFINITY;
      }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int tau = 0; tau < NT; ++tau)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      S[tau][r] *= c2;
      mx = fmaxf(mx, S[tau][r]);
    }
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));                // finite: token 0 of the chunk is attended
  const float m_new = FIRST ? mx : fmaxf(m_run, mx);
  const float alpha = FIRST ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
  m_run = m_new;
  float rowsum = 0.f;
#pragma unroll
  for (int tau = 0; tau < NT; ++tau)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      S[tau][r] = __builtin_amdgcn_exp2f(S[tau][r] - m_new);
      rowsum += S[tau][r];
    }
  l_run = FIRST ? rowsum : l_run * alpha + rowsum;
  if (!FIRST) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) O[j][r] *= alpha;
  }

  // ---- O^T += V^T P^T: 32 tokens per step; MFMA j covers d = 8*row + j ----
#pragma unroll
  for (int x = 0; x < CH / 32; ++x) {
    bf16x8 pf;
#pragma unroll
    for (int e = 0; e < 8; ++e) pf[e] = (__bf16)S[2 * x + (e >> 2)][e & 3];
    // transpose the lane's 8 tokens x 8 d block: pairs of tokens share a dword
    uint32_t tr[4][8];                                // tr[a][d]: tokens 2a, 2a+1 at d
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int kd = 0; kd < 4; ++kd) {
        const uint32_t r0 = c.vraw[x][2 * a][kd], r1 = c.vraw[x][2 * a + 1][kd];
        tr[a][2 * kd] = __builtin_amdgcn_perm(r1, r0, 0x05040100u);       // low halves: d = 2kd
        tr[a][2 * kd + 1] = __builtin_amdgcn_perm(r1, r0, 0x07060302u);   // high halves: d = 2kd+1
      }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const u32x4 vf = {tr[0][j], tr[1][j], tr[2][j], tr[3][j]};
      O[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf), pf, FIRST && x == 0 ? zero : O[j], 0, 0, 0);
    }
  }
}
// q^T fragments: column g, 8 consecutive d per 32-wide step (columns behind the group's last head: zeros)
template <int D>
__device__ __forceinline__ void dec_load_q(bf16x8 (&qf)[D / 32], const dec_params& p, int b, int kvh, int g, int q4) {
  const dec_buf buf = dec_buffer(p.q + ((int64_t)b * p.hq + (int64_t)kvh * p.G) * D, p.G * 2 * D);
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
    qf[c] = __builtin_bit_cast(bf16x8, dec_load16(buf, g * 2 * D + 16 * q4, 64 * c));
}

// The lane number, computed afresh wherever it is called: the compiler cannot carry the value of an earlier call
// over, so nothing derived from it has to stay in (or be spilled from) a register across the chunk loads and the
// matrix products, where every register counts.  (A spilled register in the persistent kernel is reloaded behind
// the next chunk's loads and has to wait for all of them.)
__device__ __forceinline__ int dec_lane_now() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// The wavefront's partial output into LDS: lane (g, q4) holds O[j][r] = o[g][d = 32*q4 + 8r + j], eight
// consecutive d per r, written as two 16-byte stores into the lane's padded row.
template <int D>
__device__ __forceinline__ void dec_stash(float* s_o, int wave, int G, int g, int q4, const f32x4 (&O)[8]) {
  if (32 * q4 >= D) return;
  f32x4* row = reinterpret_cast<f32x4*>(s_o + dec_o_at<D>(wave, G, g, 32 * q4));
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    row[2 * r] = f32x4{O[0][r], O[1][r], O[2][r], O[3][r]};
    row[2 * r + 1] = f32x4{O[4][r], O[5][r], O[6][r], O[7][r]};
  }
}

// EPT: outputs per thread (the G x D values of the group over the workgroup's threads)
template <int D, int EPT>
__global__ __launch_bounds__(64 * NW) void pa_decode_kernel(dec_params p) {
  __shared__ float s_m[NW][MAXG], s_l[NW][MAXG];
  extern __shared__ __attribute__((aligned(16))) float s_o_dyn[];   // [NW][G][D/32][OROW] partial outputs of the wavefronts

  const int kvh = p.kvh_first ? blockIdx.x : blockIdx.y, split = p.kvh_first ? blockIdx.y : blockIdx.x, b = blockIdx.z;
  // the wavefront's number as a scalar and the lane from the hardware's lane count: the thread index itself need
  // not stay in a vector register through the chunk loop, where every register counts
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int g = lane & 15, q4 = lane >> 4;    // column (query head) and k-group of this lane

  // Every kernel argument that stands before the loads is asked for at once, with one wait (left alone, the compiler
  // fetches them in four groups, a trip to memory each).
  asm volatile("" ::"s"(p.q), "s"(p.k), "s"(p.kv_len), "s"(p.gen), "s"(p.capacity), "s"(p.len_max), "s"(p.splits), "s"(p.subs),
               "s"(p.subs_magic), "s"(p.block_table), "s"(p.table_stride), "s"(p.last_page));
  // The sequence length and the generation of this (sequence, KV head)'s packets (needed only at the end) are
  // both uniform: two scalar loads, one wait.  Written as assembly so that the generation number lives in a
  // scalar register from the start (a vector register held across the chunk loop costs a spill to scratch
  // memory, and a kernel that uses scratch memory starts later).  Both words were written before this kernel
  // started, so the scalar cache, which is empty at the start of a kernel, returns what memory holds.
  uint32_t gen;
  int len_b;
  asm volatile("s_load_dword %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(gen), "=&s"(len_b)
               : "s"(p.gen + (int64_t)b * p.hkv + kvh), "s"(p.kv_len + b)
               : "memory");

  bf16x8 qf[D / 32];
  dec_load_q<D>(qf, p, b, kvh, g, q4);
  const dec_row row = dec_row_of(p, len_b);
  const int n_slots = row.n_slots;

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 O[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) O[j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // chunks are dealt round-robin to the splits (slot = wave * splits + split), so that the workgroups of a
  // (sequence, KV head) stream nearly equal amounts (13 chunks over 2 workgroups: 7 + 6 instead of 8 + 5)
  auto chunk = [&](int slot, auto first) {
    const dec_place pl = dec_place_of(p, row, slot);
    if (pl.n_tok <= 0) return;                           // chunk of the diagonal block beyond the query
    // paged cache: the block's page comes from the table (one more dependent look-up; blk < table_stride,
    // because len <= table_stride * B); a page holds the block's tokens of every KV head
    const int page = p.block_table ? dec_page(p, b, pl.blk) : 0;
    const int64_t off = dec_chunk_offset(p, b, kvh, pl, page, D);
    dec_chunk<D> c;
    dec_issue<D>(c, p.k + off, p.v + off, pl.n_tok, g, q4);
    dec_consume<D, decltype(first)::value>(c, qf, pl.n_tok, p.c2, q4, m_run, l_run, O);
  };
  int slot = wave * p.splits + split;
  if (slot < n_slots) chunk(slot, std::true_type{});
  // (mostly one chunk per wavefront.  A diagonal chunk without a token can only be a wavefront's last one.)
  while ((slot += p.splits * NW) < n_slots) chunk(slot, std::false_type{});

  // ---- merge the wavefronts through LDS: those that have a chunk ----
  auto has_chunk = [&](int w) -> bool { return w * p.splits + split < n_slots; };
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (g < p.G) {
    if (q4 == 0) { s_m[wave][g] = m_run; s_l[wave][g] = l_run; }
    dec_stash<D>(s_o_dyn, wave, p.G, g, q4, O);
  }
  __syncthreads();

  // thread e owns output (head gg, component d); with many heads per KV head a thread owns several
  const int tid = wave * 64 + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  float accs[EPT], Ms[EPT], Ls[EPT];
#pragma unroll
  for (int x = 0; x < EPT; ++x) {
    const int e = tid + x * 64 * NW;
    accs[x] = 0.f; Ms[x] = -INFINITY; Ls[x] = 0.f;
    if (e >= p.G * D) continue;
    const int gg = e / D, d = e % D;
    float M = -INFINITY, L = 0.f, acc = 0.f;
    float mw[NW], lw[NW], ow[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      mw[w] = -INFINITY; lw[w] = ow[w] = 0.f;
      if (has_chunk(w)) { mw[w] = s_m[w][gg]; lw[w] = s_l[w][gg]; ow[w] = s_o_dyn[dec_o_at<D>(w, p.G, gg, d)]; }
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, mw[w]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (!has_chunk(w)) break;
      const float wt = lw[w] > 0.f ? __builtin_amdgcn_exp2f(mw[w] - M) : 0.f;
      L = fmaf(wt, lw[w], L);
      acc = fmaf(wt, ow[w], acc);
    }
    accs[x] = acc; Ms[x] = M; Ls[x] = L;
    const int h = kvh * p.G + gg;
    if (p.splits == 1) {
      p.o[((int64_t)b * p.hq + h) * D + d] = (__bf16)(acc / L);      // L > 0: chunk 0 of the row is never empty
      if (p.lse && d == 0) p.lse[(int64_t)b * p.hq + h] = (M + log2f(L)) * 0.69314718055994530942f;
    } else if (!p.fused) {
      // a merge kernel follows: plain stores
      float* part = p.partials + (((int64_t)b * p.hq + h) * p.splits + split) * (D + 2);
      part[d] = acc;
      if (d == 0) { part[D] = M; part[D + 1] = L; }                  // an idle split leaves M = -inf, L = 0
    } else {
      uint64_t* pk = p.packets + (((int64_t)b * p.hq + h) * p.splits + split) * (D + 2);
      const uint32_t tag = dec_tag(gen, split);
      dec_put(pk + d, acc, dec_tag_of_output(tag, __builtin_bit_cast(uint32_t, M), __builtin_bit_cast(uint32_t, L)));
      if (d == 0) { dec_put(pk + D, M, tag); dec_put(pk + D + 1, L, tag); }
    }
  }
  if (p.splits == 1 || !p.fused) return;

  // ---- the workgroups of this (sequence, KV head) merge among themselves (protocol above) ----
  // Writes the outputs whose packets are all there; returns which (bit x) are left.
  auto combine = [&](unsigned todo) -> unsigned {
    unsigned left = 0;
#pragma unroll
    for (int x = 0; x < EPT; ++x) {
      const int e = tid + x * 64 * NW;
      if (e >= p.G * D || !(todo >> x & 1)) continue;
      const int gg = e / D, d = e % D;
      const int h = kvh * p.G + gg;
      uint64_t* pk = p.packets + ((int64_t)b * p.hq + h) * p.splits * (D + 2);
      bool valid = true;
      float M = -INFINITY, L = 0.f, acc = 0.f;
      uint64_t pm[MAX_FUSED_SPLITS], pl[MAX_FUSED_SPLITS], po[MAX_FUSED_SPLITS];
#pragma unroll
      for (int y = 0; y < MAX_FUSED_SPLITS; ++y) {     // all loads before any is looked at
        pm[y] = pl[y] = po[y] = 0;
        if (y < p.splits && y != split) {              // uniform over the workgroup; its own partial is in registers
          const uint64_t* ps = pk + (int64_t)y * (D + 2);
          pm[y] = dec_get(ps + D); pl[y] = dec_get(ps + D + 1); po[y] = dec_get(ps + d);
        }
      }
      // the reference point of all of them first, so that their weights do not depend on one another
      float ls[MAX_FUSED_SPLITS], ms[MAX_FUSED_SPLITS];
#pragma unroll
      for (int y = 0; y < MAX_FUSED_SPLITS; ++y) {
        ms[y] = -INFINITY; ls[y] = 0.f;
        if (y >= p.splits) break;
        if (y == split) { ms[y] = Ms[x]; ls[y] = Ls[x]; }              // this workgroup's own partial: the same bits
        else {
          const uint32_t want = dec_tag(gen, y);
          valid = valid && (uint32_t)(pm[y] >> 32) == want && (uint32_t)(pl[y] >> 32) == want
                  && (uint32_t)(po[y] >> 32) == dec_tag_of_output(want, (uint32_t)pm[y], (uint32_t)pl[y]);
          ms[y] = __builtin_bit_cast(float, (uint32_t)pm[y]); ls[y] = __builtin_bit_cast(float, (uint32_t)pl[y]);
        }
        if (ls[y] > 0.f) M = fmaxf(M, ms[y]);                          // idle splits hold no outputs
      }
#pragma unroll
      for (int y = 0; y < MAX_FUSED_SPLITS; ++y) {
        if (y >= p.splits) break;
        const float os = y == split ? accs[x] : __builtin_bit_cast(float, (uint32_t)po[y]);
        const float wt = ls[y] > 0.f ? __builtin_amdgcn_exp2f(ms[y] - M) : 0.f;
        L = fmaf(wt, ls[y], L);
        acc = ls[y] > 0.f ? fmaf(wt, os, acc) : acc;
      }
      // Every thread for itself: a packet that has not landed belongs to a workgroup that will write this output.  (A thread
      // that saw the packets of all splits knows that all their wavefronts have read the generation.)  Packets that are taken
      // back are missing to the other workgroups' threads for the same output, which has been written then.
      if (!valid) { left |= 1u << x; continue; }
      p.o[((int64_t)b * p.hq + h) * D + d] = (__bf16)(acc / L);
      if (p.lse && d == 0) p.lse[(int64_t)b * p.hq + h] = (M + log2f(L)) * 0.69314718055994530942f;
      if (p.through) dec_take_back<__HIP_MEMORY_SCOPE_AGENT>(pk + d, p.splits, D + 2);
      else dec_take_back<__HIP_MEMORY_SCOPE_WORKGROUP>(pk + d, p.splits, D + 2);
      if (e == 0) __hip_atomic_store(p.gen + (int64_t)b * p.hkv + kvh, gen + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return left;
  };
  // With few splits a workgroup that is behind the others finds their packets in place at once, without waiting for its own to
  // be acknowledged (us, without / with: 2 splits, batch 16 at 64K 12.45 / 12.31, 3 splits, batch 4 7.91 / 7.82); with
  // more, the reads that come too early cost more (4 splits 7.86 / 7.96, 7 splits 8.87 / 9.09).
  unsigned todo = ~0u;
  if (p.splits <= 3) todo = combine(todo);
  __builtin_amdgcn_s_waitcnt(0);                       // vmcnt(0): memory has acknowledged this thread's packets
  __syncthreads();                                     // ... and every other thread's of this workgroup
  if (todo) combine(todo);
}

// Large batches: persistent workgroups.  With many more (sequence, KV head, split) items than compute units the
// kernel above leaves every compute unit without a byte in flight while a workgroup looks its sequence length up and
// while it merges (one workgroup fits at a time: its wavefronts hold a whole chunk in registers).  Here a workgroup
// walks through items, and through an item in passes of NW chunks (wavefront w takes chunk w + NW * pass of the
// item's share of the row, keeping its running (max, sum, O) over the passes); a wavefront requests its chunk of the
// next pass (of this item or the next one) as soon as the registers of the current one are free, before the workgroup
// merges a finished item through LDS, and the sequence length and the page of a chunk are read two passes and one
// pass ahead.  With one split per (sequence, KV head), which is how the library launches it once there is at least
// one (sequence, KV head) pair per compute unit, the outputs are written here and no merge follows; with several
// splits the partials go to the workspace with plain stores for the merge kernel below.
template <int D>
__global__ __launch_bounds__(64 * NW) void pa_decode_stream_kernel(dec_params p, int n_items, int n_pass) {
  __shared__ float s_m[2][NW][MAXG], s_l[2][NW][MAXG];
  extern __shared__ __attribute__((aligned(16))) float s_o_dyn[];   // [2][NW][G][D/32][OROW] partial outputs of the wavefronts, two items
  // (wavefront number as a scalar; the lane number is taken afresh in every phase of a step: dec_lane_now)
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int stride = (int)gridDim.x;
  const int per_b = p.hkv * p.splits;

  struct item_t { int b, kvh, split; };
  auto item_of = [&](int w) -> item_t {
    item_t it;
    const int w2 = w < n_items ? w : n_items - 1;          // beyond the end: any valid item (its loads are not issued)
    it.b = per_b == 1 ? w2 : p.per_b_magic ? (int)__umulhi((uint32_t)w2, p.per_b_magic) : w2 / per_b;
    const int r = w2 - it.b * per_b;
    it.kvh = p.splits == 1 ? r : r / p.splits;
    it.split = r - it.kvh * p.splits;
    return it;
  };
  // The workgroup's steps: all passes of its first item (number blockIdx.x of the launch), then of the item
  // `stride` further on, and so on; a step is kept as (item number, pass) and advanced without a division.
  struct step_t { int w, pass; };
  auto after = [&](const step_t& st) -> step_t {
    return st.pass + 1 < n_pass ? step_t{st.w, st.pass + 1} : step_t{st.w + stride, 0};
  };
  // Where this wavefront's chunk of a step lies, given the sequence length:
  struct plan_t { item_t it; dec_place pl; bool has; };
  auto plan_of = [&](const step_t& st, int len) -> plan_t {
    plan_t pn;
    const int w = st.w, pass = st.pass;
    pn.it = item_of(w);
    const dec_row row = dec_row_of(p, len);
    const int slot = (wave + NW * pass) * p.splits + pn.it.split;
    pn.pl = dec_place_of(p, row, slot < row.n_slots ? slot : 0);
    pn.has = w < n_items && slot < row.n_slots && pn.pl.n_tok > 0;
    return pn;
  };
  auto page_ptr = [&](const plan_t& pn) -> const int32_t* {
    return p.block_table ? p.block_table + (int64_t)pn.it.b * p.table_stride + pn.pl.blk : p.kv_len;
  };

  // the scalar pipeline: plan and page of the step after this one, length of the one after that
  step_t st0{(int)blockIdx.x, 0};                         // the current step, and the three after it
  step_t st1 = after(st0), st2 = after(st1), st3 = after(st2);
  plan_t cur = plan_of(st0, p.kv_len[item_of(st0.w).b]);
  int cur_page = *page_ptr(cur);
  plan_t nxt = plan_of(st1, p.kv_len[item_of(st1.w).b]);
  int nxt_page = *page_ptr(nxt);
  int len2 = p.kv_len[item_of(st2.w).b];

  dec_chunk<D> c;
  bf16x8 qf[D / 32];
  auto request = [&](const plan_t& pn, int page) {
    const int lane = dec_lane_now(), g = lane & 15, q4 = lane >> 4;
    dec_load_q<D>(qf, p, pn.it.b, pn.it.kvh, g, q4);
    if (!pn.has) return;                                  // no tokens: no loads (the chunk's registers are not looked at)
    const int64_t off = dec_chunk_offset(p, pn.it.b, pn.it.kvh, pn.pl, page, D);
    dec_issue<D>(c, p.k + off, p.v + off, pn.pl.n_tok, g, q4);
  };
  request(cur, cur_page);

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 O[8];
  int n = 0;                                              // items finished so far: selects the LDS buffer
  for (; st0.w < n_items; st0 = st1, st1 = st2, st2 = st3, st3 = after(st3)) {
    const int pass = st0.pass;
    // ---- this wavefront's chunk of the step ----
    if (pass == 0) {
      m_run = -INFINITY; l_run = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) O[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    {
      const int q4 = dec_lane_now() >> 4;
      if (cur.has) dec_consume<D, false>(c, qf, cur.pl.n_tok, p.c2, q4, m_run, l_run, O);
    }
    const bool last_pass = pass == n_pass - 1;
    const int buf = n & 1;
    float* s_o = s_o_dyn + (size_t)buf * (dec_o_bytes<D>(p.G) / sizeof(float));
    if (last_pass) {
      const int lane = dec_lane_now(), g = lane & 15, q4 = lane >> 4;
      float l_all = l_run + __shfl_xor(l_run, 16);
      l_all += __shfl_xor(l_all, 32);
      if (g < p.G) {
        if (q4 == 0) { s_m[buf][wave][g] = m_run; s_l[buf][wave][g] = l_all; }
        dec_stash<D>(s_o, wave, p.G, g, q4, O);
      }
    }
    // ---- the next step's bytes are requested before this item is merged ----
    const item_t done = cur.it;
    cur = nxt; cur_page = nxt_page;
    request(cur, cur_page);
    nxt = plan_of(st2, len2);
    nxt_page = *page_ptr(nxt);
    len2 = p.kv_len[item_of(st3.w).b];
    if (!last_pass) continue;
    __syncthreads();     // the item's partials are in LDS; the other buffer is free again (its readers passed here)
    ++n;

    for (int e = wave * 64 + dec_lane_now(); e < p.G * D; e += 64 * NW) {
      const int gg = e / D, d = e % D;
      float M = -INFINITY;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) M = fmaxf(M, s_m[buf][wv][gg]);
      float L = 0.f, acc = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) {
        const float wt = s_l[buf][wv][gg] > 0.f ? __builtin_amdgcn_exp2f(s_m[buf][wv][gg] - M) : 0.f;
        L = fmaf(wt, s_l[buf][wv][gg], L);
        acc = fmaf(wt, s_o[dec_o_at<D>(wv, p.G, gg, d)], acc);
      }
      const int h = done.kvh * p.G + gg;
      if (p.splits == 1) {
        p.o[((int64_t)done.b * p.hq + h) * D + d] = (__bf16)(acc / L);      // L > 0: chunk 0 of the row is never empty
        if (p.lse && d == 0) p.lse[(int64_t)done.b * p.hq + h] = (M + log2f(L)) * 0.69314718055994530942f;
      } else {
        float* part = p.partials + (((int64_t)done.b * p.hq + h) * p.splits + done.split) * (D + 2);
        part[d] = acc;
        if (d == 0) { part[D] = M; part[D + 1] = L; }                        // an idle split leaves M = -inf, L = 0
      }
    }
  }
}

// Merges the partials of the splits: one wavefront per (sequence, query head).  The loads of
// eight splits are issued together so that their latencies overlap.
template <int D>
__global__ __launch_bounds__(64) void pa_decode_merge_kernel(dec_params p) {
  constexpr int DPL = D / 64;
  const int h = blockIdx.x, b = blockIdx.y, lane = threadIdx.x;
  const float* part = p.partials + ((int64_t)b * p.hq + h) * p.splits * (D + 2);
  float M = -INFINITY, L = 0.f;
  float acc[DPL];
#pragma unroll
  for (int e = 0; e < DPL; ++e) acc[e] = 0.f;
  for (int s0 = 0; s0 < p.splits; s0 += 8) {
    float m8[8], l8[8], o8[8][DPL];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int s = s0 + x < p.splits ? s0 + x : p.splits - 1;    // clamp: stay inside the row of partials
      const float* ps = part + (int64_t)s * (D + 2);
      m8[x] = ps[D];
      l8[x] = s0 + x < p.splits ? ps[D + 1] : 0.f;
#pragma unroll
      for (int e = 0; e < DPL; ++e) o8[x][e] = ps[lane + 64 * e];
    }
    float Mn = M;
#pragma unroll
    for (int x = 0; x < 8; ++x) if (l8[x] > 0.f) Mn = fmaxf(Mn, m8[x]);
    const float resc = L > 0.f ? __builtin_amdgcn_exp2f(M - Mn) : 0.f;
    L *= resc;
#pragma unroll
    for (int e = 0; e < DPL; ++e) acc[e] *= resc;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if (l8[x] > 0.f) {                                          // idle splits wrote no outputs
        const float wt = __builtin_amdgcn_exp2f(m8[x] - Mn);
        L = fmaf(wt, l8[x], L);
#pragma unroll
        for (int e = 0; e < DPL; ++e) acc[e] = fmaf(wt, o8[x][e], acc[e]);
      }
    }
    M = Mn;
  }
#pragma unroll
  for (int e = 0; e < DPL; ++e) p.o[((int64_t)b * p.hq + h) * D + lane + 64 * e] = (__bf16)(acc[e] / L);
  if (p.lse && lane == 0) p.lse[(int64_t)b * p.hq + h] = (M + log2f(L)) * 0.69314718055994530942f;
}

template <int D, int EPT>
int launch_decode_as(const dec_params& p, int batch, hipStream_t stream) {
  static std::atomic<unsigned long long> attr_done{0};
  if (int st = pa_allow_dynamic_lds(reinterpret_cast<const void*>(&pa_decode_kernel<D, EPT>), dec_o_bytes<D>(MAXG), attr_done)) return st;
  const dim3 grid((uint32_t)(p.kvh_first ? p.hkv : p.splits), (uint32_t)(p.kvh_first ? p.splits : p.hkv), (uint32_t)batch);
  hipLaunchKernelGGL((pa_decode_kernel<D, EPT>), grid, dim3(64 * NW), dec_o_bytes<D>(p.G), stream, p);   // at most 72 KB (G <= 16)
  return pa_note_hip(hipGetLastError());
}
template <int D>
int launch_decode(const dec_params& p, int batch, hipStream_t stream) {
  constexpr int THREADS = 64 * NW;
  if (p.G * D <= THREADS) return launch_decode_as<D, 1>(p, batch, stream);
  if (p.G * D <= 2 * THREADS) return launch_decode_as<D, 2>(p, batch, stream);
  return launch_decode_as<D, MAXG * D / THREADS>(p, batch, stream);
}

}  // namespace

// Workgroups per (sequence, KV head).  A workgroup has all loads of eight 64-token chunks in flight at once; a second pass
// over further chunks would pay the memory latency again, so a row with more chunks is cut into several workgroups.
// Where that leaves compute units idle, more of them pull on the memory system: about four chunks each, in at most half of
// the compute units (the exchange of the partials costs more with every workgroup).  us, 8 KV heads, 12 or 13 chunks,
// 2 / 3 / 4 / 6 / 8 splits: batch 1 8.5 / 7.9 / 7.7 / 8.1 / 8.9, 4 9.2 / 8.8 / 9.0 / 10.5 / 12.0, 8 9.6 / 9.5 / 10.6 / 16.7 / 19.5.
// Rows of 29 chunks or more are cut to one workgroup per compute unit, and a merge kernel follows from 7 splits on (figures at
// MAX_FUSED_SPLITS; batch 1, 48 chunks: 7 splits 11.0, 20 and a merge kernel 9.2).
int32_t pa_decode_splits(const powattn_pattern* pat, int32_t batch, int32_t hkv, int64_t capacity) {
  const int32_t mk = powattn_max_k(pat, capacity);
  if (mk < 1) return 0;
  const int64_t slots = (int64_t)mk * (pat->block / CH);
  const int64_t base = (int64_t)batch * hkv;
  int64_t s = (slots + NW - 1) / NW;                 // one pass per workgroup
  if (s > 8) s = 8;
  if (base * s < 256) {                              // not enough workgroups to cover the chip
    int64_t want = (slots + 3) / 4;
    if (want < 8) {
      if (want > 128 / base) want = 128 / base;
    } else {
      const int64_t cap = slots / 2;
      want = (256 + base - 1) / base;
      if (want > cap) want = cap;
    }
    if (want > s) s = want;
  }
  if (s > 1024) s = 1024;
  return (int32_t)s;
}

// Workspace of a decode call: the generation numbers of the (sequence, KV head) pairs (one 32-bit word each,
// padded to 256 bytes), then room for the partial results as 8-byte packets (the float form of the two-kernel
// merge uses the first half of it).
size_t pa_decode_workspace_layout(int32_t batch, int32_t hq, int32_t hkv, int32_t head_dim, int32_t n_split, size_t* header_bytes) {
  const size_t hdr = ((size_t)batch * hkv * sizeof(uint32_t) + 255) & ~(size_t)255;
  if (header_bytes) *header_bytes = hdr;
  const size_t partials = (size_t)batch * hq * n_split * (size_t)(head_dim + 2) * sizeof(uint64_t);
  return hdr + ((partials + 255) & ~(size_t)255);
}

// ---- the library's own scratch buffer, for callers that cannot allocate a workspace ----
// One array per GPU, held until the process ends; its address on a device is looked up once, with that device
// current, and kept.  The array's name is a host-side handle only: device code and HIP calls get the looked-up
// pointer.  Zero when the module is loaded, which the merge protocol above does not even need.
static __device__ __align__(256) unsigned char scratch[POWATTN_STATIC_SCRATCH_BYTES];

int pa_decode_scratch(void** ptr_out, size_t* bytes_out) {
  static std::atomic<void*> dev_ptr[64];           // per device; null = not looked up yet
  int dev = 0;
  pa_current_device(&dev, nullptr);
  void* ptr = dev_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return pa_note_hip(e);
    if (!ptr) return pa_note_hip(hipErrorInvalidSymbol);
    dev_ptr[dev].store(ptr, std::memory_order_release);   // threads that race here store the same address
  }
  *ptr_out = ptr;
  *bytes_out = sizeof(scratch);
  return POWATTN_OK;
}

int pa_launch_decode_bf16(const pa_decode_args& a) {
  if (a.n_split < 1) return POWATTN_UNSUPPORTED;
  if (a.hkv > 65535 || a.batch > 65535 || a.hq > 65535 * 16) return POWATTN_UNSUPPORTED;
  dec_params p;
  p.q = (const __bf16*)a.q; p.k = (const __bf16*)a.k; p.v = (const __bf16*)a.v; p.kv_len = a.kv_len;
  p.o = (__bf16*)a.o; p.lse = a.lse;
  size_t hdr = 0;
  pa_decode_workspace_layout(a.batch, a.hq, a.hkv, a.head_dim, a.n_split, &hdr);
  p.gen = (uint32_t*)a.workspace;
  p.packets = (uint64_t*)((char*)a.workspace + hdr);
  p.partials = (float*)((char*)a.workspace + hdr);
  p.capacity = a.capacity;
  p.len_max = (int32_t)(a.capacity < 0x7fffffff ? a.capacity : 0x7fffffff);
  p.B = a.pat.block; p.W = a.pat.window; p.S = a.pat.sink; p.flags = a.pat.flags;
  p.hq = a.hq; p.hkv = a.hkv; p.G = a.hq / a.hkv; p.splits = a.n_split; p.subs = a.pat.block / CH;
  p.subs_magic = p.subs > 1 ? (uint32_t)(((1ull << 32) + p.subs - 1) / p.subs) : 0u;
  p.c2 = a.scale * 1.44269504088896340736f;
  p.block_table = a.block_table; p.table_stride = a.table_stride;
  p.last_page = (int32_t)((a.n_pages < 0x7fffffff ? a.n_pages : 0x7fffffff) - 1);
  // few enough splits that every workgroup can afford to read all the others' partials: they merge among
  // themselves; otherwise the merge kernel follows
  p.fused = (a.n_split > 1 && a.n_split <= MAX_FUSED_SPLITS) ? 1 : 0;
  int n_cu = 1;
  pa_current_device(nullptr, &n_cu);
  // Workgroups are dealt to the eight XCDs in turn, so with the KV head as the fastest digit, and a multiple of eight of them,
  // all splits of a pair are on one XCD: their exchange is quicker, but where the launch fills the chip the loads are slower.
  // us, KV head / split fastest, 32 query heads on 8: batch 1 8.10 / 8.20, 2 8.51 / 8.70, 4 9.06 / 9.11, 8 9.62 / 9.72 (short rows
  // 7.98 / 8.43), 16 12.8 / 12.4; 16 heads on 16 8.38 / 8.52.  With four KV heads the splits of a pair are on several XCDs
  // either way, and the split fastest is quicker: 28 on 4, batch 2 10.62 / 10.29, 4 11.45 / 10.85, 8 12.04 / 11.23 (two: level).
  p.kvh_first = a.hkv % 8 == 0 && 2 * (int64_t)a.batch * a.hkv * a.n_split <= n_cu;
  p.through = 2 * (int64_t)a.batch * a.hkv * a.n_split > n_cu;
  // As many work items as compute units, or more: persistent workgroups that keep bytes in flight across items.
  // With at least one (sequence, KV head) pair per compute unit a pair is one item, walked in passes of NW chunks, and the
  // outputs are written by the same kernel; with fewer pairs but still four (sequence, KV head, split) items per
  // compute unit the splits stay (one pass each, more items to balance) and the merge kernel follows.
  {
    const int64_t pairs = (int64_t)a.batch * a.hkv;
    const int64_t max_slots = (int64_t)powattn_max_k(&a.pat, a.capacity) * p.subs;
    int stream_splits = 0;
    if (pairs >= (int64_t)n_cu) stream_splits = 1;
    else if (pairs * a.n_split >= 4 * (int64_t)n_cu && max_slots <= (int64_t)a.n_split * NW) stream_splits = a.n_split;
    const int64_t items = pairs * stream_splits;
    if (stream_splits > 0 && items <= 0x7fffffff / 4 && max_slots <= 0x7fffffff / 4) {
      p.fused = 0;
      p.splits = stream_splits;
      const int64_t per_b = (int64_t)a.hkv * stream_splits;
      p.per_b_magic = per_b > 1 && items * per_b <= 0xffffffffLL ? (uint32_t)(((1ull << 32) + per_b - 1) / per_b) : 0u;
      const int n_pass = (int)((max_slots + (int64_t)stream_splits * NW - 1) / ((int64_t)stream_splits * NW));
      const size_t lds2 = 2 * (a.head_dim == 128 ? dec_o_bytes<128>(p.G) : dec_o_bytes<64>(p.G));   // at most 144 KB
      static std::atomic<unsigned long long> attr_done[2];
      const int which = a.head_dim == 128 ? 0 : 1;
      const void* fn = which == 0 ? reinterpret_cast<const void*>(&pa_decode_stream_kernel<128>)
                                  : reinterpret_cast<const void*>(&pa_decode_stream_kernel<64>);
      if (int st = pa_allow_dynamic_lds(fn, 2 * (which == 0 ? dec_o_bytes<128>(MAXG) : dec_o_bytes<64>(MAXG)), attr_done[which])) return st;
      const dim3 pgrid((uint32_t)n_cu);
      if (a.head_dim == 128)
        hipLaunchKernelGGL((pa_decode_stream_kernel<128>), pgrid, dim3(64 * NW), lds2, a.stream, p, (int)items, n_pass);
      else
        hipLaunchKernelGGL((pa_decode_stream_kernel<64>), pgrid, dim3(64 * NW), lds2, a.stream, p, (int)items, n_pass);
      int st = pa_note_hip(hipGetLastError());
      if (st != POWATTN_OK || stream_splits == 1) return st;
      dim3 mgrid((uint32_t)a.hq, (uint32_t)a.batch);
      if (a.head_dim == 128)
        hipLaunchKernelGGL((pa_decode_merge_kernel<128>), mgrid, dim3(64), 0, a.stream, p);
      else
        hipLaunchKernelGGL((pa_decode_merge_kernel<64>), mgrid, dim3(64), 0, a.stream, p);
      return pa_note_hip(hipGetLastError());
    }
  }
  const int rc = a.head_dim == 128 ? launch_decode<128>(p, a.batch, a.stream) : launch_decode<64>(p, a.batch, a.stream);
  if (rc != POWATTN_OK) return rc;
  int st = pa_note_hip(hipGetLastError());
  if (st != POWATTN_OK || a.n_split == 1 || p.fused) return st;
  dim3 mgrid((uint32_t)a.hq, (uint32_t)a.batch);
  if (a.head_dim == 128)
    hipLaunchKernelGGL((pa_decode_merge_kernel<128>), mgrid, dim3(64), 0, a.stream, p);
  else
    hipLaunchKernelGGL((pa_decode_merge_kernel<64>), mgrid, dim3(64), 0, a.stream, p);
  return pa_note_hip(hipGetLastError());
}
