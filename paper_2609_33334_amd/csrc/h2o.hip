// H2O accumulated attention (Table "Complexity and measured overhead", footnote a): the
// causal softmax of every cached row, summed down each key column and meaned over the
// GQA group,
//   colsum[h][j] = (1/G) sum_g sum_{p >= j} exp(q_{g,p} . k_j / sqrt(d) - lse_{g,p}).
//
// Two kernels on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16):
//
// lse (skipped when the caller supplies it): a workgroup owns a 128-row block of one query
//   head.  Each of its four wavefronts keeps the block's eight 16-row tiles of Q in
//   registers and streams every fourth 16-key subtile of K through an LDS ring of its own
//   (global->LDS copies), so the loop has no barrier; the four (reference, sum) pairs of a
//   row merge once at the end.  The product is taken transposed (A = keys, B = query rows)
//   so a lane holds 4 keys of one row and keeps that row's pair in registers.
//
// colsum: a workgroup owns a 128-key block and a 512-row segment of one KV head.  For every
//   query head of the group, 64-row blocks of Q and their log-sum-exp stream through a
//   LDS ring (global->LDS copies); a wavefront takes 64 of the keys, held in registers, and
//   32 rows of every block, or 32 keys and 64 rows.  With A = query rows, a lane holds 4 rows of
//   one key: P = 2^(x - lse) is summed in the lane and crosses lanes once, at the end of
//   the segment.  A small reduction adds the segments' partial sums in a fixed order.
//
// Both passes issue per 64 logits 16 cycles of matrix product and 16 of fma, exp2 and add.
// A register-only loop of that mix takes 186 ns per 16 products and SIMD however it is
// ordered (140 ns the products alone, 111 ns the rest alone), 1.4 PFLOP/s; the passes reach
// 1.0.  What is left between the two is neither barriers nor LDS reads: a column pass with
// private streams (as the lse pass) took 311 us for 8192 rows and 32 heads against 288 us
// here, and a raised wavefront priority in either part changed nothing.
// No atomics: every partial column sum is owned by exactly one wavefront.
#include "dge_device.hpp"
#include "dge_internal.hpp"

namespace dge {
namespace {

constexpr int D = 128;
constexpr int NS = RowChunks<bf16_t, D>::kSteps;   // 4 chunk steps of 32 elements
constexpr int RowBytes = D * 2;
constexpr int ST = 16;                              // rows (keys) per streamed subtile
constexpr int kStages = 4;                          // subtiles of a wavefront's ring
constexpr int RB = 64;                              // rows per Q block (colsum)
constexpr int KB = 128;                             // keys per colsum key block
constexpr int RBL = 128;                            // rows per lse block
constexpr int NRT = RBL / 16;                       // ... its 16-row tiles, in registers

struct H2oArgs {
  const bf16_t* q;      // [H_q][T][D]
  const bf16_t* k;      // [H_kv][stride]
  const float* lse;     // [H_q][T] natural log
  float* lse_out;       // workspace [H_q][T] (when computing)
  float* colsum;        // [H_kv][T]
  SeqOffsets offs;
  int64_t kv_head_stride;
  int64_t total_rows;
  int n_q_heads, n_kv_heads, G, batch;
  int n_rblk;           // lse: 128-row blocks of the longest sequence
  int log_stripes;      // lse: 8 / gcd(8, H_kv) stripes of a KV head's blocks, its log2 ...
  int stripe_blk;       // ... of so many blocks each
  float scale_log2;
  float inv_G;
};

// A private stream of 16-row subtiles (4 KB, unit u of row r at u ^ r) per wavefront.
struct SubCopies {
  uint32_t off[4];               // byte offset of this lane's unit of copy i: row * 256 + column
  __device__ __forceinline__ explicit SubCopies(int lane) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * i + (lane >> 4);
      off[i] = (uint32_t)(r * RowBytes + ((lane & 15) ^ r) * 16);
    }
  }
  // 16 rows from base on; rows beyond base's row + lim re-read that one
  __device__ __forceinline__ void issue(const char* base, int lim, uint32_t lds) const {
    if (lim >= ST - 1) {         // wave-uniform
#pragma unroll
      for (int i = 0; i < 4; ++i) dma16_sbase(base, off[i], lds + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = (int)(off[i] / RowBytes);
        dma16_sbase(base, off[i] - (uint32_t)((r - min(r, lim)) * RowBytes), lds + i * 1024);
      }
    }
  }
};

__device__ __forceinline__ uint4 lds_frag(const char* lds, int r, int s, int g16) {
  return *reinterpret_cast<const uint4*>(lds + r * RowBytes + (((s * 4 + g16) ^ (r & 15)) * 16));
}

// ------------------------------------------------------------------------------------
// Row log-sum-exp: one (query head, 128-row block, sequence) per workgroup, whose walk over
// the keys is as long as its block is late: units run from the last blocks to the first, so
// the short ones fill the end of the launch.  Each XCD takes a contiguous eighth of the units,
// which is whole KV heads or, if 8 does not divide them, whole stripes of a head: every
// 2nd, 4th or 8th of its blocks, so that no XCD holds the late half of a head (8192 rows, 4
// query heads per KV head, both passes, unstriped and striped: 1 KV head 185 and 171 us, 2 304
// and 233, 4 427 and 351, 6 542 and 513, 12 973 and 902).  Splitting the keys,
// not the heads, over the wavefronts keeps all four busy for any group size (a wavefront
// per head of the group left three of four idle at G = 1), and 128 rows per 16-key subtile
// read a quarter of LDS per product.  The next subtile's fragments are read and its buffer
// refilled between a subtile's products and its exponentials.  8194 rows, 32 query heads:
// 275 us with 64-row blocks and one wavefront per head, 266 us here; both passes at 16 query
// heads on 8 KV heads and 4004 rows 150 -> 110 us, at 8 on 8 and 1.5-1.8K rows 65 -> 48 us.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void h2o_lse_kernel(H2oArgs a) {
  const int units = (a.stripe_blk << a.log_stripes) * a.n_q_heads * a.batch;
  int unit = xcd_unit(units);               // ((h * stripes + stripe) * stripe_blk + i, b, g)
  if (unit >= units) return;
  const int g = unit % a.G;
  unit /= a.G;
  const int b = unit % a.batch;
  unit /= a.batch;
  const int i = unit % a.stripe_blk;
  unit /= a.stripe_blk;
  const int last = (1 << a.log_stripes) - 1, stripe = unit & last, h = unit >> a.log_stripes;
  const int hq = h * a.G + g;
  // the longest walks of the stripe first; stripes deal the blocks out to and fro
  const int rblk = a.n_rblk - 1 - (i << a.log_stripes) - ((i & 1) ? last - stripe : stripe);
  const int64_t s0 = a.offs[b];
  const int N = (int)(a.offs[b + 1] - s0);
  const int r0 = rblk * RBL;
  if (r0 < 0 || r0 >= N) return;            // past the stripe, a shorter sequence of a ragged batch
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform
  const int g16 = lane >> 4, c16 = lane & 15;
  const int nsub = (min(r0 + RBL, N) + ST - 1) / ST;          // key subtiles of this block
  const int nw = (nsub - wv + 3) / 4;                         // this wavefront: wv, wv + 4, ...
  const char* kb = reinterpret_cast<const char*>(a.k + (int64_t)h * a.kv_head_stride + s0 * D);
  const char* qb = reinterpret_cast<const char*>(a.q + ((int64_t)hq * a.total_rows + s0) * D);
  __shared__ __attribute__((aligned(16))) char ring[4][kStages][ST * RowBytes];
  const SubCopies copies(lane);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)&ring[wv][0][0];
  auto issue = [&](int t) {                 // past the last subtile: that one again
    const int j0 = (wv + 4 * max(0, min(t, nw - 1))) * ST;
    copies.issue(kb + (int64_t)min(j0, N - 1) * RowBytes, max(0, N - 1 - j0),
                 lds0 + (uint32_t)(t % kStages) * (ST * RowBytes));
  };
  // query fragments (B operand: lane supplies row c16 of a tile), from asm so that no
  // compiler wait drains the copies; they land with the first subtiles
  u32x4_t qa[NRT][NS];
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    const char* row = qb + (int64_t)min(r0 + rt * 16 + c16, N - 1) * RowBytes;
#pragma unroll
    for (int s = 0; s < NS; ++s) qa[rt][s] = async_load16(row + (s * 4 + g16) * 16);
  }
#pragma unroll
  for (int t = 0; t < kStages; ++t) issue(t);
  asm_wait_vmcnt<0>();
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
    for (int s = 0; s < NS; ++s) reg_fence(qa[rt][s]);
  float m[NRT], sm[NRT];                    // reference and sum (rebase_lse_update)
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) { m[rt] = kLazyRefInit; sm[rt] = 0.0f; }
  uint4 kf[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) kf[s] = lds_frag(ring[wv][0], c16, s, g16);
  for (int t = 0; t < nw; ++t) {
    const int j0 = (wv + 4 * t) * ST;
    wait_lgkmcnt0();                        // subtile t's fragments are here
    // acc[rt][i] = logit of key j0 + 4*g16 + i for row r0 + rt*16 + c16
    f32x4_t acc[NRT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) acc[rt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) acc[rt] = mma_step(bf16_t{}, kf[s], as_uint4(qa[rt][s]), acc[rt]);
    __builtin_amdgcn_sched_barrier(0);
    issue(t + kStages);                     // into subtile t's buffer
    asm_wait_vmcnt<(kStages - 1) * 4>();    // subtile t + 1 landed
#pragma unroll
    for (int s = 0; s < NS; ++s) kf[s] = lds_frag(ring[wv][(t + 1) % kStages], c16, s, g16);
    __builtin_amdgcn_sched_barrier(0);
    float x[NRT][4];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[rt][i] = acc[rt][i];
    if (j0 + ST - 1 > r0) {                 // reaches the block's diagonal
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          x[rt][i] = j0 + 4 * g16 + i <= r0 + rt * 16 + c16 ? x[rt][i] : -INFINITY;
    }
    rebase_lse_update<NRT, 4>(x, a.scale_log2, m, sm);
  }
  asm_wait_vmcnt<0>();                      // no copy still writes into the ring
  // the four lane groups of each row, then the four wavefronts (each writes into its own
  // first buffer)
  float2* xw = reinterpret_cast<float2*>(&ring[wv][0][0]);
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    const float mm = m[rt];
    float ss = sm[rt];
    const float mx = fmaxf(fmaxf(mm, shfl_xor_f<16>(mm)), fmaxf(shfl_xor_f<32>(mm), shfl_xor_f<48>(mm)));
    ss *= rescale(mm, mx);
    ss += shfl_xor_f<16>(ss);
    ss += shfl_xor_f<32>(ss);
    if (g16 == 0) xw[rt * 16 + c16] = make_float2(mx, ss);
  }
  lds_barrier();
  if (tid < RBL && r0 + tid < N) {
    float2 v[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = reinterpret_cast<const float2*>(&ring[w][0][0])[tid];
    const float mx = fmaxf(fmaxf(v[0].x, v[1].x), fmaxf(v[2].x, v[3].x));
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) sum += v[w].y * rescale(v[w].x, mx);
    a.lse_out[(int64_t)hq * a.total_rows + s0 + r0 + tid] = (mx + __log2f(sum)) * 0.6931471805599453f;
  }
}

// ------------------------------------------------------------------------------------
// Column sums.  Work unit = (128-key block kb, 512-row segment s, sequence, KV head):
// the rows p >= 128*kb of segment s, for all G query heads of the group.  Units whose
// segment ends before the key block starts, or starts past the sequence, exit at once;
// every other unit is at most SEG rows x G heads, so the ~half of a causal grid that
// has work is evenly loaded.  The KV head counts slowest: the XCDs then hold heads, which
// cost the same, and not sequences (three sequences of 2.1K to 4.0K rows: 232 -> 165 us,
// the XCDs that held the longest one having had 1.5 times the mean work).  Each unit
// writes the partial column sums of its 128 keys to part[s][h][j]; h2o_reduce_kernel adds
// the segments in a fixed order.  From three query heads per KV head on, a wavefront takes 64
// keys x 32 rows, which read half of LDS per product that 32 keys x 64 rows do, and the ring
// has three stages: three workgroups per compute unit (138 registers, 52 KB).  At one or two
// heads a unit is too short for that (8 or 16 blocks) and spends its time on its start: 32
// keys x 64 rows load each key once instead of twice, and two stages leave room for four
// workgroups (35 KB).  8 KV heads, lse given, 32 x 64 against 64 x 32: G = 1, 1100 rows x 2
// 15.6 and 16.9 us, 7500 rows 76.5 and 81.4; G = 2, 2300 x 2 38.2 and 40.7, 7500 136.5 and
// 136.9; G = 4, 7500 258 and 251.
// ------------------------------------------------------------------------------------
constexpr int SEG = 512;
constexpr int kColCopies = RB * RowBytes / (256 * 16) + 1;     // per thread: 4 of Q, 1 of lse
constexpr int kColStageBytes = RB * RowBytes + 4 * RB * 4;     // Q block; lse once per wavefront

// 4 bytes per lane from global memory straight into LDS (see dma16_sbase).
__device__ __forceinline__ void dma4_sbase(const void* sbase, uint32_t voff, uint32_t lds_wave_base) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %3\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %1, %2\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "v"(voff), "s"(sbase), "s"(lds_wave_base)
      : "memory");
}

// The wavefront's query rows of a block (8 / NKT row tiles from LDS row rw0) against its keys.
// MASK: rows at or past row_end, and keys past a row, add nothing.
template <bool MASK, int NKT>
__device__ __forceinline__ void colsum_rows(const char* qt, const float* lt, int rw0, int r0, int row_end,
                                            int j0, int c16, int g16, const uint4 (&kf)[NKT][NS],
                                            float scale, float (&col)[NKT]) {
#pragma unroll
  for (int rt = 0; rt < 8 / NKT; ++rt) {
    const int rl = rw0 + rt * 16;
    uint4 qf[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) qf[s] = lds_frag(qt, rl + c16, s, g16);
    const float4 l4 = *reinterpret_cast<const float4*>(lt + rl + 4 * g16);
    const float l2[4] = {l4.x * kLog2e, l4.y * kLog2e, l4.z * kLog2e, l4.w * kLog2e};
    f32x4_t acc[NKT];
#pragma unroll
    for (int t = 0; t < NKT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int t = 0; t < NKT; ++t) acc[t] = mma_step(bf16_t{}, qf[s], kf[t][s], acc[t]);
    // acc[t][i] = logit of row r0 + rl + 4*g16 + i for key j0 + 16 t + c16
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < NKT; ++t) {
        float pv = fast_exp2(fmaf(acc[t][i], scale, -l2[i]));
        if constexpr (MASK) {
          const int p = r0 + rl + 4 * g16 + i;
          pv = (p < row_end && j0 + 16 * t + c16 <= p) ? pv : 0.0f;
        }
        col[t] += pv;
      }
  }
}

template <int NKT, int S>
__global__ __launch_bounds__(256, S == 2 ? 4 : 3) void h2o_colsum_kernel(H2oArgs a, float* part, int nkb_max,
                                                         int nseg_max) {
  const int units = nkb_max * nseg_max * a.n_kv_heads * a.batch;
  const int unit = xcd_unit(units);
  if (unit >= units) return;
  const int kblk = unit % nkb_max, seg = (unit / nkb_max) % nseg_max;
  const int b = (unit / (nkb_max * nseg_max)) % a.batch,
            h = unit / (nkb_max * nseg_max * a.batch);
  const int64_t s0 = a.offs[b];
  const int N = (int)(a.offs[b + 1] - s0);
  const int k0 = kblk * KB;
  const int seg_lo = seg * SEG, seg_hi = min(N, seg_lo + SEG);
  if (k0 >= N || seg_lo >= N || seg_hi <= k0) return;     // no rows p >= k0 here
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform
  const int g16 = lane >> 4, c16 = lane & 15;
  constexpr int KW = 16 * NKT, RW = 64 * 32 / KW, NW = KB / KW;   // keys, rows of a wavefront
  const int j0 = k0 + wv % NW * KW;            // this wavefront's keys
  const int rw0 = wv / NW * RW;                // and its rows of every block
  __shared__ __attribute__((aligned(16))) char ring[S][kColStageBytes];
  __shared__ float half_sum[NW][KW];

  const int rlo = max(seg_lo, k0 / RB * RB);   // first 64-row block with rows >= k0
  const int per = (seg_hi - rlo + RB - 1) / RB;
  const int nblk = per * a.G;                  // (head, row block) iterations
  const char* qh = reinterpret_cast<const char*>(a.q + (int64_t)(h * a.G) * a.total_rows * D + s0 * D);
  const float* lh = a.lse + (int64_t)(h * a.G) * a.total_rows + s0;
  // copy i of this thread fills the 16 bytes at 1024 (4 wv + i) + 16 lane of a stage
  const int cr = lane >> 4;                    // row of copy i: 4 (4 wv + i) + cr
  uint32_t ccol[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    ccol[i] = (uint32_t)(((lane & 15) ^ ((4 * (4 * wv + i) + cr) & 15)) * 16);
  int ig = 0, ir = rlo, in = 0;                // head, row and number of the next block to copy
  auto issue = [&](int slot) {
    const int64_t row = (int64_t)ig * a.total_rows + ir;
    const uint32_t lim = (uint32_t)(N - 1 - ir);
    const char* base = qh + row * RowBytes;
    const uint32_t lds = (uint32_t)(uintptr_t)(lds_ptr_t)ring[slot];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      dma16_sbase(base, min((uint32_t)(4 * (4 * wv + i) + cr), lim) * RowBytes + ccol[i],
                  lds + (4 * wv + i) * 1024);
    dma4_sbase(lh + row, min((uint32_t)lane, lim) * 4, lds + RB * RowBytes + wv * RB * 4);
    // past the last block the copies re-read it, so every wait has a fixed count
    if (++in < nblk) {
      ir += RB;
      if (ir >= seg_hi) { ir = rlo; ++ig; }
    }
  };
  // the keys (B operand: lane supplies key c16), from asm so that no compiler wait drains
  // the copies; they land with the first block
  u32x4_t ka[NKT][NS];
  {
    const char* kh = reinterpret_cast<const char*>(a.k + (int64_t)h * a.kv_head_stride + s0 * D);
#pragma unroll
    for (int t = 0; t < NKT; ++t) {
      const char* rk = kh + (int64_t)min(j0 + 16 * t + c16, N - 1) * RowBytes;
#pragma unroll
      for (int s = 0; s < NS; ++s) ka[t][s] = async_load16(rk + (s * 4 + g16) * 16);
    }
  }
#pragma unroll
  for (int t = 0; t < S - 1; ++t) issue(t);
  asm_wait_vmcnt<(S - 2) * kColCopies>();     // block 0 (and the keys) landed
  uint4 kf[NKT][NS];
#pragma unroll
  for (int t = 0; t < NKT; ++t)
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      reg_fence(ka[t][s]);
      kf[t][s] = as_uint4(ka[t][s]);
    }
  float col[NKT];
#pragma unroll
  for (int t = 0; t < NKT; ++t) col[t] = 0.0f;
  int r0 = rlo, slot = 0;
  for (int it = 0; it < nblk; ++it) {
    asm_wait_vmcnt<(S - 2) * kColCopies>();   // block it landed (own copies)
    lds_barrier();                                     // ... everyone's; the last slot is free
    issue(slot == 0 ? S - 1 : slot - 1);
    const char* qt = ring[slot];
    const float* lt = reinterpret_cast<const float*>(qt + RB * RowBytes) + wv * RB;
    // masking only in the (rare) edge blocks: the common body has no branch per logit
    if (r0 + rw0 >= j0 + KW - 1 && r0 + RB <= seg_hi)
      colsum_rows<false, NKT>(qt, lt, rw0, r0, seg_hi, j0, c16, g16, kf, a.scale_log2, col);
    else if (r0 + rw0 + RW - 1 >= j0)
      colsum_rows<true, NKT>(qt, lt, rw0, r0, seg_hi, j0, c16, g16, kf, a.scale_log2, col);
    r0 += RB;
    if (r0 >= seg_hi) r0 = rlo;
    slot = slot + 1 == S ? 0 : slot + 1;
  }
  asm_wait_vmcnt<0>();                         // no copy still writes into the ring
#pragma unroll
  for (int t = 0; t < NKT; ++t) {
    col[t] += shfl_xor_f<16>(col[t]);
    col[t] += shfl_xor_f<32>(col[t]);
  }
  if (wv >= NW && g16 == 0) {
#pragma unroll
    for (int t = 0; t < NKT; ++t) half_sum[wv % NW][16 * t + c16] = col[t];
  }
  if constexpr (NW < 4) __syncthreads();
  if (wv < NW && g16 == 0) {
    float* out = part + ((int64_t)seg * a.n_kv_heads + h) * a.total_rows + s0;
#pragma unroll
    for (int t = 0; t < NKT; ++t) {
      const int j = 16 * t + c16;
      if (j0 + j < N) out[j0 + j] = NW < 4 ? col[t] + half_sum[wv][j] : col[t];
    }
  }
}

// colsum[h][j] = (1/G) * sum over the segments that hold rows >= j's key block, in order.
__global__ __launch_bounds__(256) void h2o_reduce_kernel(H2oArgs a, const float* part) {
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t s0 = a.offs[b];
  const int N = (int)(a.offs[b + 1] - s0);
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= N) return;
  const int nseg = (N + SEG - 1) / SEG;
  float acc = 0.0f;
  for (int s = (j / KB) * KB / SEG; s < nseg; ++s)
    acc += part[((int64_t)s * a.n_kv_heads + h) * a.total_rows + s0 + j];
  a.colsum[(int64_t)h * a.total_rows + s0 + j] = acc * a.inv_G;
}

}  // namespace

size_t h2o_workspace_bytes(const dge_geom_t& g) {
  // row LSE [H_q][T] (when computed here) + segment partials [nseg][H_kv][T]
  const size_t T = (size_t)total_rows(g);
  const size_t nseg = (size_t)((max_seq_rows(g) + SEG - 1) / SEG);
  return (size_t)g.n_q_heads * T * sizeof(float) + nseg * g.n_kv_heads * T * sizeof(float) + 512;
}

hipError_t launch_h2o(const dge_geom_t& g, const void* q_all, const void* k, const float* lse,
                      float* colsum, void* ws, hipStream_t st) {
  H2oArgs a{};
  a.q = reinterpret_cast<const bf16_t*>(q_all);
  a.k = reinterpret_cast<const bf16_t*>(k);
  a.colsum = colsum;
  a.offs = seq_offsets(g);
  a.kv_head_stride = g.kv_head_stride;
  a.total_rows = total_rows(g);
  a.n_q_heads = g.n_q_heads;
  a.n_kv_heads = g.n_kv_heads;
  a.G = g.n_q_heads / g.n_kv_heads;
  a.batch = g.batch;
  a.scale_log2 = kLog2e / sqrtf((float)D);
  a.inv_G = 1.0f / (float)a.G;
  const int64_t nmax = max_seq_rows(g);
  if (nmax == 0) return hipSuccess;
  if (lse == nullptr) {
    a.lse_out = reinterpret_cast<float*>(ws);
    a.n_rblk = (int)((nmax + RBL - 1) / RBL);
    while ((g.n_kv_heads << a.log_stripes) % kXcds != 0) ++a.log_stripes;
    a.stripe_blk = (a.n_rblk + (1 << a.log_stripes) - 1) >> a.log_stripes;
    hipLaunchKernelGGL(h2o_lse_kernel,
                       dim3(xcd_grid((a.stripe_blk << a.log_stripes) * g.n_q_heads * g.batch)), dim3(256),
                       0, st, a);
    a.lse = a.lse_out;
  } else {
    a.lse = lse;
  }
  const int nkb = (int)((nmax + KB - 1) / KB);
  const int nseg = (int)((nmax + SEG - 1) / SEG);
  const size_t lse_bytes = ((size_t)g.n_q_heads * (size_t)a.total_rows * sizeof(float) + 255) / 256 * 256;
  float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + lse_bytes);
  const auto kernel = a.G <= 2 ? h2o_colsum_kernel<2, 2> : h2o_colsum_kernel<4, 3>;
  hipLaunchKernelGGL(kernel, dim3(xcd_grid(nkb * nseg * g.n_kv_heads * g.batch)),
                     dim3(256), 0, st, a, part, nkb, nseg);
  hipLaunchKernelGGL(h2o_reduce_kernel, dim3((unsigned)((nmax + 255) / 256), g.n_kv_heads, g.batch),
                     dim3(256), 0, st, a, part);
  return hipGetLastError();
}

}  // namespace dge
