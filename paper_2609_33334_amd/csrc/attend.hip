// Attention of query rows over a compacted cache: the continuation check of the
// evicted cache (Sec. 3 Eq. 1; the eviction-mass equation of App. "Why deferral can
// recover FullKV"; App. "Attention-matching loss").
//
// bf16 caches take the matrix-core kernel further down.  For fp32 caches one workgroup per
// (query row of a sequence, KV head) handles the G query heads of the group, so each cache
// row is read once for all of them.  The attended rows are
// contiguous, [0, n_kept + visible tail), and go in chunks of 256 keys:
//   - thread t computes the G logits of key c0 + t (its K row in 16-byte loads, the
//     query rows broadcast from LDS), in the log2 domain;
//   - per head, the chunk maximum and the chunk sum of 2^(x - m) are reduced across the
//     4 wavefronts, and the running (m, sum, output) are rescaled (online softmax);
//   - the output update is lane-per-dimension: for each key of the chunk a wavefront
//     reads one V row with consecutive lanes on consecutive elements.
// This is a check kernel: it reads the compacted K/V once per query row and is bound by
// that traffic and by latency, not by arithmetic.
//
// The MASS variant reads only K: from the log-partition over the retained rows and the
// caller's full-cache log-partition it writes each observation row's evicted mass
// rho = 1 - Z_R / Z = -expm1(-(lse_full - lse_R)); a second launch averages rho and the
// deficit -log(1 - rho) over each (sequence, KV head)'s rows in a fixed order.
#include "dge_device.hpp"
#include "dge_internal.hpp"

namespace dge {
namespace {

constexpr int kAttThreads = 256;
constexpr int kChunk = kAttThreads;   // keys per chunk, one per thread
constexpr int kMaxAttG = 8;           // query heads per KV head

struct AttArgs {
  const void* q;
  const void* k;
  const void* v;
  const int32_t* n_kept;
  float* out;
  float* lse;
  const float* lse_full;              // MASS: [H_q][batch * n_q] natural log, full cache
  float* rho;                         // MASS: [H_q][batch * n_q] evicted mass per row
  float* beta;                        // MASS: [batch][H_kv] mean rho
  float* l_match;                     // MASS: [batch][H_kv] mean -log(1 - rho)
  int batch, n_kv_heads, G, n_q, q_from_end, n_select, n_tail, n_out;
  int row_blocks;                     // matrix-core path: row blocks per (query head, sequence)
  float scale_log2;                   // log2(e) / sqrt(d)
};

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_t;

template <int D, bool MASS>
__global__ __launch_bounds__(kAttThreads) void cache_attention_f32_kernel(AttArgs a) {
  constexpr int kOwn = (kMaxAttG * D + kAttThreads - 1) / kAttThreads;
  const int row = blockIdx.x;                                 // b * n_q + r
  const int b = row / a.n_q, r = row - b * a.n_q;
  const int h = blockIdx.y;
  const int G = a.G;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ float qs[kMaxAttG][D];
  __shared__ float ps[kMaxAttG][kChunk];
  __shared__ float redm[kMaxAttG][4], reds[kMaxAttG][4];

  const int64_t q_rows = (int64_t)a.batch * a.n_q;
  const float* qb = reinterpret_cast<const float*>(a.q);
  for (int i = tid; i < G * D; i += kAttThreads) {
    const int g = i / D, e = i - g * D;
    qs[g][e] = qb[((int64_t)(h * G + g) * q_rows + row) * D + e];
  }
  const int nk = max(0, min(a.n_kept[b], a.n_select));
  const int nt = max(0, min(a.n_tail, a.n_tail - a.q_from_end + r + 1));
  const int n_vis = nk + nt;                                  // rows [0, n_vis) attended
  const int64_t row0 = ((int64_t)b * a.n_kv_heads + h) * a.n_out;
  const float* kc = reinterpret_cast<const float*>(a.k) + row0 * D;
  const float* vc = reinterpret_cast<const float*>(a.v) + row0 * D;

  // this thread's output elements: e = tid + kAttThreads * i (head e / D, dim e % D;
  // kAttThreads is a multiple of D, so the dim is the same for all of them)
  const int dim = tid % D;
  float o[kOwn];
#pragma unroll
  for (int i = 0; i < kOwn; ++i) o[i] = 0.0f;
  float m2[kMaxAttG], sum[kMaxAttG];                          // wave-uniform
#pragma unroll
  for (int g = 0; g < kMaxAttG; ++g) { m2[g] = -INFINITY; sum[g] = 0.0f; }
  __syncthreads();                                            // qs ready

  for (int c0 = 0; c0 < n_vis; c0 += kChunk) {
    const int j = c0 + tid;
    const bool valid = j < n_vis;
    float x[kMaxAttG];
#pragma unroll
    for (int g = 0; g < kMaxAttG; ++g) x[g] = 0.0f;
    if (valid) {
      const float* krow = kc + (int64_t)j * D;
      for (int e0 = 0; e0 < D; e0 += 4) {
        const float4 kv4 = *reinterpret_cast<const float4*>(krow + e0);
        const float kv[4] = {kv4.x, kv4.y, kv4.z, kv4.w};
#pragma unroll
        for (int g = 0; g < kMaxAttG; ++g)
          if (g < G)
#pragma unroll
            for (int t = 0; t < 4; ++t) x[g] = fmaf(kv[t], qs[g][e0 + t], x[g]);
      }
    }
    // chunk maxima per head, across the 4 wavefronts
#pragma unroll
    for (int g = 0; g < kMaxAttG; ++g) {
      if (g >= G) break;
      x[g] = valid ? x[g] * a.scale_log2 : -INFINITY;
      float mx = x[g];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
      if (lane == 0) redm[g][wv] = mx;
    }
    __syncthreads();
    float alpha[kMaxAttG];
#pragma unroll
    for (int g = 0; g < kMaxAttG; ++g) {
      if (g >= G) break;
      const float cm = fmaxf(fmaxf(redm[g][0], redm[g][1]), fmaxf(redm[g][2], redm[g][3]));
      const float nm = fmaxf(m2[g], cm);
      alpha[g] = rescale(m2[g], nm);
      m2[g] = nm;
      const float p = valid ? fast_exp2(x[g] - nm) : 0.0f;
      ps[g][tid] = p;
      float s = p;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (lane == 0) reds[g][wv] = s;
    }
    __syncthreads();                                          // ps and reds complete
#pragma unroll
    for (int g = 0; g < kMaxAttG; ++g) {
      if (g >= G) break;
      sum[g] = sum[g] * alpha[g] + ((reds[g][0] + reds[g][1]) + (reds[g][2] + reds[g][3]));
    }
    if constexpr (MASS) {
      __syncthreads();                                        // redm, reds free
      continue;
    }
    // output: o[head][dim] = o * alpha + sum_t p[head][t] * V[c0 + t][dim]
    const int n_here = min(kChunk, n_vis - c0);
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const int g = (tid + kAttThreads * i) / D;
      if (g < G) o[i] *= alpha[g];
    }
    const float* vrow = vc + (int64_t)c0 * D + dim;
#pragma unroll 8
    for (int t = 0; t < n_here; ++t) {
      const float vv = vrow[(int64_t)t * D];
#pragma unroll
      for (int i = 0; i < kOwn; ++i) {
        const int g = (tid + kAttThreads * i) / D;
        if (g < G) o[i] = fmaf(ps[g][t], vv, o[i]);
      }
    }
    __syncthreads();                                          // ps, redm, reds free
  }

  if constexpr (MASS) {
    if (tid < G) {
      const int g = tid;
      const int64_t ri = (int64_t)(h * G + g) * q_rows + row;
      const float lse_r = n_vis > 0 ? (m2[g] + __log2f(sum[g])) * 0.6931471805599453f : -INFINITY;
      // deficit log Z - log Z_R >= 0 (rounding can leave it a hair below 0 when nothing of
      // the row's attention is evicted)
      const float dlt = fmaxf(a.lse_full[ri] - lse_r, 0.0f);
      a.rho[ri] = -expm1f(-dlt);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < kOwn; ++i) {
    const int e = tid + kAttThreads * i;
    const int g = e / D;
    if (g < G) {
      const int64_t oi = ((int64_t)(h * G + g) * q_rows + row) * D + dim;
      a.out[oi] = n_vis > 0 ? o[i] / sum[g] : 0.0f;
    }
  }
  if (tid < G) {
    const int g = tid;
    a.lse[(int64_t)(h * G + g) * q_rows + row] =
        n_vis > 0 ? (m2[g] + __log2f(sum[g])) * 0.6931471805599453f : -INFINITY;
  }
}

// ---------------------------------------------------------------------------------------
// Matrix-core path (bf16, d = 64 or 128, any number of query rows).  One workgroup per
// (row block, query head, sequence): a row block is up to three 16-row tiles of the head's
// n_q rows (the 34 scoring rows are one block), and the workgroup's wavefronts deal the
// 32-key subtiles of the compacted rows out among themselves, wavefront w taking subtiles
// w, w + W, w + 2W, ...  Each wavefront keeps its own (reference, sum, output) of every row
// and nothing is shared until the end, so the loop holds no barrier and every subtile's
// loads have the wavefront's own softmax and products to land under; the W partial results
// of a row meet once in LDS, in a fixed order.  The G workgroups of a KV head are
// consecutive units of the XCD-aware order, so they share one L2 and each compacted row
// leaves HBM once.
//   Every load is a global->LDS copy of whole rows (consecutive lanes on consecutive 16-byte
//   units; loading MFMA fragments straight from global memory puts neighbouring lanes on
//   different rows, which a compute unit serves at a quarter of the rate: measured 35 bytes
//   per ns for K alone) into the wavefront's own buffers, kBuf of K and of V:
//   K: 16-byte units XOR-swizzled by row; a subtile's fragments are read into registers at
//      once and the buffer is refilled before the products.
//   V: 32-byte segments XOR-swizzled by row, read as MFMA operands by the transposing LDS
//      read ds_read_b64_tr_b16, which gives lane c of a 16-lane group four keys of
//      dimension c; refilled after the products.
//   Past the wavefront's last subtile the copies read one row of the cache, so every wait has
//   a fixed count.
//   logits:  S^T = K Q^T per 16-key half (A = keys, B = query rows): a lane holds 4 keys
//            of one row; subtiles below every row's first invisible key skip the mask;
//   softmax: per row a reference m, the same in the row's four lane groups, and a sum per
//            lane; m moves only when a sum reaches kSumLimit (then to the row's batch
//            maximum, the sums and outputs rescaled), so the common path is fma, exp2, add;
//   output:  O^T += V^T P^T per 32 keys (A = V^T, B = the lane's own 8 weights from the two
//            halves), P split into a truncated bf16 high part and the bf16 of the remainder
//            (two products, ~15 bits of weight); a lane holds 4 dimensions of its own row,
//            so the rescale of a row is local to the lane.
// The evicted-mass variant (MASS) stops after the sums.
//   FULL: float32 weights, as three truncated bf16 parts that hold all 24 bits (three
// products), and attend_row for every row whose sum or output is not finite: the products
// take the V rows of whole subtiles, hidden ones times 0, in parts of a weight and against a
// reference that may lie 2^100 below the row's maximum, so an infinity, a NaN or a value near
// the top of the range can come out as one that the weights times the visible rows are not.
// d = 64, 34 rows, 8 sequences of 2050 rows, 32 heads, attention and mass: 39 us, error
// against 64 bits 2.2e-7; with two parts 35 us and 9.7e-6, the workgroup-per-row kernel of the
// fp32 caches on bf16 1290 us and 8.1e-7.  d = 128, 70 rows: 103, 83 and 3650 us.
// What bounds it (MI355X, 34 rows x 32 heads x 8 sequences over 2050 rows each, 256
// workgroups): every compute unit reads its own 1 MB of K and V, 92 bytes per ns with one row
// tile (a quarter of that from HBM or the Infinity Cache, the rest its XCD's L2); with three
// row tiles the products and the softmax of two wavefronts per SIMD (9.2 ns per key, 4.8 of
// them matrix-core cycles, against 5.6 with one).  Measured, attention 55 -> 28 us, mass with
// its reduce launch 25 -> 18 us, against the previous kernel (the four row tiles and the key
// pairs of shared 64-key tiles over the wavefronts, two barriers per tile); 16 rows 18 and 13 us.
template <int D, int RT, bool MASS>
struct AttWave {
  static constexpr int kWaves = 8;
  static constexpr int kThreads = kWaves * kWave;
  static constexpr int kPerSimd = kWaves / 4;              // wavefronts per SIMD
  static constexpr int kBuf = (MASS ? 2 : 1) * (128 / D);  // buffers of K, and of V, per wavefront
  static constexpr int kSub = 32;                          // keys per subtile
  static constexpr int kRowBytes = D * 2;
  static constexpr int kUnits = kRowBytes / 16;            // 16-byte units per row
  static constexpr int kNS = D / 32;                       // MFMA steps over d
  static constexpr int kDT = D / 16;                       // 16-dimension output tiles
  static constexpr int kSubBytes = kSub * kRowBytes;       // one subtile of K or of V
  static constexpr int kCopies = kSubBytes / (kWave * 16); // copy instructions per subtile
  static constexpr int kVCopies = MASS ? 0 : kCopies;
  static constexpr int kWaveBytes = (MASS ? 1 : 2) * kBuf * kSubBytes;
  static constexpr int kQBytes = RT * 16 * kRowBytes;      // the block's query rows
  static constexpr int kMergeTiles = MASS ? 1 : (RT < 2 ? RT : 2);   // row tiles merged at once
  static constexpr int kMergeBytes = MASS ? 0 : kMergeTiles * kWaves * 16 * D * 4;
  static constexpr int kRingBytes = kWaves * kWaveBytes;
  static constexpr int kArea = kRingBytes > kMergeBytes ? kRingBytes : kMergeBytes;
  static constexpr int kLdsBytes = kArea + kQBytes;
};

// Row of the swizzle of V row r: its 32-byte segment s is kept at segment s ^ att_swz(r), so
// that the 8 rows of half a transposing read fall on all 64 banks.
template <int D>
__device__ __forceinline__ int att_swz(int r) {
  return D == 128 ? (r & 7) : ((r >> 1) & 3);
}

// One query row done by the whole workgroup as the fp32 kernel does it: a running maximum,
// float32 weights, the n_vis rows it sees and no others.  For the few rows whose result the
// matrix-core loop cannot vouch for; lds is free.
template <int D, bool MASS>
__device__ __forceinline__ void attend_row(const AttArgs& a, int64_t ri, const char* kc, const char* vc,
                                           int n_vis, char* lds) {
  constexpr int T = AttWave<D, 1, MASS>::kThreads, W = T / kWave;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  float* qs = reinterpret_cast<float*>(lds);                   // [D]
  float* ps = qs + D;                                          // [T] weights of a chunk
  float* red = ps + T;                                         // [2][W] maxima, sums
  const uint16_t* q = reinterpret_cast<const uint16_t*>(a.q) + ri * D;
  auto f32 = [](uint32_t bf16_bits) { return __uint_as_float(bf16_bits << 16); };
  __syncthreads();                                             // lds is free for everyone
  if (tid < D) qs[tid] = f32(q[tid]);
  float m = -INFINITY, sum = 0.0f, o = 0.0f;                   // o: dimension tid, tid < D
  __syncthreads();
  for (int c0 = 0; c0 < n_vis; c0 += T) {
    const bool valid = c0 + tid < n_vis;
    float x = -INFINITY;
    if (valid) {
      const char* row = kc + (int64_t)(c0 + tid) * (D * 2);
      float acc = 0.0f;
      for (int e = 0; e < D; e += 8) {
        const uint4 u = load16(row + e * 2);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc = fmaf(f32(w[i]), qs[e + 2 * i], acc);
          acc = fmaf(f32(w[i] >> 16), qs[e + 2 * i + 1], acc);
        }
      }
      x = acc * a.scale_log2;
    }
    float mx = x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if (lane == 0) red[wv] = mx;
    __syncthreads();
    float nm = m;
#pragma unroll
    for (int w = 0; w < W; ++w) nm = fmaxf(nm, red[w]);
    const float alpha = rescale(m, nm), p = valid ? fast_exp2(x - nm) : 0.0f;
    m = nm;
    ps[tid] = p;
    float s = p;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) red[W + wv] = s;
    __syncthreads();                                           // ps and the sums are complete
    float cs = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w) cs += red[W + w];
    sum = sum * alpha + cs;
    if (!MASS && tid < D) {
      const uint16_t* v = reinterpret_cast<const uint16_t*>(vc) + (int64_t)c0 * D + tid;
      const int n = min(T, n_vis - c0);
      o *= alpha;
#pragma unroll 8
      for (int t = 0; t < n; ++t) o = fmaf(ps[t], f32(v[(int64_t)t * D]), o);
    }
    __syncthreads();                                           // ps and red are free
  }
  const float lse_r = n_vis > 0 ? (m + __log2f(sum)) * 0.6931471805599453f : -INFINITY;
  if constexpr (MASS) {
    if (tid == 0) a.rho[ri] = -expm1f(-fmaxf(a.lse_full[ri] - lse_r, 0.0f));
  } else {
    if (tid < D) a.out[ri * D + tid] = n_vis > 0 ? o / sum : 0.0f;
    if (tid == 0) a.lse[ri] = lse_r;
  }
}

template <int D, int RT, bool MASS, bool FULL>
__global__ __launch_bounds__((AttWave<D, RT, MASS>::kThreads), (AttWave<D, RT, MASS>::kPerSimd))
void cache_attention_wave_kernel(AttArgs a) {
  using AT = AttWave<D, RT, MASS>;
  constexpr int NS = AT::kNS, W = AT::kWaves;
  const int units = a.batch * a.n_kv_heads * a.G * a.row_blocks;
  const int unit = xcd_unit(units);
  if (unit >= units) return;
  const int rb = unit % a.row_blocks, hb = unit / a.row_blocks;
  const int hq = hb % (a.n_kv_heads * a.G), b = hb / (a.n_kv_heads * a.G);
  const int h = hq / a.G;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g16 = lane >> 4, c16 = lane & 15;
  const int r0 = rb * RT * 16;                                 // first row of the block
  const int64_t q_rows = (int64_t)a.batch * a.n_q;
  const int64_t row_base = (int64_t)hq * q_rows + (int64_t)b * a.n_q;
  const int nk = max(0, min(a.n_kept[b], a.n_select));
  const int r_last = min(a.n_q, r0 + RT * 16) - 1;             // last row of the block
  auto visible = [&](int r) { return nk + max(0, min(a.n_tail, a.n_tail - a.q_from_end + r + 1)); };
  const int n_vis_max = visible(r_last), n_vis_min = visible(r0);
  const int64_t row0 = ((int64_t)b * a.n_kv_heads + h) * a.n_out;
  const char* kc = reinterpret_cast<const char*>(a.k) + row0 * AT::kRowBytes;
  const char* vc = MASS ? nullptr : reinterpret_cast<const char*>(a.v) + row0 * AT::kRowBytes;
  __shared__ __attribute__((aligned(1024))) char lds[AT::kLdsBytes];
  __shared__ float mfin[W][RT * 16], sfin[W][RT * 16], mrow[RT * 16], irow[RT * 16];
  __shared__ int again[FULL ? RT * 16 : 1];                    // rows left to attend_row

  if (n_vis_max == 0) {                                        // nothing visible: no loads
    for (int r = r0 + wv; r <= r_last; r += W) {
      if constexpr (MASS) {
        if (lane == 0) a.rho[row_base + r] = 1.0f;
      } else {
        if (lane == 0) a.lse[row_base + r] = -INFINITY;
        for (int e = lane; e < D; e += kWave) a.out[(row_base + r) * D + e] = 0.0f;
      }
    }
    return;
  }

  float m[RT], ssum[RT];
  f32x4_t o[MASS ? 1 : RT][MASS ? 1 : AT::kDT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    m[i] = kLazyRefInit;
    ssum[i] = 0.0f;
  }
#pragma unroll
  for (int i = 0; i < (MASS ? 1 : RT); ++i)
#pragma unroll
    for (int dt = 0; dt < (MASS ? 1 : AT::kDT); ++dt) o[i][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // the full-cache log-partition of row tid, before the copies: it is needed at the very end
  // and would otherwise cost a round trip of its own there
  float full = 0.0f;
  if constexpr (MASS) full = async_load4(a.lse_full + row_base + min(r0 + tid, r_last));

  // the block's query rows (rows past its last one read that row; their results are dropped)
  char* qlds = lds + AT::kArea;
  {
    const char* qb = reinterpret_cast<const char*>(a.q) + (row_base + r0) * AT::kRowBytes;
    const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)qlds);
    for (int i = wv; i < AT::kQBytes / (kWave * 16); i += W) {
      const int e = i * kWave + lane, r = e / AT::kUnits, u = (e % AT::kUnits) ^ (r % AT::kUnits);
      dma16_sbase(qb, (uint32_t)(min(r, r_last - r0) * AT::kRowBytes + u * 16), dst + i * kWave * 16);
    }
  }

  const int nt = (n_vis_max + AT::kSub - 1) / AT::kSub;
  char* kbuf = lds + wv * AT::kWaveBytes;                      // [kBuf] K subtiles, then V's
  char* vbuf = kbuf + AT::kBuf * AT::kSubBytes;
  // Copy of subtile t's rows of base: lane l of instruction i fills 16-byte position
  // e = 64 i + l and fetches the unit that belongs there.  The unit's offset within the
  // instruction's kilobyte repeats every P instructions and is kept (off); a subtile that
  // reaches past the last visible row derives clamped rows instead (rows past it read it,
  // those keys are masked; a subtile past the end reads row 0), from a lane number that the
  // empty asm keeps out of the loop's registers.
  constexpr int PK = D == 128 ? 4 : 1, PV = D == 128 ? 2 : 1;
  auto swz_k = [](int r, int p) { return p ^ (r % AT::kUnits); };
  auto swz_v = [](int r, int p) { return (((p >> 1) ^ att_swz<D>(r)) << 1) | (p & 1); };
  uint32_t off_k[PK], off_v[MASS ? 1 : PV];
#pragma unroll
  for (int i = 0; i < PK; ++i) {
    const int e = i * kWave + lane, r = e / AT::kUnits;
    off_k[i] = (uint32_t)((r * AT::kUnits + swz_k(r, e % AT::kUnits)) * 16 - i * kWave * 16);
  }
#pragma unroll
  for (int i = 0; i < (MASS ? 1 : PV); ++i) {
    const int e = i * kWave + lane, r = e / AT::kUnits;
    off_v[i] = (uint32_t)((r * AT::kUnits + swz_v(r, e % AT::kUnits)) * 16 - i * kWave * 16);
  }
  auto copy = [&](const char* base, int t, char* buf, const uint32_t* off, int P, auto swz) {
    const bool real = t < nt;                                  // wave-uniform
    base += real ? (int64_t)t * AT::kSubBytes : 0;
    const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)buf);
    if (t * AT::kSub + AT::kSub <= n_vis_max) {
#pragma unroll
      for (int i = 0; i < AT::kCopies; ++i)
        dma16_sbase(base + i * kWave * 16, off[i % P], dst + i * kWave * 16);
    } else {
      const int last = real ? n_vis_max - 1 - t * AT::kSub : 0;
      int l = lane;
      asm volatile("" : "+v"(l));
#pragma unroll
      for (int i = 0; i < AT::kCopies; ++i) {
        const int e = i * kWave + l, r = e / AT::kUnits;
        dma16_sbase(base, (uint32_t)((min(r, last) * AT::kUnits + swz(r, e % AT::kUnits)) * 16),
                    dst + i * kWave * 16);
      }
    }
  };
  auto copy_k = [&](int t, int s) { copy(kc, t, kbuf + s * AT::kSubBytes, off_k, PK, swz_k); };
  auto copy_v = [&](int t, int s) {
    if constexpr (!MASS) copy(vc, t, vbuf + s * AT::kSubBytes, off_v, PV, swz_v);
  };

  // kBuf subtiles of K and V in flight, K before V
  constexpr int kAhead = AT::kBuf * (AT::kCopies + AT::kVCopies);
#pragma unroll
  for (int s = 0; s < AT::kBuf; ++s) {
    copy_k(wv + s * W, s);
    copy_v(wv + s * W, s);
  }
  asm_wait_vmcnt<kAhead>();                                    // the query rows and full
  if constexpr (MASS) reg_fence(full);
  wg_barrier();
  u32x4_t qf[RT][NS];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int r = i * 16 + c16;
      qf[i][st] = __builtin_bit_cast(
          u32x4_t, load16(qlds + r * AT::kRowBytes + (((st * 4 + g16) ^ (r % AT::kUnits)) * 16)));
    }

  for (int t0 = wv; t0 < nt; t0 += AT::kBuf * W) {
#pragma unroll
   for (int s = 0; s < AT::kBuf; ++s) {
    const int t = t0 + s * W;
    asm_wait_vmcnt<kAhead - AT::kCopies>();                    // K of subtile t
    uint4 kf[2][NS];
#pragma unroll
    for (int su = 0; su < 2; ++su)
#pragma unroll
      for (int st = 0; st < NS; ++st) {
        const int r = 16 * su + c16;
        kf[su][st] = load16(kbuf + s * AT::kSubBytes + r * AT::kRowBytes +
                            (((st * 4 + g16) ^ (r % AT::kUnits)) * 16));
      }
    wait_lgkmcnt0();                                           // fragments in registers
    copy_k(t + AT::kBuf * W, s);
    const int j0 = t * AT::kSub;
    uint4 ph[MASS ? 1 : RT], pl[MASS ? 1 : RT], pr[FULL && !MASS ? RT : 1];
    if (t < nt) {                                              // wave-uniform
    const bool masked = j0 + AT::kSub > n_vis_min;             // some key may be hidden
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      f32x4_t acc[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int st = 0; st < NS; ++st)
#pragma unroll
        for (int su = 0; su < 2; ++su) acc[su] = mma_step(bf16_t{}, kf[su][st], as_uint4(qf[i][st]), acc[su]);
      // x[4 su + q] = logit of key j0 + 16 su + 4 g16 + q for this lane's row of tile i
      float x[8];
#pragma unroll
      for (int su = 0; su < 2; ++su)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          x[4 * su + q] = acc[su][q];
      if (masked) {
        // the row's limit is derived here (the empty asm keeps it out of the loop's registers)
        int r = r0 + i * 16 + c16;
        asm volatile("" : "+v"(r));
        const int lim = visible(min(r, r_last));
#pragma unroll
        for (int su = 0; su < 2; ++su)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (j0 + 16 * su + 4 * g16 + q >= lim) x[4 * su + q] = -INFINITY;
      }
      float pv[8];
      auto weigh = [&](float ref) {
#pragma unroll
        for (int q = 0; q < 8; ++q) pv[q] = fast_exp2(fmaf(x[q], a.scale_log2, -ref));
        return ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
      };
      float ns = ssum[i] + weigh(m[i]);
      // a row whose sum (in any of its lane groups) reaches kSumLimit moves its reference,
      // the same in all four lane groups
      int ov = !(ns < kSumLimit) ? 1 : 0;
      if (__any(ov)) {
        ov |= __shfl_xor(ov, 16, 64);
        ov |= __shfl_xor(ov, 32, 64);
        float mx = x[0];
#pragma unroll
        for (int q = 1; q < 8; ++q) mx = fmaxf(mx, x[q]);
        mx *= a.scale_log2;
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (ov) {
          const float nr = fmaxf(mx, m[i] + kLazyBound);
          const float f = fast_exp2(m[i] - nr);
          ns = ssum[i] * f + weigh(nr);
          if constexpr (!MASS) {
#pragma unroll
            for (int dt = 0; dt < AT::kDT; ++dt)
#pragma unroll
              for (int q = 0; q < 4; ++q) o[i][dt][q] *= f;
          }
          m[i] = nr;
        }
      }
      ssum[i] = ns;
      if constexpr (!MASS) {
        // P ~ hi + lo: hi = the upper half of each float (a bf16 truncation), lo = the
        // remainder, also truncated; packed two weights per register.  FULL: the remainder of
        // lo has at most 8 significant bits and is the third part
        uint32_t hb[4], lb[4], rb[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t u0 = __float_as_uint(pv[2 * q]), u1 = __float_as_uint(pv[2 * q + 1]);
          const float l0 = pv[2 * q] - __uint_as_float(u0 & 0xffff0000u);
          const float l1 = pv[2 * q + 1] - __uint_as_float(u1 & 0xffff0000u);
          hb[q] = __builtin_amdgcn_perm(u1, u0, 0x07060302u);
          lb[q] = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);
          if constexpr (FULL) {
            const float r0 = l0 - __uint_as_float(__float_as_uint(l0) & 0xffff0000u);
            const float r1 = l1 - __uint_as_float(__float_as_uint(l1) & 0xffff0000u);
            rb[q] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
          }
        }
        ph[i] = make_uint4(hb[0], hb[1], hb[2], hb[3]);
        pl[i] = make_uint4(lb[0], lb[1], lb[2], lb[3]);
        if constexpr (FULL) pr[i] = make_uint4(rb[0], rb[1], rb[2], rb[3]);
      }
    }
    }
    if constexpr (!MASS) {
      asm_wait_vmcnt<kAhead - AT::kVCopies>();                 // V of subtile t
      // V^T operand of dimension tile dt: lane group g16's keys 4 g16 .. +3 of each half; all
      // of them go to registers (K's are free by now) so that the buffer refills at once
      const int vr = 4 * g16 + (c16 >> 2);
      const uint32_t va = (uint32_t)(uintptr_t)(lds_ptr_t)(vbuf + s * AT::kSubBytes) +
                          vr * AT::kRowBytes + att_swz<D>(vr) * 32 + (c16 & 3) * 8;
      uint4 vf[AT::kDT];
#pragma unroll
      for (int dt = 0; dt < AT::kDT; ++dt) {
        const uint32_t at = va ^ (dt * 32);
        const uint2 w0 = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_t)(uintptr_t)at));
        const uint2 w1 = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_t)(uintptr_t)(at + 16 * AT::kRowBytes)));
        vf[dt] = make_uint4(w0.x, w0.y, w1.x, w1.y);
      }
      wait_lgkmcnt0();
      copy_v(t + AT::kBuf * W, s);
      if (t < nt) {
#pragma unroll
        for (int dt = 0; dt < AT::kDT; ++dt)
#pragma unroll
          for (int i = 0; i < RT; ++i) {
            o[i][dt] = mma_step(bf16_t{}, vf[dt], ph[i], o[i][dt]);
            o[i][dt] = mma_step(bf16_t{}, vf[dt], pl[i], o[i][dt]);
            if constexpr (FULL) o[i][dt] = mma_step(bf16_t{}, vf[dt], pr[i], o[i][dt]);
          }
      }
    }
   }
  }
  asm_wait_vmcnt<0>();                                         // no copy still writes

  // the wavefronts' references and sums of each row, then their outputs, two row tiles at
  // a time through the ring area (16-byte units XOR-swizzled by row)
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    float st = ssum[i];
    st += __shfl_xor(st, 16, 64);
    st += __shfl_xor(st, 32, 64);
    if (g16 == 0) {
      mfin[wv][i * 16 + c16] = m[i];
      sfin[wv][i * 16 + c16] = st;
    }
  }
  __syncthreads();
  if (tid < RT * 16) {                                         // row tid of the block
    float mf = mfin[0][tid], sf = 0.0f;
#pragma unroll
    for (int w = 1; w < W; ++w) mf = fmaxf(mf, mfin[w][tid]);
#pragma unroll
    for (int w = 0; w < W; ++w) sf += sfin[w][tid] * rescale(mfin[w][tid], mf);
    const float lse_r = sf > 0.0f ? (mf + __log2f(sf)) * 0.6931471805599453f : -INFINITY;
    if (r0 + tid <= r_last) {
      // deficit log Z - log Z_R >= 0 (rounding can leave it a hair below 0)
      if constexpr (MASS) a.rho[row_base + r0 + tid] = -expm1f(-fmaxf(full - lse_r, 0.0f));
      else a.lse[row_base + r0 + tid] = lse_r;
    }
    if constexpr (FULL) again[tid] = r0 + tid <= r_last && !(sf > 0.0f && sf < INFINITY);
    if constexpr (!MASS) {
      mrow[tid] = mf;
      irow[tid] = sf > 0.0f ? 1.0f / sf : 0.0f;
    }
  }
  if constexpr (!MASS) {
    constexpr int U = D / 4;                                   // 16-byte units per output row
    constexpr int MT = AT::kMergeTiles;
    float4* area = reinterpret_cast<float4*>(lds);             // [tile][wavefront][16 rows][U]
    __syncthreads();
#pragma unroll
    for (int i0 = 0; i0 < RT; i0 += MT) {
      if (i0 > 0) __syncthreads();                             // the previous tiles are read
#pragma unroll
      for (int i = i0; i < i0 + MT && i < RT; ++i) {
        const float f = rescale(m[i], mrow[i * 16 + c16]);
#pragma unroll
        for (int dt = 0; dt < AT::kDT; ++dt)
          area[(((i - i0) * W + wv) * 16 + c16) * U + ((dt * 4 + g16) ^ c16)] =
              make_float4(o[i][dt][0] * f, o[i][dt][1] * f, o[i][dt][2] * f, o[i][dt][3] * f);
      }
      __syncthreads();
      const int rows = min(MT * 16, r_last + 1 - r0 - i0 * 16);   // rows of these tiles to write
      for (int e = tid; e < rows * U; e += AT::kThreads) {
        const int row = e / U, u = e % U, c = row & 15;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const float4 p = area[(((row >> 4) * W + w) * 16 + c) * U + (u ^ c)];
          sum.x += p.x;
          sum.y += p.y;
          sum.z += p.z;
          sum.w += p.w;
        }
        const float inv = irow[i0 * 16 + row];
        sum = make_float4(sum.x * inv, sum.y * inv, sum.z * inv, sum.w * inv);
        *reinterpret_cast<float4*>(a.out + (row_base + r0 + i0 * 16 + row) * D + 4 * u) = sum;
        if constexpr (FULL) {                                  // NaN unless all four are finite
          if (!((sum.x + sum.y + sum.z + sum.w) * 0.0f == 0.0f)) again[i0 * 16 + row] = 1;
        }
      }
    }
  }
  if constexpr (FULL) {
    __syncthreads();
    for (int r = r0; r <= r_last; ++r)                         // uniform
      if (again[r - r0]) attend_row<D, MASS>(a, row_base + r, kc, vc, visible(r), lds);
  }
}

// beta[b][h] and l_match[b][h]: means of rho and -log(1 - rho) over the G * n_q rows of
// (sequence b, KV head h), one wavefront each, summed in a fixed order.
__global__ __launch_bounds__(64) void mass_reduce_kernel(AttArgs a) {
  const int b = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
  const int n = a.G * a.n_q;
  const int64_t q_rows = (int64_t)a.batch * a.n_q;
  float s_rho = 0.0f, s_def = 0.0f;
  for (int i = lane; i < n; i += 64) {
    const int g = i / a.n_q, r = i - g * a.n_q;
    const float rho = a.rho[(int64_t)(h * a.G + g) * q_rows + b * a.n_q + r];
    s_rho += rho;
    s_def += -log1pf(-rho);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    s_rho += __shfl_xor(s_rho, off, 64);
    s_def += __shfl_xor(s_def, off, 64);
  }
  if (lane == 0) {
    a.beta[b * a.n_kv_heads + h] = s_rho / (float)n;
    a.l_match[b * a.n_kv_heads + h] = s_def / (float)n;
  }
}

template <int D, bool MASS>
hipError_t launch_att_f32(const AttArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((cache_attention_f32_kernel<D, MASS>), dim3(a.batch * a.n_q, a.n_kv_heads),
                     dim3(kAttThreads), 0, st, a);
  if constexpr (MASS)
    hipLaunchKernelGGL(mass_reduce_kernel, dim3(a.batch, a.n_kv_heads), dim3(64), 0, st, a);
  return hipGetLastError();
}

template <int D, int RT, bool MASS, bool FULL>
hipError_t launch_att_wave(const AttArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((cache_attention_wave_kernel<D, RT, MASS, FULL>),
                     dim3(xcd_grid(a.batch * a.n_kv_heads * a.G * a.row_blocks)),
                     dim3((AttWave<D, RT, MASS>::kThreads)), 0, st, a);
  if constexpr (MASS)
    hipLaunchKernelGGL(mass_reduce_kernel, dim3(a.batch, a.n_kv_heads), dim3(64), 0, st, a);
  return hipGetLastError();
}

// Row blocks of at most three 16-row tiles (what a wavefront's registers hold next to the
// outputs), as equal as they come: 4 tiles are two blocks of two.
template <int D, bool MASS, bool FULL>
hipError_t launch_att_blocks(AttArgs a, hipStream_t st) {
  const int tiles = (a.n_q + 15) / 16;
  a.row_blocks = (tiles + 2) / 3;
  const int rt = (tiles + a.row_blocks - 1) / a.row_blocks;
  if (rt == 1) return launch_att_wave<D, 1, MASS, FULL>(a, st);
  if (rt == 2) return launch_att_wave<D, 2, MASS, FULL>(a, st);
  return launch_att_wave<D, 3, MASS, FULL>(a, st);
}

// FULL weights (see the kernel) but for the calls that have always had weights of two parts:
// the attention at d = 128 and at most 64 rows.  The evicted mass has no weights; beyond 64
// rows it keeps attend_row for sums that are not finite.
template <int D, bool MASS>
hipError_t launch_att_rows(const AttArgs& a, hipStream_t st) {
  if (a.n_q > 64 || (!MASS && D == 64)) return launch_att_blocks<D, MASS, true>(a, st);
  return launch_att_blocks<D, MASS, false>(a, st);
}

template <bool MASS>
hipError_t launch_att_typed(const dge_geom_t& g, const AttArgs& a, hipStream_t st) {
  if (g.dtype == DGE_BF16)
    return g.head_dim == 128 ? launch_att_rows<128, MASS>(a, st) : launch_att_rows<64, MASS>(a, st);
  return g.head_dim == 128 ? launch_att_f32<128, MASS>(a, st) : launch_att_f32<64, MASS>(a, st);
}

}  // namespace

int cache_attention_max_group() { return kMaxAttG; }

hipError_t launch_cache_attention(const dge_geom_t& g, const void* q, int n_q, int q_from_end,
                                  const void* k_c, const void* v_c, int n_select, int n_tail,
                                  const int32_t* n_kept, float* out, float* lse,
                                  hipStream_t st) {
  AttArgs a{};
  a.q = q;
  a.k = k_c;
  a.v = v_c;
  a.n_kept = n_kept;
  a.out = out;
  a.lse = lse;
  a.batch = g.batch;
  a.n_kv_heads = g.n_kv_heads;
  a.G = g.n_q_heads / g.n_kv_heads;
  a.n_q = n_q;
  a.q_from_end = q_from_end;
  a.n_select = n_select;
  a.n_tail = n_tail;
  a.n_out = n_select + n_tail;
  a.scale_log2 = kLog2e / sqrtf((float)g.head_dim);
  return launch_att_typed<false>(g, a, st);
}

hipError_t launch_evicted_mass(const dge_geom_t& g, const void* q, int n_q, int q_from_end,
                               const void* k_c, int n_select, int n_tail, const int32_t* n_kept,
                               const float* lse_full, float* rho, float* beta, float* l_match,
                               hipStream_t st) {
  AttArgs a{};
  a.q = q;
  a.k = k_c;
  a.n_kept = n_kept;
  a.lse_full = lse_full;
  a.rho = rho;
  a.beta = beta;
  a.l_match = l_match;
  a.batch = g.batch;
  a.n_kv_heads = g.n_kv_heads;
  a.G = g.n_q_heads / g.n_kv_heads;
  a.n_q = n_q;
  a.q_from_end = q_from_end;
  a.n_select = n_select;
  a.n_tail = n_tail;
  a.n_out = n_select + n_tail;
  a.scale_log2 = kLog2e / sqrtf((float)g.head_dim);
  return launch_att_typed<true>(g, a, st);
}

}  // namespace dge
