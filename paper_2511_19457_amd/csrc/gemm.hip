// Implicit-GEMM convolution on the gfx950 matrix cores (MFMA), dense and
// zero-skipping.  Fully connected layers run through the same kernel as a
// 1x1 convolution over m "pixels".
//
// GEMM view of conv (NHWC activations, [c_out][kh][kw][c_in] weights):
//   rows  m = (n, oh, ow)                      M = n * ho * wo
//   cols  j = output channel                   N = c_out
//   depth k = (r, s, c) = (r*kw + s)*c_in + c  K = kh * kw * c_in
//   A[m][k] = x[n][oh*sh - ph + r*dh][ow*sw - pw + s*dw][c]  (0 outside)
//   B[j][k] = w[j][r][s][c]                     (row j of w, contiguous in k)
//
// Work-group = 256 threads = 4 waves in a 2 x 2 layout; the tile is
// BM x BN with BM = 32*TM, BN = 32*TN, each wave owning (BM/2) x (BN/2) as
// TM x TN MFMA 16x16 blocks.  The K loop walks chunks of 32 k values; A and B
// chunks are staged global -> registers -> LDS (double buffered, one barrier
// per chunk) and fed to v_mfma_f32_16x16x32_{bf16,f16} (one per block per
// chunk) or v_mfma_f32_16x16x4_f32 (eight per block per chunk).
//
// Zero skipping (SparOA Section 2.1: zero activations can be skipped without
// changing the output): the skip variant reads the activation bitmap written
// by the measurement kernel at one bit per (pixel, 8 channels).  At start-up
// each work-group ORs, for every pixel its tile gathers at every tap, those
// bits into an LDS bit vector over K/8 (the nonzero 8-wide K slices of its
// tile), turns it into one flag per 32-wide chunk, and compacts the nonzero
// chunk indices into an LDS list (ballot + popcount prefix).  The main loop
// then walks only that list: skipped chunks cost neither global/LDS traffic
// nor MFMA issue.  Because the chunk order and the MFMA block decomposition
// are those of the dense variant, and a skipped chunk would only have added
// exact zeros, the skip output equals the dense output bit for bit (for
// finite weights).
#include <type_traits>

#include "commit.h"
#include "common.h"
#include "dtype.h"

namespace sparoa {
namespace {

constexpr int kThreads = 256;
constexpr int kBK = 32;            // K values per chunk (skip granularity)
constexpr int kMaxChunks = 2048;   // K <= 65536 on the skip path
constexpr int kMaxVecWords = kMaxChunks * kBK / 8 / 32;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
  const char *x;
  const char *w;
  const char *bias;
  const char *residual;
  char *y;
  float *partial;
  const uint32_t *mask;
  unsigned long long *executed;
  int64_t M, N, K;
  int64_t H, W, Cin, Ho, Wo, Kw, sh, sw, ph, pw, dh, dw, taps;
  int64_t nchunks, chunks_per_split;
  int64_t x_bytes, w_bytes;  // buffer-descriptor ranges (second-generation kernel)
  float inv_wo, inv_ho;      // 1 / Wo, 1 / Ho rounded once on the host (float divmod)
  // 32-bit tile walk of the second-generation kernel (every value below
  // 2^24; the host checks the tile count): column tiles, row x column tiles
  // per split, chunks per tap, kernel rows, and the reciprocals of the
  // divisors rounded once (float divmod)
  int ntn32, ntmn32, cpt32, kh32;
  float inv_ntmn, inv_cpt, inv_kw, inv_dh, inv_dw;
  // column groups of the tile walk: gw column tiles a group (the last one
  // lastw), gt = row tiles x gw
  int gw32, gt32, lastw32;
  // first output row of the launch, and the rows that skip together (the
  // reported tile rows; both multiples of them)
  int row0, skip_rows;
  float inv_gt, inv_gw, inv_lastw;
  int act;
  int split;
  DeviceRoute route;
  sparoa_counts *om_counts;  // non-null: the epilogue measures y (OutMeasure)
  uint32_t *om_mask;
  unsigned long long *om_words;  // grouped count commit words, or null
};

template <int DT>
__device__ __forceinline__ f32x4 mfma_chunk(const char *a_row, const char *b_row, f32x4 acc,
                                            int g) {
  if constexpr (DT == SPAROA_BF16) {
    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(a_row + 16 * g);
    const bf16x8 b = *reinterpret_cast<const bf16x8 *>(b_row + 16 * g);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
  } else if constexpr (DT == SPAROA_F16) {
    const f16x8 a = *reinterpret_cast<const f16x8 *>(a_row + 16 * g);
    const f16x8 b = *reinterpret_cast<const f16x8 *>(b_row + 16 * g);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
  } else {
    // Lane group g holds k = 16h + 4g + e of both operands; the four MFMAs
    // over e cover the 16 k values of half h.
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 a = *reinterpret_cast<const f32x4 *>(a_row + 64 * h + 16 * g);
      const f32x4 b = *reinterpret_cast<const f32x4 *>(b_row + 64 * h + 16 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
    }
    return acc;
  }
}

// q = n / d, r = n % d for 0 <= n < 2^24 and 0 < d < 2^24: the float
// quotient is within one of the true one, then one integer correction,
// written as selects (no branch: a kernel's start keeps one basic block, so
// its kernel-argument loads are issued together rather than one round trip
// per block)
__device__ __forceinline__ void divmod_small(int n, int d, float inv_d, int &q, int &r) {
  const int q0 = (int)((float)n * inv_d);
  const int r0 = n - q0 * d;
  const bool lo = r0 < 0, hi = r0 >= d;
  q = lo ? q0 - 1 : (hi ? q0 + 1 : q0);
  r = lo ? r0 + d : (hi ? r0 - d : r0);
}


// Bit t set for the taps t of [0, k) whose input coordinate o + t d lies in
// [0, n): t from ceil(-o / d) to ceil((n - o) / d), clipped to [0, k <= 32)
// (no branch; inv_d = 1 / d rounded once).
__device__ __forceinline__ uint32_t taps_inside(int o, int n, int k, int d, float inv_d) {
  int lo, hi, rem;
  divmod_small(max(-o, 0) + d - 1, d, inv_d, lo, rem);
  divmod_small(max(n - o, 0) + d - 1, d, inv_d, hi, rem);
  lo = min(lo, k);
  hi = min(hi, k);
  const uint32_t mhi = hi >= 32 ? ~0u : (1u << hi) - 1u;
  const uint32_t mlo = lo >= 32 ? ~0u : (1u << lo) - 1u;
  return hi > lo ? mhi & ~mlo : 0u;
}

// Reads n <= 32 bits starting at bit `pos` of a bitmap.
__device__ __forceinline__ uint32_t read_bits(const uint32_t *m, int64_t pos, int n) {
  const int64_t wd = pos >> 5;
  const int off = (int)(pos & 31);
  uint32_t v = m[wd] >> off;
  if (off + n > 32) v |= m[wd + 1] << (32 - off);
  return n == 32 ? v : (v & ((1u << n) - 1u));
}

// ORs n <= 32 bits into an LDS bitmap at bit `pos`.
__device__ __forceinline__ void lds_or_bits(uint32_t *m, int pos, uint32_t v, int n) {
  if (!v) return;
  const int wd = pos >> 5, off = pos & 31;
  atomicOr(m + wd, v << off);
  if (off && off + n > 32) atomicOr(m + wd + 1, v >> (32 - off));
}

template <int DT, int TM, int TN, bool VEC, bool SKIP>
__global__ __launch_bounds__(kThreads) void gemm_kernel(GemmArgs a) {
  using E = Elem<DT>;
  constexpr int ESZ = E::size;
  constexpr int BM = 32 * TM, BN = 32 * TN;
  constexpr int ROWB = kBK * ESZ + 16;   // LDS row stride (padding: conflict-free reads)
  constexpr int VPR = kBK * ESZ / 16;    // 16-byte vectors per chunk row
  constexpr int EPV = 16 / ESZ;          // elements per vector
  constexpr int AV = BM * VPR / kThreads;  // A vectors per thread
  constexpr int BV = BN * VPR / kThreads;  // B vectors per thread
  static_assert(AV >= 1 && BV >= 1, "tile too small for the work-group");

  __shared__ __attribute__((aligned(16))) char smem[2][(BM + BN) * ROWB];
  __shared__ int list[SKIP ? kMaxChunks : 1];
  __shared__ uint32_t nzvec[SKIP ? kMaxVecWords : 1];
  __shared__ int list_len;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t m0 = (int64_t)blockIdx.x * BM, n0 = (int64_t)blockIdx.y * BN;
  const int64_t c_begin = (int64_t)blockIdx.z * a.chunks_per_split;
  const int64_t c_end = min(c_begin + a.chunks_per_split, a.nchunks);

  // ---- per-thread A rows (fixed over the K loop) --------------------------
  // A vector q = tid + kThreads*u covers row q / VPR, vector column q % VPR.
  int64_t a_pix[AV];  // n * H * W, or -1 when the row is past M
  int a_h0[AV], a_w0[AV];
  const uint32_t cin = (uint32_t)a.Cin, kw = (uint32_t)a.Kw, kdim = (uint32_t)a.K;
  const int H = (int)a.H, W = (int)a.W, dh = (int)a.dh, dw = (int)a.dw;
#pragma unroll
  for (int u = 0; u < AV; ++u) {
    const int q = tid + kThreads * u;
    const int64_t m = m0 + q / VPR;
    if (m < a.M) {
      const int64_t ow = m % a.Wo, oh = (m / a.Wo) % a.Ho, nn = m / (a.Wo * a.Ho);
      a_pix[u] = nn * a.H * a.W;
      a_h0[u] = (int)(oh * a.sh - a.ph);
      a_w0[u] = (int)(ow * a.sw - a.pw);
    } else {
      a_pix[u] = -1;
      a_h0[u] = a_w0[u] = 0;
    }
  }

  // ---- chunk list (skip variant) -------------------------------------------
  int64_t count = c_end - c_begin;
  bool use_list = SKIP;
  if constexpr (SKIP) {
    if (a.route.counts) {
      use_list = device_route_skip(a.route);
      if (a.route.path_out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid == 0)
        *a.route.path_out = (use_list ? 1u : 0u) | ((uint32_t)a.route.bw_bit << 1);
    }
  }
  if constexpr (!SKIP) {
    if (a.route.path_out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid == 0)
      *a.route.path_out = (uint32_t)a.route.bw_bit << 1;
  }
  if (SKIP && use_list) {
    const int cpg = (int)((a.Cin + 7) / 8);  // bitmap blocks per pixel
    const int kv_words = (int)((a.taps * cpg + 31) / 32);
    for (int i = tid; i < kv_words; i += kThreads) nzvec[i] = 0u;
    __syncthreads();
    for (int64_t p = tid; p < (int64_t)BM * a.taps; p += kThreads) {
      const int r_in = (int)(p / a.taps);
      const int tap = (int)(p - (int64_t)r_in * a.taps);
      const int64_t m = m0 + r_in;
      if (m >= a.M) continue;
      const int64_t ow = m % a.Wo, oh = (m / a.Wo) % a.Ho, nn = m / (a.Wo * a.Ho);
      const int64_t r = tap / a.Kw, s = tap - r * a.Kw;
      const int64_t ih = oh * a.sh - a.ph + r * a.dh, iw = ow * a.sw - a.pw + s * a.dw;
      if (ih < 0 || ih >= a.H || iw < 0 || iw >= a.W) continue;
      const int64_t pix = (nn * a.H + ih) * a.W + iw;
      for (int b = 0; b < cpg; b += 32) {
        const int nb = min(32, cpg - b);
        lds_or_bits(nzvec, tap * cpg + b, read_bits(a.mask, pix * cpg + b, nb), nb);
      }
    }
    __syncthreads();
    if (wave == 0) {
      int total = 0;
      for (int64_t base = c_begin; base < c_end; base += 64) {
        const int64_t j = base + lane;
        bool nz = false;
        if (j < c_end) {
          // walk the chunk's k range one (tap, 8-channel block) run at a time
          uint32_t k = (uint32_t)(j * kBK);
          const uint32_t kend = (uint32_t)min(j * kBK + kBK, a.K);
          while (k < kend) {
            const uint32_t tap = k / cin, c = k - tap * cin;
            const uint32_t bit = tap * (uint32_t)cpg + c / 8;
            nz |= (nzvec[bit >> 5] >> (bit & 31)) & 1u;
            const uint32_t cnext = (c / 8 + 1) * 8;
            k = tap * cin + (cnext < cin ? cnext : cin);
          }
        }
        const uint64_t bal = __ballot(nz);
        const int before = __popcll(bal & ((1ull << lane) - 1ull));
        if (nz) list[total + before] = (int)j;
        total += __popcll(bal);
      }
      if (lane == 0) {
        list_len = total;
        if (a.executed && blockIdx.y == 0 && total)
          atomicAdd(a.executed, (unsigned long long)total);
      }
    }
    __syncthreads();
    count = list_len;
  }

  // ---- global -> register staging of one chunk -----------------------------
  uint4 ra[AV], rb[BV];
  auto load_chunk = [&](int64_t j) {
    const int64_t kbase = j * kBK;
#pragma unroll
    for (int u = 0; u < AV; ++u) {
      const int q = tid + kThreads * u;
      uint4 v = make_uint4(0, 0, 0, 0);
      if constexpr (VEC) {
        const uint32_t k = (uint32_t)kbase + (uint32_t)(q % VPR) * EPV;
        if (a_pix[u] >= 0 && k < kdim) {
          const uint32_t tap = k / cin, c = k - tap * cin;
          const uint32_t r = tap / kw, s = tap - r * kw;
          const int ih = a_h0[u] + (int)r * dh, iw = a_w0[u] + (int)s * dw;
          if (ih >= 0 && ih < H && iw >= 0 && iw < W)
            v = *reinterpret_cast<const uint4 *>(
                a.x + ((a_pix[u] + (int64_t)ih * W + iw) * a.Cin + c) * ESZ);
        }
      } else {
        typename E::raw e[EPV];
#pragma unroll
        for (int t = 0; t < EPV; ++t) {
          e[t] = 0;
          const uint32_t k = (uint32_t)kbase + (uint32_t)(q % VPR) * EPV + t;
          if (a_pix[u] >= 0 && k < kdim) {
            const uint32_t tap = k / cin, c = k - tap * cin;
            const uint32_t r = tap / kw, s = tap - r * kw;
            const int ih = a_h0[u] + (int)r * dh, iw = a_w0[u] + (int)s * dw;
            if (ih >= 0 && ih < H && iw >= 0 && iw < W)
              e[t] = reinterpret_cast<const typename E::raw *>(
                  a.x)[(a_pix[u] + (int64_t)ih * W + iw) * a.Cin + c];
          }
        }
        __builtin_memcpy(&v, e, 16);
      }
      ra[u] = v;
    }
#pragma unroll
    for (int u = 0; u < BV; ++u) {
      const int q = tid + kThreads * u;
      const int64_t jn = n0 + q / VPR;
      const int64_t k = kbase + (q % VPR) * EPV;
      uint4 v = make_uint4(0, 0, 0, 0);
      if constexpr (VEC) {
        if (jn < a.N && k < a.K) v = *reinterpret_cast<const uint4 *>(a.w + (jn * a.K + k) * ESZ);
      } else {
        typename E::raw e[EPV];
#pragma unroll
        for (int t = 0; t < EPV; ++t)
          e[t] = (jn < a.N && k + t < a.K)
                     ? reinterpret_cast<const typename E::raw *>(a.w)[jn * a.K + k + t]
                     : (typename E::raw)0;
        __builtin_memcpy(&v, e, 16);
      }
      rb[u] = v;
    }
  };
  auto store_chunk = [&](int buf) {
#pragma unroll
    for (int u = 0; u < AV; ++u) {
      const int q = tid + kThreads * u;
      *reinterpret_cast<uint4 *>(&smem[buf][(q / VPR) * ROWB + (q % VPR) * 16]) = ra[u];
    }
#pragma unroll
    for (int u = 0; u < BV; ++u) {
      const int q = tid + kThreads * u;
      *reinterpret_cast<uint4 *>(&smem[buf][(BM + q / VPR) * ROWB + (q % VPR) * 16]) = rb[u];
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto chunk_at = [&](int64_t i) -> int64_t {
    return (SKIP && use_list) ? (int64_t)list[i] : c_begin + i;
  };

  const int g = lane >> 4, rl = lane & 15;
  if (count > 0) {
    load_chunk(chunk_at(0));
    store_chunk(0);
    __syncthreads();
    for (int64_t i = 0; i < count; ++i) {
      const int buf = (int)(i & 1);
      const bool more = i + 1 < count;
      if (more) load_chunk(chunk_at(i + 1));
      const char *As = &smem[buf][0];
      const char *Bs = &smem[buf][BM * ROWB];
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) {
        const char *arow = As + (wm * (BM / 2) + tm * 16 + rl) * ROWB;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          const char *brow = Bs + (wn * (BN / 2) + tn * 16 + rl) * ROWB;
          acc[tm][tn] = mfma_chunk<DT>(arow, brow, acc[tm][tn], g);
        }
      }
      if (more) store_chunk(buf ^ 1);
      __syncthreads();
    }
  }

  // ---- epilogue ------------------------------------------------------------
  // MFMA 16x16 output layout: lane holds rows 4*(lane/16) + v, column lane%16.
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t row = m0 + wm * (BM / 2) + tm * 16 + 4 * g + v;
        const int64_t col = n0 + wn * (BN / 2) + tn * 16 + rl;
        if (row >= a.M || col >= a.N) continue;
        const float val = acc[tm][tn][v];
        if (a.split > 1) {
          a.partial[((int64_t)blockIdx.z * a.M + row) * a.N + col] = val;
        } else {
          float o = val;
          if (a.bias) o += E::to_f32(reinterpret_cast<const typename E::raw *>(a.bias)[col]);
          if (a.residual)
            o += E::to_f32(reinterpret_cast<const typename E::raw *>(a.residual)[row * a.N + col]);
          reinterpret_cast<typename E::raw *>(a.y)[row * a.N + col] = E::from_f32(apply_act(o, a.act));
        }
      }
}

// Sums the K-split partials in split order, adds bias and residual, then
// applies the activation.  Grouped form: up to kGroupMax reductions of one
// dtype in one launch, work-groups dealt to the jobs in proportion to their
// size.  A thread finishes 8 consecutive outputs (16-byte partial, bias and
// residual loads, one 16-byte store) when N % 8 == 0, else one.
struct ReduceGroup {
  int n;
  int wg_begin[kGroupMax + 1];
  const float *partial[kGroupMax];
  int split[kGroupMax];
  int64_t M[kGroupMax], N[kGroupMax];
  const char *bias[kGroupMax], *residual[kGroupMax];
  int act[kGroupMax];
  char *y[kGroupMax];
  sparoa_counts *om_counts[kGroupMax];  // non-null: measure y (16-bit, N % 8 == 0)
  uint32_t *om_mask[kGroupMax];
  unsigned long long *om_words[kGroupMax];
};

template <int DT>
__global__ __launch_bounds__(256) void split_reduce_group(ReduceGroup g) {
  using E = Elem<DT>;
  using raw = typename E::raw;
  // this work-group's job: the starts at or below blockIdx.x, counted over
  // fixed indices (their loads are issued together, not one per step)
  int j = 0;
#pragma unroll
  for (int q = 1; q < kGroupMax; ++q) j += (q < g.n && (int)blockIdx.x >= g.wg_begin[q]) ? 1 : 0;
  const int64_t b0 = blockIdx.x - g.wg_begin[j], nb = g.wg_begin[j + 1] - g.wg_begin[j];
  const int64_t M = g.M[j], N = g.N[j], total = M * N;
  const float *partial = g.partial[j];
  const int split = g.split[j], act = g.act[j];
  const raw *bias = reinterpret_cast<const raw *>(g.bias[j]);
  const raw *res = reinterpret_cast<const raw *>(g.residual[j]);
  raw *y = reinterpret_cast<raw *>(g.y[j]);
  // output measurement: vector v = block v at (1 row, 8 channels); a wave's
  // 64 consecutive vectors are two whole bitmap words (as in measure_lanebit)
  sparoa_counts *om = E::size == 2 ? g.om_counts[j] : nullptr;
  uint32_t *om_mask = g.om_mask[j];   // null: counts only
  const int lane = threadIdx.x & 63;
  const int64_t om_words = om_mask ? (total / 8 + 31) / 32 : 0;
  uint32_t om_zeros = 0, om_nz = 0;
  if (N % 8 == 0) {
    // the column advances by a fixed step mod N (one division per thread)
    const int64_t step = nb * 256;
    int64_t col = ((b0 * 256 + threadIdx.x) * 8) % N;
    const int64_t col_step = (step * 8) % N;
    for (int64_t v = b0 * 256 + threadIdx.x; v < total / 8;
         v += step, col = col + col_step >= N ? col + col_step - N : col + col_step) {
      const int64_t i = v * 8;
      float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      // the slices' partial sums added in slice order (the rounding of the
      // reduction is fixed), four slices' loads in flight at a time
      int z = 0;
      for (; z + 4 <= split; z += 4) {
        float4 lo[4], hi[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          lo[u] = *reinterpret_cast<const float4 *>(partial + (z + u) * total + i);
          hi[u] = *reinterpret_cast<const float4 *>(partial + (z + u) * total + i + 4);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          o[0] += lo[u].x; o[1] += lo[u].y; o[2] += lo[u].z; o[3] += lo[u].w;
          o[4] += hi[u].x; o[5] += hi[u].y; o[6] += hi[u].z; o[7] += hi[u].w;
        }
      }
      for (; z < split; ++z) {
        const float4 lo = *reinterpret_cast<const float4 *>(partial + z * total + i);
        const float4 hi = *reinterpret_cast<const float4 *>(partial + z * total + i + 4);
        o[0] += lo.x; o[1] += lo.y; o[2] += lo.z; o[3] += lo.w;
        o[4] += hi.x; o[5] += hi.y; o[6] += hi.z; o[7] += hi.w;
      }
      raw t[8];
      if (bias) {
        if constexpr (E::size == 2) {
          const uint4 q = *reinterpret_cast<const uint4 *>(bias + col);
          __builtin_memcpy(t, &q, 16);
        } else {
          for (int e = 0; e < 8; ++e) t[e] = bias[col + e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += E::to_f32(t[e]);
      }
      if (res) {
        if constexpr (E::size == 2) {
          const uint4 q = *reinterpret_cast<const uint4 *>(res + i);
          __builtin_memcpy(t, &q, 16);
        } else {
          for (int e = 0; e < 8; ++e) t[e] = res[i + e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += E::to_f32(t[e]);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = E::from_f32(apply_act(o[e], act));
      if constexpr (E::size == 2) {
        uint4 q;
        __builtin_memcpy(&q, t, 16);
        *reinterpret_cast<uint4 *>(y + i) = q;
        if (om) {
          uint32_t nzb = 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const bool z = (t[e] & 0x7FFFu) == 0u;
            om_zeros += z ? 1u : 0u;
            nzb |= z ? 0u : 1u;
          }
          om_nz += nzb;
          const uint64_t bal = __ballot(nzb != 0u);
          const int64_t w0 = (v - lane) >> 5;
          if (lane == 0 && w0 < om_words) om_mask[w0] = (uint32_t)bal;
          if (lane == 32 && w0 + 1 < om_words) om_mask[w0 + 1] = (uint32_t)(bal >> 32);
        }
      } else {
        for (int e = 0; e < 8; ++e) y[i + e] = t[e];
      }
    }
    if (om) om_commit(om_zeros, om_nz, om, g.om_words[j], b0, nb);
  } else {
    for (int64_t i = b0 * 256 + threadIdx.x; i < total; i += nb * 256) {
      float o = 0.f;
      for (int z = 0; z < split; ++z) o += partial[z * total + i];
      const int64_t col = i % N;
      if (bias) o += E::to_f32(bias[col]);
      if (res) o += E::to_f32(res[i]);
      y[i] = E::from_f32(apply_act(o, act));
    }
  }
}

// ---------------------------------------------------------------------------
// Second-generation implicit GEMM for the common case: 16-bit data, groups 1,
// C_in % 64 == 0.  A K chunk is 64 channels of one tap, so the tap and
// channel offset of a chunk are work-group-uniform scalars (no per-vector
// division), and a thread's gathered pixels only move by the tap offset.
// Work-group = WGM x WGN waves; a wave owns 16 WTM pixels x 16 WTN channels,
// which sets the LDS bytes read per MFMA.  Chunks go straight from memory to
// a ring of S stages in LDS (buffer loads with an LDS destination: no staging
// registers and no LDS write instructions); a tap outside the image has its
// offset past the descriptor's range and lands as zeros.  One barrier per
// chunk; a wave reads a chunk's MFMA operands from LDS, and sends the loads
// that refill the stage freed by the barrier, between the MFMAs of the chunk
// before.  The MFMA's rows are channels, so a lane ends with 8 consecutive
// output channels of a pixel per block pair, four lanes with 32, and the
// epilogue needs no LDS (but for output rows that start anywhere, C_out % 8).
// Bounds, measured with the other parts switched off (4096^3 fp16, 128 x 256:
// 117 us): MFMAs alone 97 us (1.6 PFLOP/s with its start and end), loads
// alone 95 us (17 TB/s out of the L2s); small tiles are bound by the loads
// (64 x 64: 293 us with or without MFMAs).  Against the form that staged
// chunks through registers, with two barriers' worth of LDS writes and an
// epilogue through LDS: 4096^3 155 -> 117 us; 2048 x 768 x 3072 31 -> 19 us;
// 3 x 3 512 -> 512 at 7 x 7, N = 32 29 -> 18 us; 3 x 3 256 -> 256 at 56 x 56,
// N = 32 164 -> 137 us (about 16 less with the rows past whole rounds apart,
// ig_head_rows); K = 64 alone (start and epilogue), 4096 x 4096 20 ->
// 12 us.  The ring's depth, beyond what one chunk's MFMAs cover, and more
// waves of smaller tiles change nothing; branches and scalar arithmetic in
// the loop did (a step written with guards: 20 % slower).
// Work-groups walk their tiles XCD by XCD (tile_of).  The skip form walks
// only the (tap, 64-channel) chunks in which some gathered pixel of the tile
// is nonzero, in dense order, so its output equals the dense form's bit for
// bit.
constexpr int kBK2 = 64;
constexpr int kMaxChunks2 = 1024;          // K <= 65536 on the skip path

// s_waitcnt immediate: at most n vector-memory operations outstanding, the
// other counters not waited for.
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }
constexpr int kLgkmcnt0 = 15 | (7 << 4) | (3 << 14);   // LDS operations done

// Waits until all but the `chunks` <= C newest chunks' loads (L per chunk) of
// this wave have landed.
template <int C, int L>
__device__ __forceinline__ void wait_chunks(int chunks) {
  static_assert(C * L < 64, "vmcnt range");
  if constexpr (C > 0) {
    if (chunks < C) return wait_chunks<C - 1, L>(chunks);
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(C * L));
}

// A 16-byte-per-lane buffer load whose data goes to LDS: lane l's 16 bytes
// land at LDS address lds + 16 l (lds uniform), zeros where the offset lies
// past the descriptor's range.  In assembly and not by the builtin: the
// compiler cannot tell the ring's stages apart and would wait for every load
// in flight before each LDS read; the waits are written out at the barriers
// instead (wait_chunks).  No register is written, so the compiler's own
// counting of other loads only waits longer than it has to.  (m0 is bound by
// the operand, so the compiler knows what it holds; one wait state between its
// write and its use.)
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, uint32_t lds, int voffset, int soffset) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "{m0}"(lds), "v"(voffset), "s"(rsrc), "s"(soffset)
               : "memory");
}
__device__ __forceinline__ u32x4 buffer_words(const void *p, int64_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(p);
  return u32x4{(uint32_t)b, (uint32_t)(b >> 32) & 0xFFFFu, (uint32_t)bytes, (uint32_t)kBufDword3};
}

// Tile walk of the second-generation kernels: work-group -> (K split, row
// tile, column tile).  Work-groups are dealt round-robin to the 8 XCDs, so
// XCD i gets the i-th contiguous range of tile ids (SPREAD: every eighth),
// and a tile id walks (split, column group, row tile, column tile of the
// group) with the column tiles innermost: the tiles that gather the same input rows run together in
// one XCD's L2.  The groups (host: ig_column_groups) keep an XCD to a part
// of the weights where these are what its L2 would re-read.  (32-bit
// arithmetic with float-reciprocal division: a 64-bit division by a runtime
// value is a long scalar sequence on the critical path of every
// work-group's start.)
struct TileId {
  int tile, zsplit, mt, nt;
};
template <bool SPREAD = false>
__device__ __forceinline__ TileId tile_of(const GemmArgs &a) {
  TileId t;
  const int vid = (int)blockIdx.x, ntiles = (int)gridDim.x;
  // (XCD i holds the i-th range: q + 1 tiles for the first r XCDs, q after)
  t.tile = SPREAD ? vid : (vid & 7) * (ntiles >> 3) + min(vid & 7, ntiles & 7) + (vid >> 3);
  int rest, grp;
  divmod_small(t.tile, a.ntmn32, a.inv_ntmn, t.zsplit, rest);
  divmod_small(rest, a.gt32, a.inv_gt, grp, rest);
  const bool last = (grp + 1) * a.gw32 >= a.ntn32;
  divmod_small(rest, last ? a.lastw32 : a.gw32, last ? a.inv_lastw : a.inv_gw, t.mt, t.nt);
  t.nt += grp * a.gw32;
  return t;
}

// Chunk j of the walk (C channels of ESZ bytes of one tap) as its loads need
// it: 31 - r | 31 - s << 5 | kofs / 16 << 10, with the kernel row r and column
// s of its tap and its byte offset kofs < 2^18 in a weight row; PART: bit 31
// marks the last chunk of a tap (C_in % C != 0: the partial one).
template <int C, int ESZ, bool PART>
__device__ __forceinline__ uint32_t walk_entry(const GemmArgs &a, int j) {
  int t, cb, r, sx;
  divmod_small(j, a.cpt32, a.inv_cpt, t, cb);
  divmod_small(t, (int)a.Kw, a.inv_kw, r, sx);
  const uint32_t e =
      (uint32_t)((31 - r) | (31 - sx) << 5 | ((t * (int)a.Cin + cb * C) * ESZ / 16) << 10);
  return PART && cb == a.cpt32 - 1 ? e | 0x80000000u : e;
}
// A walk entry read as scalars (it is the same in every lane).  xofs: byte
// offset of the chunk's channels from a row's first gathered pixel, from kofs
// and the per-row and per-column differences of the two layouts.
struct WalkStep {
  int kofs, xofs;
  uint32_t rsh, ssh;   // 31 - r, 31 - s: moves tap bit r / s to bit 31
  uint32_t last;       // PART: all ones in a tap's last chunk, else 0
};
struct WalkGeom {
  uint32_t dr, ds, base;
};
template <int ESZ>
__device__ __forceinline__ WalkGeom walk_geom(const GemmArgs &a) {
  WalkGeom g;
  g.dr = (uint32_t)(((int)a.dh * (int)a.W - (int)a.Kw) * (int)a.Cin * ESZ);
  g.ds = (uint32_t)(((int)a.dw - 1) * (int)a.Cin * ESZ);
  g.base = 31u * (g.dr + g.ds);
  return g;
}
template <bool PART>
__device__ __forceinline__ WalkStep walk_step(const WalkGeom &g, uint32_t entry) {
  const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)entry);
  WalkStep w;
  w.rsh = e & 31u;
  w.ssh = e >> 5 & 31u;
  w.last = PART ? (uint32_t)((int)e >> 31) : 0u;
  w.kofs = (int)((PART ? e & 0x7fffffffu : e) >> 10 << 4);
  w.xofs = (int)((uint32_t)w.kofs + g.base - w.rsh * g.dr - w.ssh * g.ds);
  return w;
}

// ORs the bitmap bits of every pixel that rows [m0, m0 + rows) gather at
// every tap into nzvec, bit tap * (C_in / 8) + channel block (plus a cleared
// spare word for windows past the end).  Whole work-group, NT threads; ends
// with a barrier.  (32-bit index arithmetic: pixel indices are below 2^24.)
template <int NT>
__device__ __forceinline__ void gather_nonzero_bits(const GemmArgs &a, int m0, int rows,
                                                    uint32_t *nzvec) {
  const int tid = threadIdx.x;
  const int H = (int)a.H, W = (int)a.W, Ho = (int)a.Ho, Wo = (int)a.Wo, kw = (int)a.Kw;
  const int cpg = (int)(a.Cin / 8);  // bitmap blocks per pixel
  const int kv_words = (int)((a.taps * cpg + 31) / 32) + 1;
  for (int i = tid; i < kv_words; i += NT) nzvec[i] = 0u;
  __syncthreads();
  const int taps = (int)a.taps, ntp = rows * taps;
  const float inv_taps = 1.0f / (float)taps, inv_kw = 1.0f / (float)kw;
  for (int p = tid; p < ntp; p += NT) {
    int r_in, tap, t1, ow, nn, oh, r, sx;
    divmod_small(p, taps, inv_taps, r_in, tap);
    const int m = m0 + r_in;
    if (m >= (int)a.M) continue;
    divmod_small(m, Wo, a.inv_wo, t1, ow);
    divmod_small(t1, Ho, a.inv_ho, nn, oh);
    divmod_small(tap, kw, inv_kw, r, sx);
    const int ih = oh * (int)a.sh - (int)a.ph + r * (int)a.dh;
    const int iw = ow * (int)a.sw - (int)a.pw + sx * (int)a.dw;
    if (ih < 0 || ih >= H || iw < 0 || iw >= W) continue;
    const int64_t pix = ((int64_t)nn * H + ih) * W + iw;
    for (int b = 0; b < cpg; b += 32) {
      const int nb = min(32, cpg - b);
      lds_or_bits(nzvec, tap * cpg + b, read_bits(a.mask, pix * cpg + b, nb), nb);
    }
  }
  __syncthreads();
}

// Whether chunk j (channels [C cb, min(C cb + C, Cin)) of tap t) has a
// nonzero: up to C / 8 bits from bit t cpg + (C / 8) cb of nzvec -- PART:
// read through a 64-bit window, since with cpg % (C / 8) != 0 they may
// straddle a word; whole chunks: inside one word.
template <int C, bool PART>
__device__ __forceinline__ bool chunk_nonzero(const GemmArgs &a, const uint32_t *nzvec, int j) {
  const int cpg = (int)(a.Cin / 8);
  int t, cb;
  divmod_small(j, a.cpt32, a.inv_cpt, t, cb);
  const int pos = t * cpg + (C / 8) * cb;
  if constexpr (PART) {
    const int nb = min(C / 8, cpg - (C / 8) * cb);
    const uint64_t win = (uint64_t)nzvec[pos >> 5] | ((uint64_t)nzvec[(pos >> 5) + 1] << 32);
    return ((win >> (pos & 31)) & ((1ull << nb) - 1ull)) != 0ull;
  } else {
    return ((nzvec[pos >> 5] >> (pos & 31)) & ((1u << (C / 8)) - 1u)) != 0u;
  }
}

// Split execution: a row tile's own route, from the zero counts of the
// samples its rows come from (one double division, >=, as sparoa_route).
__device__ __forceinline__ bool split_route_skips(const GemmArgs &a, int m0, int rows) {
  const int64_t last = min((int64_t)m0 + rows, a.M) - 1;
  const int64_t s0 = m0 / a.route.rows_per_sample, s1 = last / a.route.rows_per_sample;
  unsigned long long z = 0;
  for (int64_t q = s0; q <= s1; ++q) z += a.route.sample_zeros[q];
  const double n = (double)((unsigned long long)(s1 - s0 + 1) *
                            (unsigned long long)a.route.sample_numel);
  return (double)z / n >= a.route.sparsity_thr;
}

// PART: C_in % 64 != 0, a tap's last chunk is partial (a separate
// instantiation: the per-lane channel test and the per-chunk weight offset
// cost the whole-chunk kernels up to 10 %).
template <int DT, int WGM, int WGN, int WTM, int WTN, int S, bool PART>
__global__ __launch_bounds__(64 * WGM * WGN, 2) void igemm_kernel(GemmArgs a) {
  constexpr int NW = WGM * WGN;        // waves
  constexpr int NT = 64 * NW;          // threads per work-group
  constexpr int ROW = kBK2 * 2;        // bytes of a chunk row: 8 vectors of 16 bytes
  using E = Elem<DT>;
  using raw = typename E::raw;
  static_assert(E::size == 2, "16-bit types");
  constexpr int BM = WGM * 16 * WTM, BN = WGN * 16 * WTN;
  // a wave's 16-byte LDS-destination load covers 8 chunk rows
  constexpr int AV = BM / 8 / NW, BV = BN / 8 / NW;
  static_assert(AV >= 1 && BV >= 1 && BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile too small");
  static_assert(WTN % 4 == 0 && NW % 4 == 0, "a lane's 16 channels; B row swizzle");
  constexpr int L = AV + BV;           // loads in flight per wave and chunk
  constexpr int NG = WTN / 4;          // 64-channel groups of a wave
  constexpr int STAGE = (BM + BN) * ROW;

  __shared__ __attribute__((aligned(1024))) char smem[S * STAGE];
  __shared__ uint32_t list[kMaxChunks2];   // the chunks this tile walks, in order (walk_entry)
  __shared__ uint32_t nzvec[kMaxVecWords + 1];
  __shared__ int list_len;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  // The set-up's kernel arguments are requested in one round trip: this
  // empty statement needs them at the top (the compiler otherwise loads each
  // group just before its first use, behind branches, one round trip each).
  asm volatile("" ::"s"(a.M), "s"(a.N), "s"(a.H), "s"(a.W), "s"(a.Cin), "s"(a.Ho), "s"(a.Wo),
               "s"(a.Kw), "s"(a.sh), "s"(a.sw), "s"(a.ph), "s"(a.pw), "s"(gridDim.x),
               "s"(a.route.counts), "s"(a.route.path_out), "s"(a.om_counts));
  const bool om = a.om_counts != nullptr;
  // the device route's counts: their latency overlaps the tile's offset
  // arithmetic and the dense walk's list writes
  const RouteCountsReq rq = route_counts_request(a.route);
  const TileId tl = tile_of(a);
  const int zsplit = tl.zsplit;
  const int m0 = a.row0 + tl.mt * BM, n0 = tl.nt * BN;
  // a skip unit of several tiles is counted by its first
  const int unit = (int)a.skip_rows, u0 = m0 & ~(unit - 1);
  const bool first_tile = tl.tile == 0, first_col = tl.nt == 0 && u0 == m0;
  const int cps = (int)a.chunks_per_split;
  const int c_begin = zsplit * cps;
  const int c_end = min(c_begin + cps, (int)a.nchunks);
  const int M = (int)a.M, N = (int)a.N;

  // ---- LDS layout and this lane's share of the loads.  A wave's load fills
  // 8 rows of 128 bytes, lane l the slot l & 7 of row l >> 3.  Rows hold
  // their 16-byte vectors swizzled: slot = vector ^ f(row), so that the
  // operand reads of any 8 consecutive lanes hit distinct banks.  Pixel rows
  // are read 16 consecutive ones at a time, f = row & 7.  Channel rows are
  // read in the order that leaves a lane 8 consecutive output channels per
  // block pair (MFMA row 4 q + t of block b is channel 32 (b / 2) + 8 q +
  // 4 (b % 2) + t), f = (row >> 3 & 1) * 4 + (row & 3).
  const int lrow = lane >> 3;
  const int cgA = (lane & 7) ^ lrow;
  const int cgB = (lane & 7) ^ (((wave & 1) << 2) | (lrow & 3));

  // ---- gathered pixels of this lane's A rows (fixed over the K loop).
  // Loads go through buffer descriptors: a 32-bit byte offset per lane, and
  // an offset past the end (taps in the padding) reads 0 without touching
  // memory.
  const u32x4 xr = buffer_words(a.x, a.x_bytes), wr = buffer_words(a.w, a.w_bytes);
  int a_offb[AV];      // byte offset of (n, h0, w0, channel cgA*8)
  uint32_t orow[AV], ocol[AV];  // bit r / s: kernel row r / column s lies outside the image
  const int H = (int)a.H, W = (int)a.W, Ho = (int)a.Ho, Wo = (int)a.Wo, Cin = (int)a.Cin;
  const int kw = (int)a.Kw, dh = (int)a.dh, dw = (int)a.dw;
  const float inv_wo = a.inv_wo, inv_ho = a.inv_ho;
#pragma unroll
  for (int u = 0; u < AV; ++u) {
    const int m = m0 + 8 * (u * NW + wave) + lrow;
    const int mm = m < M ? m : 0;
    int t1, ow, nn, oh;
    divmod_small(mm, Wo, inv_wo, t1, ow);
    divmod_small(t1, Ho, inv_ho, nn, oh);
    const int h0 = oh * (int)a.sh - (int)a.ph, w0 = ow * (int)a.sw - (int)a.pw;
    a_offb[u] = (((nn * H + h0) * W + w0) * Cin + cgA * 8) * 2;
    orow[u] = ~taps_inside(h0, H, a.kh32, dh, a.inv_dh);
    ocol[u] = ~taps_inside(w0, W, kw, dw, a.inv_dw);
  }
  int b_offb[BV];
#pragma unroll
  for (int u = 0; u < BV; ++u) {
    const int jn = n0 + 8 * (u * NW + wave) + lrow;
    b_offb[u] = ((jn < N ? jn : 0) * (int)a.K + cgB * 8) * 2;
  }

  // ---- the walk: the dense one is written while the route's counts are in
  // flight; a skipping tile overwrites it with its list.  Skipping: by the
  // tile's own samples (split execution), by the device route, or because the
  // host chose the skip path (a bitmap and neither of them).
  int count = c_end - c_begin;
  bool use_list = a.mask != nullptr;
  if (!use_list || a.route.counts || a.route.sample_zeros)   // (a dense walk is possible)
    for (int i = tid; i < count; i += NT) list[i] = walk_entry<kBK2, 2, PART>(a, c_begin + i);
  if (a.route.sample_zeros) {
    use_list = split_route_skips(a, u0, unit);
    if (!use_list && a.executed && first_col && tid == 0 && count)
      atomicAdd(a.executed, (unsigned long long)count);  // a dense tile runs every chunk
  } else {
    if (a.route.counts) use_list = route_counts_skip(rq, a.route);
    if (a.route.path_out && first_tile && tid == 0)
      *a.route.path_out = (a.route.counts && use_list ? 1u : 0u) | ((uint32_t)a.route.bw_bit << 1);
  }
  if (use_list) {
    gather_nonzero_bits<NT>(a, u0, unit, nzvec);
    if (wave == 0) {
      int total = 0;
      for (int base = c_begin; base < c_end; base += 64) {
        const int j = base + lane;
        const bool nz = j < c_end && chunk_nonzero<kBK2, PART>(a, nzvec, min(j, c_end - 1));
        const uint64_t bal = __ballot(nz);
        const int before = __popcll(bal & ((1ull << lane) - 1ull));
        if (nz) list[total + before] = walk_entry<kBK2, 2, PART>(a, j);
        total += __popcll(bal);
      }
      if (lane == 0) {
        list_len = total;
        if (a.executed && first_col && total)
          atomicAdd(a.executed, (unsigned long long)total);
      }
    }
    __syncthreads();
    count = list_len;
  }

  // ---- the epilogue's bias and residual vectors: a lane holds channels 32 p +
  // 8 g + [0, 8) of each block pair p, of pixel rl of its WTM pixel blocks.
  // The 64 x 64 tile requests them behind the first chunks (its latency passes
  // under the K loop), the others behind the K loop, before the first store (a
  // load issued behind stores waits for them): 16 more registers through the K
  // loop halve the resident waves of the 128 x 64 tile (30000 x 768 x 264 46 us
  // and 74).
  constexpr bool kEarly = WTM == 1 && NW == 4;
  const int g = lane >> 4, rl = lane & 15;
  const bool vec_n = N % 8 == 0;
  const int mw = m0 + wm * WTM * 16 + rl, nw = n0 + wn * WTN * 16 + 8 * g;
  const raw *bias = reinterpret_cast<const raw *>(a.bias);
  const raw *res = reinterpret_cast<const raw *>(a.residual);
  raw *y = reinterpret_cast<raw *>(a.y);
  uint4 bias_q[NG][2], res_q[WTM][NG][2];
  // Rows past M and channels past C_out read the last ones, unused: with a
  // branch around each load, zeros on its other side, the compiler waited for
  // each before the next (bf16 with residual, M x N x K in us: 3136 x 256 x 256
  // 6.20, 5.82 so; 2352 x 2048 x 512 16.2, 15.1; 86436 x 1024 x 128 150, 125).
  auto request_epilogue = [&]() __attribute__((always_inline)) {
    if (bias && vec_n) {
#pragma unroll
      for (int q = 0; q < NG; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          bias_q[q][h] = *reinterpret_cast<const uint4 *>(bias + min(nw + 64 * q + 32 * h, N - 8));
    }
    if (res && vec_n) {
#pragma unroll
      for (int tm = 0; tm < WTM; ++tm)
#pragma unroll
        for (int q = 0; q < NG; ++q)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            res_q[tm][q][h] = *reinterpret_cast<const uint4 *>(
                res + (int64_t)min(mw + 16 * tm, M - 1) * N + min(nw + 64 * q + 32 * h, N - 8));
    }
  };

  // ---- the K loop ----------------------------------------------------------
  const uint32_t ring =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem + wave * 1024;
  // PART: bit 31 where this lane's 8 channels of a tap's last chunk lie past
  // C_in (zero on both sides).  (With the chunk's place in its tap found by an
  // integer remainder at every load 1700 x 320 x 440 took 8.1 us, 7.8 so.)
  const int tail = PART ? (Cin - (a.cpt32 - 1) * kBK2) * 2 : ROW;
  const uint32_t pastA = cgA * 16 < tail ? 0u : 0x80000000u;
  const uint32_t pastB = cgB * 16 < tail ? 0u : 0x80000000u;
  // load u of one chunk's L (A rows, then B rows) into the stage at LDS
  // address dst; an offset with bit 31 set is out of range
  auto load_part = [&](const WalkStep &e, uint32_t dst, int u) __attribute__((always_inline)) {
    if (u < AV) {
      const uint32_t out = orow[u] << e.rsh | ocol[u] << e.ssh | (pastA & e.last);
      const uint32_t off = (uint32_t)(a_offb[u] + e.xofs) | (out & 0x80000000u);
      load_to_lds(xr, dst + u * (NW * 1024), (int)off, 0);
    } else {
      load_to_lds(wr, dst + BM * ROW + (u - AV) * (NW * 1024),
                  b_offb[u - AV] | (int)(pastB & e.last), e.kofs);
    }
  };

  f32x4 acc[WTM][WTN];
#pragma unroll
  for (int i = 0; i < WTM; ++i)
#pragma unroll
    for (int j = 0; j < WTN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int fB = (((rl >> 2) & 1) << 2) | (rl & 3);
  int offA[2], offB[2];   // this lane's operand offsets of the two k-steps
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    offA[ks] = (wm * WTM * 16 + rl) * ROW + 16 * ((4 * ks + g) ^ (rl & 7));
    offB[ks] = (BM + wn * WTN * 16 + 8 * (rl >> 2) + (rl & 3)) * ROW + 16 * ((4 * ks + g) ^ fB);
  }
  struct Operands {
    u32x4 a[2][WTM], b[2][WTN];   // of a chunk's two k-steps
  };
  // read q of an operand set's R (k-step 0 first, channel rows before pixels)
  constexpr int R = 2 * (WTM + WTN), MF = 2 * WTM * WTN, RSPAN = MF * 3 / 4;
  auto read_part = [&](Operands &o, int slot, int q) __attribute__((always_inline)) {
    const int ks = q / (WTM + WTN), v = q % (WTM + WTN);
    const char *st = smem + slot * STAGE;
    if (v < WTN)
      o.b[ks][v] = *reinterpret_cast<const u32x4 *>(st + offB[ks] +
                                                    (32 * (v >> 1) + 4 * (v & 1)) * ROW);
    else
      o.a[ks][v - WTN] = *reinterpret_cast<const u32x4 *>(st + offA[ks] + (v - WTN) * 16 * ROW);
  };
  auto multiply = [&](const Operands &o, int q) __attribute__((always_inline)) {
    const int ks = q / (WTM * WTN), tm = q / WTN % WTM, b = q % WTN;
    if constexpr (DT == SPAROA_BF16)
      acc[tm][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, o.b[ks][b]), __builtin_bit_cast(bf16x8, o.a[ks][tm]),
          acc[tm][b], 0, 0, 0);
    else
      acc[tm][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
          __builtin_bit_cast(f16x8, o.b[ks][b]), __builtin_bit_cast(f16x8, o.a[ks][tm]),
          acc[tm][b], 0, 0, 0);
  };
  const WalkGeom geom = walk_geom<2>(a);
  const int n = __builtin_amdgcn_readfirstlane(count);
  if (kEarly && n == 0) request_epilogue();
  __syncthreads();   // the walk is written
  // One step per chunk.  On entry the step's operands are in registers (or
  // on their way from LDS).  After its barrier the next chunk's stage is
  // complete and every wave has read this chunk's stage, which the loads of
  // chunk i + S then refill between this chunk's MFMAs, while the next
  // chunk's operands are read: a wave's LDS reads have a whole chunk of
  // MFMAs to land.  The steady steps (STEADY: a next chunk and a refill
  // exist) are written out for a whole turn of the ring and of the operand
  // pair, with no branch and constant stages: at one or two waves per SIMD a
  // step's scalar instructions are time.
  uint32_t next;   // walk entry of the step's refill
  auto step = [&](auto steady, Operands &cur, Operands &nxt, int slot, int i)
                  __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady)::value;
    const bool more = STEADY || i + 1 < n, refill = STEADY || i + S < n;
    const uint32_t dst = ring + slot * STAGE;
    const WalkStep e = walk_step<PART>(geom, next);
    if (more) {
      if constexpr (STEADY) wait_chunks<S - 2, L>(S - 2);
      else wait_chunks<S - 2, L>(min(S - 2, n - 2 - i));
      __builtin_amdgcn_s_waitcnt(kLgkmcnt0);   // this wave has read its stage
      asm volatile("s_barrier" ::: "memory");
      next = list[STEADY ? i + 1 + S : min(i + 1 + S, n - 1)];
    }
    const int nslot = slot == S - 1 ? 0 : slot + 1;
#pragma unroll
    for (int m = 0; m < MF; ++m) {
      __builtin_amdgcn_sched_barrier(0);
      multiply(cur, m);
      if (more) {
#pragma unroll
        for (int q = m * R / RSPAN; q < (m + 1) * R / RSPAN && q < R; ++q) read_part(nxt, nslot, q);
      }
      if (refill) {
#pragma unroll
        for (int u = m * L / MF; u < (m + 1) * L / MF; ++u) load_part(e, dst, u);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  if (n > 0) {
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (s < n) {
        const WalkStep e = walk_step<PART>(geom, list[s]);
#pragma unroll
        for (int u = 0; u < L; ++u) load_part(e, ring + s * STAGE, u);
      }
    if (kEarly && a.split == 1) request_epilogue();
    // (where they are requested the vectors are newer than the first chunks,
    // so the first waits take more of the loads than they need)
    wait_chunks<S - 1, L>(min(S - 1, n - 1));
    asm volatile("s_barrier" ::: "memory");
    Operands p, q;
#pragma unroll
    for (int r = 0; r < R; ++r) read_part(p, 0, r);
    next = list[min(S, n - 1)];
    constexpr int U = S % 2 ? 2 * S : S;   // a turn of the ring and of (p, q)
    int i = 0;
    // (the last step of a turn prefetches the walk entry of chunk i + U + S)
    for (; i + U + S < n; i += U) {
#pragma unroll
      for (int d = 0; d < U; ++d)
        step(std::true_type{}, d % 2 ? q : p, d % 2 ? p : q, d % S, i + d);
    }
    for (; i < n; i += U) {
#pragma unroll
      for (int d = 0; d < U; ++d)
        if (i + d < n) step(std::false_type{}, d % 2 ? q : p, d % 2 ? p : q, d % S, i + d);
    }
  }

  // ---- epilogue, from registers: 16-byte vectors of bias, residual and output
  // (four lanes of a pixel write 64 consecutive bytes)
  uint32_t om_zeros = 0, om_nz = 0;
  // Output rows that start anywhere (N % 8 != 0): a wave's blocks pass through
  // LDS in the ring's place, 16 pixels x 64 channels at a time, so that its
  // lanes store 64 consecutive channels element by element.  (Stored by the
  // lanes that hold them, a store touched 16 rows: bf16 8619 x 1308 x 64 50 us,
  // 3000 x 1308 x 1024 48; this way 27.5 and 32.)
  if (!vec_n) {
    constexpr int TS = 64 + 4;   // row stride: four rows of blocks hit distinct banks
    static_assert(NW * 16 * TS * 4 <= S * STAGE, "the ring's place");
    __syncthreads();   // every wave has read its last stage
    float *const mine = reinterpret_cast<float *>(smem) + wave * (16 * TS);
    float *const part = a.split > 1 ? a.partial + (int64_t)zsplit * M * N : nullptr;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int col = n0 + wn * WTN * 16 + 64 * q + lane;
      const float bf = !part && bias && col < N ? E::to_f32(bias[col]) : 0.f;
#pragma unroll
      for (int tm = 0; tm < WTM; ++tm) {
        const int row0 = m0 + wm * WTM * 16 + 16 * tm;
        raw rv[16];
        if (res && !part) {   // before the stores: a load issued behind them waits
#pragma unroll
          for (int r = 0; r < 16; ++r)
            rv[r] = row0 + r < M && col < N ? res[(int64_t)(row0 + r) * N + col] : (raw)0;
        }
#pragma unroll
        for (int b = 0; b < 4; ++b)
          *reinterpret_cast<f32x4 *>(mine + rl * TS + 32 * (b >> 1) + 8 * g + 4 * (b & 1)) =
              acc[tm][4 * q + b];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float v = mine[r * TS + lane];
          if (row0 + r >= M || col >= N) continue;
          const int64_t o = (int64_t)(row0 + r) * N + col;
          if (part) {
            part[o] = v;
          } else {
            if (bias) v += bf;
            if (res) v += E::to_f32(rv[r]);
            y[o] = E::from_f32(apply_act(v, a.act));
          }
        }
      }
    }
    return;   // (N % 64 == 0 whenever the output is measured)
  }
  if (a.split > 1) {
#pragma unroll
    for (int tm = 0; tm < WTM; ++tm) {
      const int row = mw + 16 * tm;
      if (row >= M) continue;
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        const int col = nw + 64 * q;
        float *dst = a.partial + ((int64_t)zsplit * M + row) * N + col;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int c = 32 * (b >> 1) + 4 * (b & 1);
          if (col + c < N) *reinterpret_cast<f32x4 *>(dst + c) = acc[tm][4 * q + b];
        }
      }
    }
    return;
  }
  if (!kEarly) request_epilogue();
  // output measurement (N % 64 == 0): the eight (1, 8) blocks of a pixel's
  // 64-channel group are one bitmap byte, met by two ballots
  const int mbytes = om && a.om_mask ? (int)(4 * (((int64_t)M * (N / 8) + 31) / 32)) : 0;
#pragma unroll
  for (int tm = 0; tm < WTM; ++tm) {
    const int row = mw + 16 * tm;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      uint32_t nzb[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = nw + 64 * q + 32 * h;
        const bool valid = row < M && col < N;
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = acc[tm][4 * q + 2 * h + (e >> 2)][e & 3];
        raw t[8];
        if (bias) {
          __builtin_memcpy(t, &bias_q[q][h], 16);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] += E::to_f32(t[e]);
        }
        if (res) {
          __builtin_memcpy(t, &res_q[tm][q][h], 16);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] += E::to_f32(t[e]);
        }
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          w[e] = E::pack2(apply_act(o[2 * e], a.act), apply_act(o[2 * e + 1], a.act));
        uint4 q4;
        __builtin_memcpy(&q4, w, 16);
        if (valid) *reinterpret_cast<uint4 *>(y + (int64_t)row * N + col) = q4;
        nzb[h] = 0;
        if (om) {
          const uint32_t nz = nonzeros16<4>(w);
          om_zeros += valid ? 8u - nz : 0u;
          nzb[h] = valid && nz ? 1u : 0u;
          om_nz += nzb[h];
        }
      }
      if (mbytes) {
        const uint64_t b0 = __ballot(nzb[0] != 0u), b1 = __ballot(nzb[1] != 0u);
        // rows past M still clear their bytes when they lie inside the
        // bitmap's last word (bits past the last block are 0)
        const int byte = row * (N / 64) + (nw - 8 * g) / 64 + q;
        if (g == 0 && nw + 64 * q < N && byte < mbytes) {
          uint32_t v = 0;
#pragma unroll
          for (int p = 0; p < 4; ++p)
            v |= ((uint32_t)(b0 >> (rl + 16 * p)) & 1u) << p |
                 ((uint32_t)(b1 >> (rl + 16 * p)) & 1u) << (4 + p);
          reinterpret_cast<uint8_t *>(a.om_mask)[byte] = (uint8_t)v;
        }
      }
    }
  }
  if (om) om_commit(om_zeros, om_nz, a.om_counts, a.om_words, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// Implicit GEMM of few tiles: small tiles whose waves split K.  Where a layer
// has too few 64 x 64 tiles to fill the chip, its time is the chain of chunks
// of one tile and, with K split over work-groups, a reduction launch.  Here a
// tile is 16 TM x 16 TN outputs, small enough to give every CU one, and wave w
// of a work-group takes chunks w, w + NW, ... of it: the wave's own ring of S
// chunks in LDS (the loads of igemm_kernel), so the K loop has no barrier;
// the NW partial tiles meet in LDS at the end, added in wave order.  A chunk
// is 128 bytes of channels of one tap: 64 at 16 bits, 32 in fp32.
// What bounds it is latency: launch, set-up, one memory round trip, a few
// chunks, the reduction and the commit.
// Skipping is by the rows the tiling query reports: a wave drops those of its
// chunks whose gathered input is zero over the unit the tile lies in,
// so the output equals the dense form's bit for bit.

template <int DT, int TM, int TN, int NW, int S, bool PART>
__global__ __launch_bounds__(64 * NW, 2) void igemm_lk_kernel(GemmArgs a) {
  using E = Elem<DT>;
  using raw = typename E::raw;
  constexpr int ESZ = E::size;
  constexpr int NT = 64 * NW;
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr int C = 128 / ESZ;         // channels of a chunk
  constexpr int ROW = 128;
  constexpr int L = 2 * (TM + TN);     // loads of a chunk: 8 rows each
  constexpr int STAGE = (BM + BN) * ROW;
  constexpr int CS = BN + 4;           // fp32 row stride of a partial tile
  constexpr int PART_BYTES = BM * CS * 4;
  constexpr int ITEMS = BM * BN / 8;   // epilogue items: 8 channels of a pixel
  constexpr int EIT = (ITEMS + NT - 1) / NT;
  constexpr int RING = NW * S * STAGE, RED = NW * PART_BYTES;
  static_assert(L * (S - 1) < 64, "vmcnt range");

  __shared__ __attribute__((aligned(1024))) char smem[RING > RED ? RING : RED];
  __shared__ uint32_t list[NW][(kMaxChunks2 + NW - 1) / NW];
  __shared__ uint32_t nzvec[kMaxVecWords + 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (the set-up's kernel arguments in one round trip, as in igemm_kernel)
  asm volatile("" ::"s"(a.M), "s"(a.N), "s"(a.K), "s"(a.H), "s"(a.W), "s"(a.Cin), "s"(a.Ho),
               "s"(a.Wo), "s"(a.Kw), "s"(a.sh), "s"(a.sw), "s"(a.ph), "s"(a.pw), "s"(gridDim.x),
               "s"(a.route.counts), "s"(a.route.path_out), "s"(a.om_counts), "s"(a.nchunks));
  const bool om = a.om_counts != nullptr;
  const RouteCountsReq rq = route_counts_request(a.route);
  // (two waves, more tiles than CUs: an XCD's share is not one part of the
  // rows, which with a padded batch would give one XCD all of the work; fp32
  // 100352 x 64, 1024 channels, a quarter of the samples in use 164 us with a
  // contiguous share, 54 so; all in use 170 either way)
  const TileId tl = tile_of<NW == 2 && TM == 4>(a);
  const int m0 = a.row0 + tl.mt * BM, n0 = tl.nt * BN;
  const int M = (int)a.M, N = (int)a.N, n = (int)a.nchunks;
  const int H = (int)a.H, W = (int)a.W, Ho = (int)a.Ho, Wo = (int)a.Wo, Cin = (int)a.Cin;
  const int kw = (int)a.Kw;

  // ---- this lane's rows of the loads: load q of a chunk fills rows 8 q + l /
  // 8, slot l % 8 holding vector (l % 8) ^ (row % 8)
  const int lrow = lane >> 3, cg = (lane & 7) ^ lrow;
  const u32x4 xr = buffer_words(a.x, a.x_bytes), wr = buffer_words(a.w, a.w_bytes);
  int a_offb[2 * TM], b_offb[2 * TN];
  uint32_t orow[2 * TM], ocol[2 * TM];  // bit r / s: kernel row r / column s outside the image
#pragma unroll
  for (int u = 0; u < 2 * TM; ++u) {
    const int m = m0 + 8 * u + lrow;
    int t1, ow, nn, oh;
    divmod_small(m < M ? m : 0, Wo, a.inv_wo, t1, ow);
    divmod_small(t1, Ho, a.inv_ho, nn, oh);
    const int h0 = oh * (int)a.sh - (int)a.ph, w0 = ow * (int)a.sw - (int)a.pw;
    a_offb[u] = ((nn * H + h0) * W + w0) * Cin * ESZ + 16 * cg;
    orow[u] = ~taps_inside(h0, H, a.kh32, (int)a.dh, a.inv_dh);
    ocol[u] = ~taps_inside(w0, W, kw, (int)a.dw, a.inv_dw);
  }
#pragma unroll
  for (int u = 0; u < 2 * TN; ++u) {
    const int jn = n0 + 8 * u + lrow;
    b_offb[u] = (jn < N ? jn : 0) * (int)a.K * ESZ + 16 * cg;
  }

  // ---- this wave's walk (its own list: no barrier on the dense path)
  uint32_t *const mine = list[wave];
  const WalkGeom geom = walk_geom<ESZ>(a);
  int nloc = n > wave ? (n - wave + NW - 1) / NW : 0;
  bool use_list = a.mask != nullptr;
  if (!use_list || a.route.counts || a.route.sample_zeros)   // (a dense walk is possible)
    for (int i = lane; i < nloc; i += 64) mine[i] = walk_entry<C, ESZ, PART>(a, wave + NW * i);
  const int unit = a.skip_rows, u0 = m0 & ~(unit - 1);
  const bool counts_here = tl.nt == 0 && u0 == m0;   // one tile per unit counts executed blocks
  if (a.route.sample_zeros) {
    use_list = split_route_skips(a, u0, unit);
    if (!use_list && a.executed && counts_here && tid == 0)
      atomicAdd(a.executed, (unsigned long long)n);  // a dense unit runs every chunk
  } else {
    if (a.route.counts) use_list = route_counts_skip(rq, a.route);
    if (a.route.path_out && tl.tile == 0 && tid == 0)
      *a.route.path_out = (a.route.counts && use_list ? 1u : 0u) | ((uint32_t)a.route.bw_bit << 1);
  }
  if (use_list) {
    gather_nonzero_bits<NT>(a, u0, unit, nzvec);
    int total = 0;
    for (int base = 0; base < nloc; base += 64) {
      const int i = base + lane, j = wave + NW * min(i, nloc - 1);
      const bool nz = i < nloc && chunk_nonzero<C, PART>(a, nzvec, j);
      const uint64_t bal = __ballot(nz);
      const int before = __popcll(bal & ((1ull << lane) - 1ull));
      if (nz) mine[total + before] = walk_entry<C, ESZ, PART>(a, j);
      total += __popcll(bal);
    }
    nloc = total;
    if (lane == 0 && a.executed && counts_here && total)
      atomicAdd(a.executed, (unsigned long long)total);
  }
  nloc = __builtin_amdgcn_readfirstlane(nloc);

  // ---- the K loop
  const uint32_t ring =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem + wave * (S * STAGE);
  const char *const stages = smem + wave * (S * STAGE);
  // PART: bit 31 where this lane's channels of a tap's last chunk lie past C_in
  const int tail = PART ? (Cin - (a.cpt32 - 1) * C) * ESZ : ROW;
  const uint32_t past = cg * 16 < tail ? 0u : 0x80000000u;
  auto load_chunk = [&](int i, int slot) __attribute__((always_inline)) {
    const WalkStep e = walk_step<PART>(geom, mine[i]);
    const uint32_t dst = ring + slot * STAGE;
#pragma unroll
    for (int u = 0; u < 2 * TM; ++u) {
      const uint32_t out = orow[u] << e.rsh | ocol[u] << e.ssh | (past & e.last);
      const uint32_t off = (uint32_t)(a_offb[u] + e.xofs) | (out & 0x80000000u);
      load_to_lds(xr, dst + u * 1024, (int)off, 0);
    }
#pragma unroll
    for (int u = 0; u < 2 * TN; ++u)
      load_to_lds(wr, dst + BM * ROW + u * 1024, b_offb[u] | (int)(past & e.last), e.kofs);
  };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int g = lane >> 4, rl = lane & 15;
  int opoff[2];   // operand offset of the chunk's two halves: row rl, vector 4 h + g
#pragma unroll
  for (int h = 0; h < 2; ++h) opoff[h] = rl * ROW + 16 * ((4 * h + g) ^ (rl & 7));
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s < nloc) load_chunk(s, s);

  // (the epilogue's bias and residual vectors, behind the first chunks)
  const bool vec_n = N % 8 == 0;
  const raw *bias = reinterpret_cast<const raw *>(a.bias);
  const raw *res = reinterpret_cast<const raw *>(a.residual);
  raw *y = reinterpret_cast<raw *>(a.y);
  constexpr int QV = ESZ / 2;   // 16-byte vectors of 8 elements
  uint4 bias_q[EIT][QV], res_q[EIT][QV];
  // (rows past M and channels past C_out read the last ones, unused)
#pragma unroll
  for (int it = 0; it < EIT; ++it) {
    const int q = min(tid + it * NT, ITEMS - 1);
    const int row = min(m0 + q / (BN / 8), M - 1), col = min(n0 + q % (BN / 8) * 8, N - 8);
    if (bias && vec_n) {
#pragma unroll
      for (int v = 0; v < QV; ++v)
        bias_q[it][v] = *reinterpret_cast<const uint4 *>(bias + col + v * (16 / ESZ));
    }
    if (res && vec_n) {
#pragma unroll
      for (int v = 0; v < QV; ++v)
        res_q[it][v] =
            *reinterpret_cast<const uint4 *>(res + (int64_t)row * N + col + v * (16 / ESZ));
    }
  }

  int slot = 0;
  for (int i = 0; i < nloc; ++i) {
    // chunk i has landed when at most the newer chunks' loads are outstanding
    // (and, waited for too, the epilogue vectors issued behind the first S)
    wait_chunks<S - 1, L>(min(S - 1, nloc - 1 - i));
    asm volatile("" ::: "memory");
    const char *st = stages + slot * STAGE;
    u32x4 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int b = 0; b < TM; ++b)
        fa[h][b] = *reinterpret_cast<const u32x4 *>(st + opoff[h] + b * 16 * ROW);
#pragma unroll
      for (int b = 0; b < TN; ++b)
        fb[h][b] = *reinterpret_cast<const u32x4 *>(st + opoff[h] + (BM + b * 16) * ROW);
    }
    if (i + S < nloc) {
      __builtin_amdgcn_s_waitcnt(kLgkmcnt0);   // the stage is read: refill it
      load_chunk(i + S, slot);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
          if constexpr (DT == SPAROA_BF16)
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, fb[h][tn]), __builtin_bit_cast(bf16x8, fa[h][tm]),
                acc[tm][tn], 0, 0, 0);
          else if constexpr (DT == SPAROA_F16)
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                __builtin_bit_cast(f16x8, fb[h][tn]), __builtin_bit_cast(f16x8, fa[h][tm]),
                acc[tm][tn], 0, 0, 0);
          else {
            const f32x4 va = __builtin_bit_cast(f32x4, fa[h][tm]);
            const f32x4 vb = __builtin_bit_cast(f32x4, fb[h][tn]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[tm][tn] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(vb[e], va[e], acc[tm][tn], 0, 0, 0);
          }
        }
    slot = slot == S - 1 ? 0 : slot + 1;
  }

  // ---- the partial tiles meet in LDS, in the rings' place (a lane holds 4
  // consecutive channels 4 g + [0, 4) of pixel rl of each block)
  __syncthreads();
  float *const red = reinterpret_cast<float *>(smem);
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
      *reinterpret_cast<f32x4 *>(red + wave * (BM * CS) + (16 * tm + rl) * CS + 16 * tn + 4 * g) =
          acc[tm][tn];
  __syncthreads();
  // Output rows that start anywhere: consecutive lanes take consecutive
  // channels element by element, each its own channel throughout (fp32 4200 x
  // 324 x 64 16.2 us with 8 channels a lane, 14.2 so).
  if (!vec_n) {
    static_assert(NT % BN == 0, "a lane's channel");
    constexpr int RS = NT / BN, PER = (BM + RS - 1) / RS, U = PER < 8 ? PER : 8;
    const int c = tid % BN, col = n0 + c;
    const float bf = bias && col < N ? E::to_f32(bias[col]) : 0.f;
    for (int i0 = 0; i0 < PER; i0 += U) {
      float v[U], rf[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {   // the loads before the stores
        const int r = tid / BN + (i0 + u) * RS;
        const bool valid = r < BM && m0 + r < M && col < N;
        rf[u] = res && valid ? E::to_f32(res[(int64_t)(m0 + r) * N + col]) : 0.f;
        v[u] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v[u] += red[w * (BM * CS) + min(r, BM - 1) * CS + c];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = tid / BN + (i0 + u) * RS;
        if (bias) v[u] += bf;
        if (res) v[u] += rf[u];
        if (r < BM && m0 + r < M && col < N)
          y[(int64_t)(m0 + r) * N + col] = E::from_f32(apply_act(v[u], a.act));
      }
    }
    return;   // (N % 8 == 0 whenever the output is measured)
  }
  uint32_t om_zeros = 0, om_nz = 0;
#pragma unroll
  for (int it = 0; it < EIT; ++it) {
    const int q = tid + it * NT;
    if (q - lane >= ITEMS) break;   // whole waves
    const int r = q / (BN / 8), c = q % (BN / 8) * 8;
    const int row = m0 + r, col = n0 + c;
    const bool valid = q < ITEMS && row < M && col < N;
    f32x4 lo = f32x4{0.f, 0.f, 0.f, 0.f}, hi = lo;
    if (valid) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {   // (waves without a chunk hold zeros)
        lo += *reinterpret_cast<const f32x4 *>(red + w * (BM * CS) + r * CS + c);
        hi += *reinterpret_cast<const f32x4 *>(red + w * (BM * CS) + r * CS + c + 4);
      }
    }
    float o[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    raw t[8];
    if (bias) {
      __builtin_memcpy(t, bias_q[it], 8 * ESZ);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] += E::to_f32(t[e]);
    }
    if (res) {
      __builtin_memcpy(t, res_q[it], 8 * ESZ);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] += E::to_f32(t[e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = apply_act(o[e], a.act);
    if constexpr (ESZ == 4) {
      if (valid) {
        float *d = reinterpret_cast<float *>(a.y) + (int64_t)row * N + col;
        *reinterpret_cast<float4 *>(d) = make_float4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<float4 *>(d + 4) = make_float4(o[4], o[5], o[6], o[7]);
      }
    } else {
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = E::pack2(o[2 * e], o[2 * e + 1]);
      uint4 q4;
      __builtin_memcpy(&q4, w, 16);
      if (valid) *reinterpret_cast<uint4 *>(y + (int64_t)row * N + col) = q4;
      if (om) {
        const uint32_t nz = nonzeros16<4>(w);
        om_zeros += valid ? 8u - nz : 0u;
        const bool nzb = valid && nz != 0u;
        om_nz += nzb ? 1u : 0u;
        if (a.om_mask) {
          // A pixel's BN / 8 bits of the bitmap: a byte of it, or bits of one or
          // two words, set and cleared by atomics (each bit has one owner, so
          // neither the order nor what the words held matters).
          constexpr int LB = BN / 8;   // lanes (and bits) of a pixel's row
          const uint64_t bal = __ballot(nzb), have = __ballot(valid);
          const uint32_t bits = (uint32_t)(bal >> (lane & ~(LB - 1))) & ((1u << LB) - 1u);
          const uint32_t own = (uint32_t)(have >> (lane & ~(LB - 1))) & ((1u << LB) - 1u);
          if (LB == 8 && N % 64 == 0) {   // a byte of the bitmap: stored
            if ((lane & (LB - 1)) == 0 && own)
              reinterpret_cast<uint8_t *>(a.om_mask)[(int64_t)row * (N / 64) + col / 64] =
                  (uint8_t)bits;
          } else if ((lane & (LB - 1)) == 0 && own) {
            const int64_t bit = (int64_t)row * (N / 8) + col / 8;
            const int sh = (int)(bit & 31);
            uint32_t *wd = a.om_mask + (bit >> 5);
            const uint64_t set = (uint64_t)bits << sh, clr = (uint64_t)(own & ~bits) << sh;
            if ((uint32_t)set) atomicOr(wd, (uint32_t)set);
            if ((uint32_t)clr) atomicAnd(wd, ~(uint32_t)clr);
            if ((uint32_t)(set >> 32)) atomicOr(wd + 1, (uint32_t)(set >> 32));
            if ((uint32_t)(clr >> 32)) atomicAnd(wd + 1, ~(uint32_t)(clr >> 32));
          }
        }
      }
    }
  }
  if (om) {
    if (a.om_mask && tl.tile == 0 && tid == 0) {   // bits past the last block are 0
      const int64_t nb = (int64_t)M * (N / 8);
      if (BN == 64 && N % 64 == 0) {
        for (int64_t b = nb / 8; b & 3; ++b) reinterpret_cast<uint8_t *>(a.om_mask)[b] = 0;
      } else if (nb & 31) {
        atomicAnd(a.om_mask + (nb >> 5), (1u << (nb & 31)) - 1u);
      }
    }
    om_commit(om_zeros, om_nz, a.om_counts, a.om_words, blockIdx.x, gridDim.x);
  }
}

// ---------------------------------------------------------------------------
// Direct MFMA conv for inputs with at most 4 channels (image stems: ResNet's
// 7x7/2 and MobileNetV2's 3x3/2 over RGB), where the implicit GEMM's 8- or
// 64-channel K chunks would be mostly padding and its gathers scalar.  A
// work-group computes `rw` output rows of one image (all Wo pixels, all
// C_out <= 64 channels).  It stages the input rows they need, zero-padded on
// both sides, in LDS as [row][PWP][4] (channels padded to 4 with zeros), so K
// is laid out as (kernel row r, tap pair j, tap parity, channel): an
// 8-element block of K is two taps x 4 channels, contiguous and 8-byte
// aligned in the patch.  K = kh * ceil(kw/2) blocks, four per
// v_mfma_f32_16x16x32 k-step; a tap past kw (odd kw) and blocks past the last
// kernel row read zero.  The weights, laid out the same way, pass through LDS
// once into registers, where a wave keeps all C_out channels: a 16-pixel
// block's patch operands are read once for all of them.  Each wave walks
// whole 16-pixel blocks of a row; the MFMA's rows are channels, so a lane
// ends with 4 NB consecutive channels of its pixel and finishes them from
// registers.  Bound by its output stores (51 MB on ResNet-50's at N = 32);
// one work-group per row with a wave per 16 channels, the patch re-read for
// each and the tile staged in LDS took 75 us there, this form 29 us (at N = 8
// 24 -> 12.5 us, at N = 1 13 -> 6.7 us; more waves per CU spilled: 37 us).
// Skip form: MFMAs whose patch operand is zero in all 64 lanes are not issued
// (they would add exact zeros), so the skip output equals the dense output
// bit for bit; executed_blocks counts the (row block, k-step) pairs issued.
// Output measurement: a lane's 8 channels are one (1, 8) block of the output,
// so the epilogue also counts zeros and nonzero blocks when asked
// (counts-only measurement of y, one ticketed commit per work-group).
constexpr int kScMaxKSteps = 8;
constexpr int kScMaxRB = 8;            // Wo <= 128
constexpr int kScPatchBytes = 48 * 1024;  // bound of the eligible shapes (small_c_eligible)
constexpr int kScLdsBytes = 64 * 1024;    // LDS of a work-group

struct SmallCArgs {
  const char *x, *w, *bias, *residual;
  char *y;
  unsigned long long *executed;
  int H, W, C, Ho, Wo, Cout, kh, kw, sh, sw, ph, pw;
  int PWP, bpr, act;
  int pair;                // an input row is whole dwords (W C even)
  int rw, groups;          // output rows per work-group (1, 2 or 4), work-groups per image
  int prows;               // patch rows: (rw - 1) sh + kh
  int patch_off;           // LDS byte offset of the patch (0: it replaces the weights)
  float inv_bpr, inv_pwp;  // rounded once
  int mode;  // 0 dense, 1 skip, 2 device route
  DeviceRoute route;
  // counts-only output measurement at block (1 pixel, 8 channels): non-null
  // om_counts holds {0, numel, nb, nb} on entry; om_words: count-commit words
  sparoa_counts *om_counts;
  unsigned long long *om_words;
};

template <int DT, int KS, int NB>
__global__ __launch_bounds__(256, 2) void conv_small_c_kernel(SmallCArgs a) {
  using E = Elem<DT>;
  using raw = typename E::raw;
  constexpr int CO = 16 * NB;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ unsigned long long exec_part[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, rl = lane & 15;
  SPAROA_ARGS_UP_FRONT("s"(a.x), "s"(a.w), "s"(a.H), "s"(a.W), "s"(a.C), "s"(a.Ho), "s"(a.kh),
                       "s"(a.kw), "s"(a.sh), "s"(a.ph), "s"(a.pw), "s"(a.PWP), "s"(a.rw),
                       "s"(a.groups), "s"(a.prows), "s"(a.patch_off), "s"(a.mode),
                       "s"(a.route.counts));
  const RouteCountsReq rq = route_counts_request(a.route);
  const int img = (int)(blockIdx.x / (unsigned)a.groups);
  const int oh0 = (int)(blockIdx.x % (unsigned)a.groups) * a.rw;
  const int ih0 = oh0 * a.sh - a.ph, rowe = a.W * a.C;

  // ---- weights -> LDS as K blocks [CO][WP] of 16 bytes, one block of
  // padding per channel (conflict-free reads).  Consecutive lanes take
  // consecutive blocks of a channel; a block's two taps are 4 C consecutive
  // bytes, read with one 16-byte load from the dword below them (the last
  // blocks: from the tensor's end, a multiple of 32 bytes) and moved into
  // place.
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      (void *)a.w, (short)0, CO * a.kh * a.kw * a.C * 2, kBufDword3);
  constexpr int WB = 4 * KS, WP = WB + 1;
  constexpr int WIT = (WB * CO + 255) / 256;
  const int tapb = 2 * a.C, wlast = CO * a.kh * a.kw * a.C * 2 - 16;
  const uint64_t cmask = a.C == 4 ? ~0ull : (1ull << (8 * tapb)) - 1ull;
  u32x4 wv[WIT];
  int woff[WIT];   // byte offset of the block, negative past the kernel
  bool whi[WIT];   // the block has a second tap
#pragma unroll
  for (int u = 0; u < WIT; ++u) {
    const int v = tid + 256 * u, co = v / WB, blk = v % WB;
    int r, j;
    divmod_small(blk, a.bpr, a.inv_bpr, r, j);
    const bool in = co < CO && r < a.kh;
    woff[u] = in ? ((co * a.kh + r) * a.kw + 2 * j) * tapb : -1;
    whi[u] = 2 * j + 1 < a.kw;
    wv[u] = __builtin_amdgcn_raw_buffer_load_b128(
        wr, in ? min(woff[u] & ~3, wlast) : (int)0x80000000, 0, 0);
  }
  // ---- patch[row][q][c4] (q = input column + pw): zero outside the image
  // and for channels >= C.  The buffer range starts at the first input row
  // the image has (a work-group's rows stay within 32 bits whatever x holds).
  const int ihb = max(ih0, 0), nin = max(min(ih0 + a.prows, a.H) - ihb, 0);
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(a.x + ((int64_t)img * a.H + ihb) * rowe * 2), (short)0, nin * rowe * 2, kBufDword3);
  char *const patch = smem + a.patch_off;
  const int npx = a.prows * a.PWP, xlast = nin * rowe * 2 - 8;
  // PAIR: rows of whole dwords (W C even), at least one pair of them: a
  // pixel's 2 C <= 8 bytes come with one 8-byte load from the dword below
  // them; else element by element
  auto stage_patch = [&](auto pair) __attribute__((always_inline)) {
    constexpr bool PAIR = decltype(pair)::value;
    constexpr int U = 4;
    for (int p0 = tid; p0 < npx; p0 += 256 * U) {
      uint64_t t[U];
      int off[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int pr, q;
        divmod_small(p0 + 256 * u, a.PWP, a.inv_pwp, pr, q);
        const int ih = ih0 + pr, iw = q - a.pw;
        const bool in = ih >= ihb && ih < a.H && iw >= 0 && iw < a.W && pr < a.prows;
        off[u] = in ? ((ih - ihb) * rowe + iw * a.C) * 2 : -1;
        if constexpr (PAIR) {
          typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
          const u32x2 d = __builtin_amdgcn_raw_buffer_load_b64(
              xr, in ? min(off[u] & ~3, xlast) : (int)0x80000000, 0, 0);
          t[u] = (uint64_t)d.x | (uint64_t)d.y << 32;
        } else {
          t[u] = 0;
#pragma unroll
          for (int c = 0; c < 4; ++c)
            t[u] |= (uint64_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                        xr, in && c < a.C ? off[u] + 2 * c : (int)0x80000000, 0, 0)
                    << (16 * c);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + 256 * u;
        if constexpr (PAIR) t[u] = t[u] >> (8 * max(off[u] - min(off[u] & ~3, xlast), 0)) & cmask;
        if (p < npx) *reinterpret_cast<uint64_t *>(patch + (size_t)p * 8) = off[u] < 0 ? 0 : t[u];
      }
    }
  };
  auto stage = [&]() __attribute__((always_inline)) {
    if (a.pair && xlast >= 0) stage_patch(std::true_type{});
    else stage_patch(std::false_type{});
  };
  if (a.patch_off) stage();
#pragma unroll
  for (int u = 0; u < WIT; ++u) {
    const int v = tid + 256 * u, s = woff[u] - min(woff[u] & ~3, wlast);   // bytes to drop, < 16
    uint64_t lo = (uint64_t)wv[u][0] | (uint64_t)wv[u][1] << 32;
    uint64_t hi = (uint64_t)wv[u][2] | (uint64_t)wv[u][3] << 32;
    const bool far = s >= 8;
    lo = far ? hi : lo;
    hi = far ? 0ull : hi;
    const int sb = 8 * (s & 7);
    lo = lo >> sb | (sb ? hi << (64 - sb) : 0ull);
    hi >>= sb;
    const uint64_t second = a.C == 4 ? hi : lo >> (8 * tapb) | hi << (64 - 8 * tapb);
    const bool in = woff[u] >= 0;
    const uint64_t q[2] = {in ? lo & cmask : 0ull, in && whi[u] ? second & cmask : 0ull};
    uint4 q4;
    __builtin_memcpy(&q4, q, 16);
    if (v < WB * CO) *reinterpret_cast<uint4 *>(smem + (v / WB * WP + v % WB) * 16) = q4;
  }
  __syncthreads();

  // ---- weight operands: MFMA row 4 q + v of block b is channel
  // 4 NB q + 4 b + v; lane group g holds K block 4 t + g.  The patch side
  // keeps each block's offset and the all-ones / zero masks of its taps.
  u32x4 wop[NB][KS];
  int koff[KS];
  uint32_t mlo[KS], mhi[KS];
#pragma unroll
  for (int t = 0; t < KS; ++t) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
      wop[b][t] = *reinterpret_cast<const u32x4 *>(
          smem + ((4 * NB * (rl >> 2) + 4 * b + (rl & 3)) * WP + 4 * t + g) * 16);
    int r, j;
    divmod_small(4 * t + g, a.bpr, a.inv_bpr, r, j);
    const bool lo_ok = r < a.kh, hi_ok = lo_ok && 2 * j + 1 < a.kw;
    mlo[t] = lo_ok ? 0xFFFFFFFFu : 0u;
    mhi[t] = hi_ok ? 0xFFFFFFFFu : 0u;
    koff[t] = (min(r, a.kh - 1) * a.PWP + 2 * j) * 8;
  }
  if (!a.patch_off) {   // the patch takes the weights' place
    __syncthreads();
    stage();
    __syncthreads();
  }
  bool skip = a.mode == 1;
  if (a.mode == 2) {
    skip = route_counts_skip(rq, a.route);
    if (a.route.path_out && blockIdx.x == 0 && tid == 0)
      *a.route.path_out = (skip ? 1u : 0u) | ((uint32_t)a.route.bw_bit << 1);
  }
  constexpr int V = NB >= 2 ? NB / 2 : 1;   // output vectors of a lane: 8 channels (4: NB 1)
  constexpr int CV = NB >= 2 ? 8 : 4;
  const raw *bias = reinterpret_cast<const raw *>(a.bias);
  float bf[4 * NB];
#pragma unroll
  for (int e = 0; e < 4 * NB; ++e) bf[e] = bias ? E::to_f32(bias[4 * NB * g + e]) : 0.f;

  // ---- a wave's row (wave % rw) and share of its 16-pixel blocks
  const int wrow = wave % a.rw, nparts = 4 / a.rw;
  const int RB = (a.Wo + 15) / 16;
  const int oh = oh0 + wrow;
  unsigned long long executed = 0;
  uint32_t om_zeros = 0, om_nz = 0;
  const int64_t row0 = ((int64_t)img * a.Ho + oh) * a.Wo;
  // (one 16-pixel block; GEN: with the skip test and a residual)
  auto block = [&](auto gen, int rb) __attribute__((always_inline)) {
    constexpr bool GEN = decltype(gen)::value;
    const int ow = rb * 16 + rl;
    // (pixels past Wo read a valid one, unused)
    const char *px = patch + (wrow * a.sh * a.PWP + min(ow, a.Wo - 1) * a.sw) * 8;
    u32x4 aops[KS];
#pragma unroll
    for (int t = 0; t < KS; ++t) {   // all reads first
      // two 8-byte reads: a block starts on an 8-byte (not 16-byte) boundary
      const uint2 lo = *reinterpret_cast<const uint2 *>(px + koff[t]);
      const uint2 hi = *reinterpret_cast<const uint2 *>(px + koff[t] + 8);
      aops[t] = u32x4{lo.x & mlo[t], lo.y & mlo[t], hi.x & mhi[t], hi.y & mhi[t]};
    }
    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      const u32x4 aop = aops[t];
      if (GEN && skip && __ballot((aop[0] | aop[1] | aop[2] | aop[3]) != 0u) == 0ull) continue;  // exact
      if (GEN) executed += 1;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if constexpr (DT == SPAROA_BF16)
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wop[b][t]),
                                                           __builtin_bit_cast(bf16x8, aop), acc[b],
                                                           0, 0, 0);
        else
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, wop[b][t]),
                                                          __builtin_bit_cast(f16x8, aop), acc[b],
                                                          0, 0, 0);
      }
    }
    // ---- epilogue: channels 4 NB g + [0, 4 NB) of pixel ow
    const bool valid = ow < a.Wo;
    const int64_t o = (row0 + ow) * CO + 4 * NB * g;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      raw t8[CV];
      float f[CV];
#pragma unroll
      for (int e = 0; e < CV; ++e)
        f[e] = acc[CV / 4 * v + (e >> 2)][e & 3] + bf[CV * v + e];
      if (GEN && a.residual && valid) {
        __builtin_memcpy(t8, reinterpret_cast<const raw *>(a.residual) + o + CV * v, 2 * CV);
#pragma unroll
        for (int e = 0; e < CV; ++e) f[e] += E::to_f32(t8[e]);
      }
      uint32_t w[CV / 2];
#pragma unroll
      for (int e = 0; e < CV / 2; ++e)
        w[e] = E::pack2(apply_act(f[2 * e], a.act), apply_act(f[2 * e + 1], a.act));
      if (valid) __builtin_memcpy(reinterpret_cast<raw *>(a.y) + o + CV * v, w, 2 * CV);
      if (a.om_counts) {
        uint32_t nz = nonzeros16<CV / 2>(w);
        om_zeros += valid ? CV - nz : 0u;
        if constexpr (NB == 1) {   // a block is two lanes' channels: counted by the even group
          const uint32_t other = __shfl_xor(nz, 16, 64);   // (every lane takes part)
          nz = (g & 1) ? 0u : nz + other;
        }
        om_nz += valid && nz ? 1u : 0u;
      }
    }
  };
  const int rb0 = oh < a.Ho ? wave / a.rw : RB;
  if (skip || a.residual) {
    for (int rb = rb0; rb < RB; rb += nparts) block(std::true_type{}, rb);
  } else {
    for (int rb = rb0; rb < RB; rb += nparts) block(std::false_type{}, rb);
  }
  if (a.executed && skip) {
    if (lane == 0) exec_part[wave] = executed;
    __syncthreads();
    if (tid == 0) {
      const unsigned long long tot = exec_part[0] + exec_part[1] + exec_part[2] + exec_part[3];
      if (tot) atomicAdd(a.executed, tot);
    }
  }
  if (a.om_counts) om_commit(om_zeros, om_nz, a.om_counts, a.om_words, blockIdx.x, gridDim.x);
}

template <int DT, int WGM, int WGN, int WTM, int WTN, int S, bool PART>
void launch_ig(dim3 grid, hipStream_t st, const GemmArgs &a) {
  hipLaunchKernelGGL((igemm_kernel<DT, WGM, WGN, WTM, WTN, S, PART>), grid,
                     dim3(64 * WGM * WGN), 0, st, a);
}

// Tile configurations of the second-generation kernel (BM x BN); 64 x 128
// with a ring of 3 stages (two work-groups per CU) or of 5 (Deep: one).
enum IgCfg { kIg64x64 = 1, kIg64x128, kIg64x128Deep, kIg128x64, kIg128x128, kIg128x128Many, kIg128x256 };

template <int DT>
bool dispatch_ig(int cfg, bool part, dim3 grid, hipStream_t st, const GemmArgs &a) {
  if (part) {   // partial chunks: the two tiles the chooser takes for them
    switch (cfg) {
      case kIg64x64: launch_ig<DT, 4, 1, 1, 4, 4, true>(grid, st, a); return true;
      case kIg128x64: launch_ig<DT, 8, 1, 1, 4, 3, true>(grid, st, a); return true;
    }
    return false;
  }
  switch (cfg) {
    case kIg64x64: launch_ig<DT, 4, 1, 1, 4, 4, false>(grid, st, a); return true;
    case kIg64x128: launch_ig<DT, 4, 2, 1, 4, 3, false>(grid, st, a); return true;
    case kIg64x128Deep: launch_ig<DT, 4, 2, 1, 4, 5, false>(grid, st, a); return true;
    case kIg128x64: launch_ig<DT, 8, 1, 1, 4, 3, false>(grid, st, a); return true;
    case kIg128x128: launch_ig<DT, 4, 2, 2, 4, 3, false>(grid, st, a); return true;
    case kIg128x128Many: launch_ig<DT, 2, 2, 4, 4, 2, false>(grid, st, a); return true;
    case kIg128x256: launch_ig<DT, 2, 4, 4, 4, 3, false>(grid, st, a); return true;
  }
  return false;
}

// Tiles of the few-tile kernel (rows x columns); Long: 8 waves, Many: 2.
enum LkCfg {
  kLkNone, kLk16x16, kLk16x16Long, kLk16x32, kLk16x32Long, kLk16x64, kLk32x32, kLk32x64, kLk64x64,
  kLk64x64Many
};
struct LkTile {
  int cfg = kLkNone, bm = 0, bn = 0;
};

template <int DT, int TM, int TN, int NW, int S>
void launch_lk(bool part, dim3 grid, hipStream_t st, const GemmArgs &a) {
  if constexpr (DT != SPAROA_F32) {
    if (part) {
      hipLaunchKernelGGL((igemm_lk_kernel<DT, TM, TN, NW, S, true>), grid, dim3(64 * NW), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((igemm_lk_kernel<DT, TM, TN, NW, S, false>), grid, dim3(64 * NW), 0, st, a);
}

template <int DT>
bool dispatch_lk(int cfg, bool part, dim3 grid, hipStream_t st, const GemmArgs &a) {
  switch (cfg) {
    case kLk16x16: launch_lk<DT, 1, 1, 4, 4>(part, grid, st, a); return true;
    case kLk16x16Long: launch_lk<DT, 1, 1, 8, 4>(part, grid, st, a); return true;
    case kLk16x32: launch_lk<DT, 1, 2, 4, 4>(part, grid, st, a); return true;
    case kLk16x32Long: launch_lk<DT, 1, 2, 8, 3>(part, grid, st, a); return true;
    case kLk16x64: launch_lk<DT, 1, 4, 4, 3>(part, grid, st, a); return true;
    case kLk32x32: launch_lk<DT, 2, 2, 2, 4>(part, grid, st, a); return true;
    case kLk32x64: launch_lk<DT, 2, 4, 4, 3>(part, grid, st, a); return true;
  }
  if constexpr (DT == SPAROA_F32) {
    switch (cfg) {
      case kLk64x64: launch_lk<DT, 4, 4, 4, 2>(part, grid, st, a); return true;
      case kLk64x64Many: launch_lk<DT, 4, 4, 2, 2>(part, grid, st, a); return true;
    }
  }
  return false;
}

__global__ void set_u64(unsigned long long *p, unsigned long long v) { *p = v; }

template <int DT, int TM, int TN, bool VEC, bool SKIP>
void launch_tile(dim3 grid, hipStream_t st, const GemmArgs &a) {
  hipLaunchKernelGGL((gemm_kernel<DT, TM, TN, VEC, SKIP>), grid, dim3(kThreads), 0, st, a);
}

template <int DT, bool VEC, bool SKIP>
bool dispatch_tile(int bm, int bn, dim3 grid, hipStream_t st, const GemmArgs &a) {
  if constexpr (DT == SPAROA_F32) {  // fp32 tiles: 64 x 64 (LDS budget)
    if (bm != 64 || bn != 64) return false;
    launch_tile<DT, 2, 2, VEC, SKIP>(grid, st, a);
    return true;
  }
  if (bm == 128 && bn == 128) launch_tile<DT, 4, 4, VEC, SKIP>(grid, st, a);
  else if (bm == 128 && bn == 64) launch_tile<DT, 4, 2, VEC, SKIP>(grid, st, a);
  else if (bm == 64 && bn == 128) launch_tile<DT, 2, 4, VEC, SKIP>(grid, st, a);
  else if (bm == 64 && bn == 64) launch_tile<DT, 2, 2, VEC, SKIP>(grid, st, a);
  else return false;
  return true;
}

template <int DT>
bool dispatch(int bm, int bn, bool vec, bool skip, dim3 grid, hipStream_t st, const GemmArgs &a) {
  if (vec)
    return skip ? dispatch_tile<DT, true, true>(bm, bn, grid, st, a)
                : dispatch_tile<DT, true, false>(bm, bn, grid, st, a);
  return skip ? dispatch_tile<DT, false, true>(bm, bn, grid, st, a)
              : dispatch_tile<DT, false, false>(bm, bn, grid, st, a);
}

struct Shape {
  int64_t M, N, K, ho, wo;
};

Shape shape_of(const sparoa_conv_desc &d) {
  Shape s;
  s.ho = (d.h + 2 * d.ph - d.dh * (d.kh - 1) - 1) / d.sh + 1;
  s.wo = (d.w + 2 * d.pw - d.dw * (d.kw - 1) - 1) / d.sw + 1;
  s.M = d.n * s.ho * s.wo;
  s.N = d.c_out;
  s.K = d.kh * d.kw * d.c_in;
  return s;
}

}  // namespace

sparoa_status launch_set_u64(uint64_t *p, uint64_t v, hipStream_t stream) {
  hipLaunchKernelGGL(set_u64, dim3(1), dim3(1), 0, stream, reinterpret_cast<unsigned long long *>(p),
                     (unsigned long long)v);
  SPAROA_LAUNCH_CHECK("set_u64");
  return SPAROA_OK;
}

sparoa_status launch_split_reduce_group(const SplitReduceJob *jobs, int n, hipStream_t stream) {
  if (n < 1 || n > kGroupMax) return fail(SPAROA_ERR_INVALID_ARG, "split reduce: group size");
  ReduceGroup g;
  g.n = n;
  int64_t wg = 0;
  for (int j = 0; j < n; ++j) {
    const SplitReduceJob &r = jobs[j];
    if (r.dt != jobs[0].dt) return fail(SPAROA_ERR_INVALID_ARG, "split reduce: mixed dtypes");
    // 16-byte vectors need N % 8 == 0 and 16-byte aligned rows of bias / residual / y
    const int64_t items = r.N % 8 == 0 ? r.M * r.N / 8 : r.M * r.N;
    int64_t blocks = cdiv(items, 256);
    if (blocks > 2048) blocks = 2048;
    g.wg_begin[j] = (int)wg;
    g.partial[j] = r.partial;
    g.split[j] = r.split;
    g.M[j] = r.M;
    g.N[j] = r.N;
    g.bias[j] = static_cast<const char *>(r.bias);
    g.residual[j] = static_cast<const char *>(r.residual);
    g.act[j] = (int)r.act;
    g.y[j] = static_cast<char *>(r.y);
    g.om_counts[j] = r.om_counts;
    g.om_mask[j] = r.om_mask;
    g.om_words[j] = om_words_for(r.om_words, r.M * r.N, blocks);
    if (r.om_counts && (elem_size(r.dt) != 2 || r.N % 8 != 0))
      return fail(SPAROA_ERR_UNSUPPORTED, "split reduce: output measurement needs 16-bit, N % 8 == 0");
    wg += blocks;
  }
  g.wg_begin[n] = (int)wg;
  switch (jobs[0].dt) {
    case SPAROA_BF16:
      hipLaunchKernelGGL(split_reduce_group<SPAROA_BF16>, dim3((unsigned)wg), dim3(256), 0, stream, g);
      break;
    case SPAROA_F16:
      hipLaunchKernelGGL(split_reduce_group<SPAROA_F16>, dim3((unsigned)wg), dim3(256), 0, stream, g);
      break;
    case SPAROA_F32:
      hipLaunchKernelGGL(split_reduce_group<SPAROA_F32>, dim3((unsigned)wg), dim3(256), 0, stream, g);
      break;
  }
  SPAROA_LAUNCH_CHECK("split_reduce_group");
  return SPAROA_OK;
}

sparoa_status launch_split_reduce(const SplitReduceJob &job, hipStream_t stream) {
  return launch_split_reduce_group(&job, 1, stream);
}

namespace {
// Shapes the direct small-channel kernel serves (image stems).
bool small_c_eligible(const sparoa_conv_desc &d) {
  if (d.dtype == SPAROA_F32 || d.groups != 1 || d.dh != 1 || d.dw != 1) return false;
  if (d.c_in > 4 || d.kw > 8 || d.kh > 32) return false;
  if (!(d.c_out == 16 || d.c_out == 32 || d.c_out == 64)) return false;
  const Shape s = shape_of(d);
  if (s.wo > 16 * kScMaxRB || d.n * s.ho >= ((int64_t)1 << 31)) return false;
  if (cdiv(d.kh * ((d.kw + 1) / 2), 4) > kScMaxKSteps) return false;
  // one output row's patch [kh][PW + 1][4] beside its input rows and weights,
  // or beside its fp32 outputs, within kScPatchBytes
  const int64_t patch = cdiv(d.kh * (d.sw * (s.wo - 1) + d.kw + 1) * 8, 16) * 16;
  const int64_t staged = 2 * (cdiv(d.kh * d.w * d.c_in, 8) * 8 +
                              cdiv(d.c_out * d.kh * d.kw * d.c_in, 8) * 8);
  const int64_t tile = 16 * cdiv(s.wo, 16) * (d.c_out + 4) * 4;
  return patch + (staged > tile ? staged : tile) <= kScPatchBytes;
}

template <int DT, int KS>
void launch_small_c_kernel(int nb, dim3 grid, unsigned lds, hipStream_t st, const SmallCArgs &a) {
  if (nb == 4)
    hipLaunchKernelGGL((conv_small_c_kernel<DT, KS, 4>), grid, dim3(256), lds, st, a);
  else if (nb == 2)
    hipLaunchKernelGGL((conv_small_c_kernel<DT, KS, 2>), grid, dim3(256), lds, st, a);
  else
    hipLaunchKernelGGL((conv_small_c_kernel<DT, KS, 1>), grid, dim3(256), lds, st, a);
}

sparoa_status launch_small_c(const sparoa_conv_desc &d, const void *x, const void *w,
                             const void *bias, const void *residual, sparoa_act act, void *y,
                             bool skip, uint64_t *executed, hipStream_t stream,
                             const DeviceRoute *route, const OutMeasure *om) {
  if (om && om->mask)
    return fail(SPAROA_ERR_UNSUPPORTED, "small-channel conv: fused measurement is counts-only");
  const Shape s = shape_of(d);
  SmallCArgs a;
  a.x = static_cast<const char *>(x);
  a.w = static_cast<const char *>(w);
  a.bias = static_cast<const char *>(bias);
  a.residual = static_cast<const char *>(residual);
  a.y = static_cast<char *>(y);
  a.executed = reinterpret_cast<unsigned long long *>(skip ? executed : nullptr);
  a.H = (int)d.h; a.W = (int)d.w; a.C = (int)d.c_in;
  a.Ho = (int)s.ho; a.Wo = (int)s.wo; a.Cout = (int)d.c_out;
  a.kh = (int)d.kh; a.kw = (int)d.kw; a.sh = (int)d.sh; a.sw = (int)d.sw;
  a.ph = (int)d.ph; a.pw = (int)d.pw;
  a.PWP = (int)(d.sw * (s.wo - 1) + d.kw + 1);   // one column past the last tap
  a.pair = d.w * d.c_in % 2 == 0;
  a.bpr = (int)((d.kw + 1) / 2);
  const int ksteps = (int)cdiv(d.kh * a.bpr, 4);
  a.inv_bpr = 1.0f / (float)a.bpr;
  a.inv_pwp = 1.0f / (float)a.PWP;
  // Output rows per work-group: weights are laid out once per work-group and
  // neighbouring rows share input rows, so 4 where that still leaves 384
  // work-groups, else 2, else 1 (ResNet-50's stem at N = 8, 896 rows: 2 rows
  // 12.5 us, 1 row 17.9 us; at N = 1, 112 rows, latency).  Where a row has
  // fewer 16-pixel blocks than its share of the four waves, more rows cost a
  // wave nothing: taken while there are more work-groups than CUs (7 x 7, 64
  // channels, rows x Wo: 714 x 6 11.3 -> 6.5 us, 602 x 14 12.3 -> 7.0; at fewer
  // work-groups a second block for a wave, 192 x 48 5.3 and 6.1).
  const int64_t rows = d.n * s.ho;
  const int wbytes = (4 * ksteps + 1) * (int)d.c_out * 16;
  auto patch_bytes = [&](int64_t rw) { return ((rw - 1) * d.sh + d.kh) * a.PWP * 8; };
  a.rw = rows >= 4 * 384 ? 4 : (rows >= 2 * 384 ? 2 : 1);
  while (a.rw < 4 && cdiv(s.wo, 16) < 4 / a.rw && d.n * cdiv(s.ho, a.rw) > 256) a.rw *= 2;
  while (a.rw > 1 && wbytes + patch_bytes(a.rw) > kScLdsBytes) a.rw /= 2;
  a.prows = (a.rw - 1) * a.sh + a.kh;
  const int64_t both = wbytes + patch_bytes(a.rw);
  a.patch_off = both <= kScLdsBytes ? wbytes : 0;
  const unsigned lds = (unsigned)(a.patch_off ? both
                                              : (patch_bytes(a.rw) > wbytes ? patch_bytes(a.rw)
                                                                            : wbytes));
  a.groups = (int)cdiv(s.ho, a.rw);
  a.act = act;
  a.mode = route && route->counts ? 2 : (skip ? 1 : 0);
  a.route = route ? *route : DeviceRoute{nullptr, 0.0, 0, 0, nullptr};
  a.om_counts = om ? om->counts : nullptr;
  const dim3 grid((unsigned)(d.n * a.groups));
  a.om_words = om ? om_words_for(om->words, s.M * s.N, grid.x) : nullptr;
  const int nb = (int)d.c_out / 16;
  switch (ksteps) {
#define SPAROA_SC(K)                                                                         \
  case K:                                                                                    \
    if (d.dtype == SPAROA_BF16) launch_small_c_kernel<SPAROA_BF16, K>(nb, grid, lds, stream, a); \
    else launch_small_c_kernel<SPAROA_F16, K>(nb, grid, lds, stream, a);                     \
    break;
    SPAROA_SC(1) SPAROA_SC(2) SPAROA_SC(3) SPAROA_SC(4)
    SPAROA_SC(5) SPAROA_SC(6) SPAROA_SC(7) SPAROA_SC(8)
#undef SPAROA_SC
    default: return fail(SPAROA_ERR_UNSUPPORTED, "small-channel conv: k-steps");
  }
  SPAROA_LAUNCH_CHECK("conv_small_c_kernel");
  return SPAROA_OK;
}

// The second-generation kernel takes 16-bit convs whose channel count is a
// multiple of its 64-wide K chunk.
bool ig_eligible(const sparoa_conv_desc &d) {
  // 32-bit byte offsets into x and w; pixel indices below 2^24 (float divmod)
  if (d.n * d.h * d.w * d.c_in >= ((int64_t)1 << 30)) return false;
  if (shape_of(d).M >= ((int64_t)1 << 24) || d.kw > 32 || d.kh > 32) return false;
  if (d.c_out * d.kh * d.kw * d.c_in >= ((int64_t)1 << 30)) return false;
  // C_in a multiple of 8 (16-byte vectors); a tap's last chunk may be
  // partial (its channels past C_in read zero), from 48 channels up (below,
  // most of a chunk would be padding)
  return d.dtype != SPAROA_F32 && d.groups == 1 &&
         (d.c_in % kBK2 == 0 || (d.c_in % 8 == 0 && d.c_in >= 48)) &&
         d.kh * d.kw * cdiv(d.c_in, kBK2) <= kMaxChunks2 &&
         d.kh * d.kw * (d.c_in / 8) <= (int64_t)kMaxVecWords * 32;
}

// Column groups of the tile walk: the 8 XCDs' L2s read x once per group and
// the weights once per XCD of a group, so of 1, 2, 4 and 8 groups the one
// with the fewest bytes.
int64_t ig_column_groups(int64_t ntn, int64_t x_bytes, int64_t w_bytes) {
  int64_t best = 1;
  for (int64_t g = 2; g <= 8 && g <= ntn; g *= 2)
    if (x_bytes * g + w_bytes * (8 / g) < x_bytes * best + w_bytes * (8 / best)) best = g;
  return best;
}

// Tile of the second-generation kernel.  128 pixels where 128 x 64 tiles fill
// the chip, else 64.  Then the widest tile that still gives about one per CU:
// what bounds these kernels is the L2's delivery into LDS (17 - 20 TB/s over
// the chip, whatever the depth of the ring), and a tile of BM x BN takes
// 128 (BM + BN) bytes per chunk for BM BN products.  Measured (fp16, residual,
// one tile column of each row; M x N x K in us):
//   64 rows:  64 x 64 up to 256 tiles (2048 x 512 x 1024 9.6, 64 x 128 10.8),
//     else 64 x 128 (6272 x 256 x 256 7.0, 64 x 64 7.3), its deep ring from
//     32 chunks (6272 x 256 x 2304 16.2, 3 stages 17.4; x 1024 11.4, 11.3);
//   128 rows: 128 x 256 where it gives 192 to 256 tiles, or more of them and
//     12 chunks (25088 x 256 x 1024 23.1, 128 x 128 26.7; 50176 x 256 x 2304
//     65.2 and 72.2, x 576 32.6 and 31.6);
//     128 x 128 for up to 256 tiles of it (25088 x 128 x 1152 12.3, 128 x 64
//     12.6; x 2304 22.4 and 25.1), above that its form of four waves, two
//     work-groups per CU (50176 x 128 x 576 18.5, eight waves 22.9); 128 x 64
//     elsewhere.
// (partial chunks, C_in % 64 != 0: 64 channels wide only)
GemmTileChoice ig_choose(const Shape &s, int64_t c_in) {
  auto tiles = [&](int bm, int bn) { return cdiv(s.M, bm) * cdiv(s.N, bn); };
  GemmTileChoice t;
  t.kchunk = kBK2;
  const bool whole = c_in % t.kchunk == 0;
  const int64_t chunks = (s.K / c_in) * cdiv(c_in, t.kchunk);
  // BN-wide tiles waste at most an eighth of their columns
  auto wide = [&](int bn) { return whole && cdiv(s.N, bn) * bn - s.N <= s.N / 8; };
  if (tiles(128, 64) >= 240) {
    t.bm = 128;
    const int64_t n256 = tiles(128, 256), n128 = tiles(128, 128);
    if (wide(256) && n256 >= 192 && (n256 <= 256 || chunks >= 12)) {
      t.cfg = kIg128x256; t.bn = 256;
    } else if (wide(128) && n128 >= 160) {
      t.cfg = n128 <= 256 ? kIg128x128 : kIg128x128Many; t.bn = 128;
    } else {
      t.cfg = kIg128x64; t.bn = 64;
    }
  } else {
    t.bm = 64;
    if (wide(128) && tiles(64, 64) > 256) {
      t.cfg = chunks >= 32 ? kIg64x128Deep : kIg64x128; t.bn = 128;
    } else {
      t.cfg = kIg64x64; t.bn = 64;
    }
  }
  // chunks: whole or partial 64-channel blocks of each tap
  const int64_t tl = tiles(t.bm, 64), nchunks = chunks;
  int64_t split = 1;
  if (tl < 192) {   // (64 x 64 tiles: the wider ones are taken from 192 on)
    // The workspace that the query names, asked for also where the few-tile
    // kernel takes the layer (lk_choose) and leaves it unused; the rest are
    // layers of more than 256 tiles of 32 x 64, or of more than 512 chunks.
    // About one work-group per CU: more splits cost more partial traffic than
    // they gain (FC 64 x 4096 x 4096: split 4 15.1 us, split 8 17.8 us)
    split = cdiv(256, tl);
    if (split > 8) split = 8;
    if (split > nchunks / 4) split = nchunks / 4;
    if (split < 1) split = 1;
    // the reduction is a launch of its own (about 6 us on small outputs):
    // split only where the chunks it takes off a tile's walk (about 0.3 us
    // each on these under-filled grids) are worth more
    if (split > 1 && nchunks * (split - 1) < 20 * split) split = 1;
  }
  t.split_k = (int)split;
  return t;
}

// The tile of a few-tile layer that also writes a bitmap of its output.  Tiles
// narrower than 64 channels set and clear their bits by atomics, 32 of them on
// every word with 16 channels a tile, 16 with 32, and these end the kernel.
// Where they cost more than the wider tile's longer chain of chunks, the next
// tile up with the same number of waves (the same sums, bit for bit): rows
// that share words (under 256 channels), long rows (1024 up), and grids of 33
// to 64 work-groups, whose commits go straight to the counters.  Routed and
// measured, bf16, M x N x K in us, narrow and wide (and 64 x 64 tiles): 400 x
// 64 x 64 8.5, 5.9 (6.5); 196 x 128 x 512 9.0, 6.7 (8.7); 784 x 64 x 2304 10.7,
// 8.7 (12.0); 16 x 2048 x 64 8.2, 6.0 (6.8); 49 x 256 x 256 7.0, 6.1 (7.4);
// elsewhere 196 x 256 x 512 6.8, 7.3 (8.7); 100 x 512 x 1088 7.6, 8.3 (11.4);
// one row of tiles 1 x 64 x 1088 6.5, 7.2 (10.6).
LkTile lk_bitmap_tile(LkTile l, const Shape &s) {
  const int64_t wgs = cdiv(s.M, l.bm) * cdiv(s.N, l.bn);
  const bool wide = s.N < 256 ? s.M > 16 : s.N >= 1024 || (wgs > 32 && wgs <= 64);
  if (!wide) return l;
  if (l.cfg == kLk16x16 || l.cfg == kLk16x32) {
    l.cfg = kLk16x64;
    l.bn = 64;
  } else if (l.cfg == kLk16x16Long) {
    l.cfg = kLk16x32Long;
    l.bn = 32;
  }
  return l;
}

// Tile of the few-tile kernel, or none.  The narrowest of 16 x 16, 16 x 32,
// 16 x 64 and 32 x 64 of which there are at most 256, one per CU: their K loop
// is a chain of memory round trips, so a second tile on a CU costs as much
// again (fp16, K = 1024: 1024 x 512 16 x 64, 512 tiles, 9.5 us; 32 x 64, 256
// tiles, 6.7).  Against the 64-row tiles with K split over work-groups and
// their reduction (M x N x K, fp16): 784 x 128 x 1152 4.8 us and 7.9; 196 x
// 256 x 1024 4.5 and 7.8; 49 x 512 x 4608 6.4 and 10.2; 196 x 1024 x 256 4.3
// and 5.4; 2048 x 256 x 1024 6.7 and 8.0.  8 waves from 18 chunks (32: 5.1 and
// 5.3 us with 4; 16: 4.6 and 4.5).  Under 4 chunks the 32 x 64 tile's four
// waves have no work: 32 x 32 with two (2048 x 256 x 128 4.6 and 4.8).  Above
// 512 chunks a wave's chain is longer than a split's (288 chunks 12.6 us and
// 14.4, 0.24 and 0.19 us for each eight more).
// fp32 has no other kernel with whole 128-byte chunks, so 64 x 64 tiles beyond
// these where they win: four waves up to 256 tiles, else two, two work-groups
// a CU.  Against the general kernel, whose four work-groups a CU hide short
// walks and ragged stores better (M x N x K, us): up to 256 tiles from 2
// chunks (2488 x 256 x 32 8.6 and 7.7, x 64 8.8 and 8.9, x 512 16.6 and 23.3),
// from 16 with ragged rows (3000 x 300 x 64 11.0 and 9.3, x 512 18.9 and 24.9);
// up to 512 from 2 (6272 x 256 x 64 10.2 and 11.0, x 2048 77 and 109); up to
// 1024 from 12, where their rounds of 512 tiles are as full as rounds of 256
// (2048 x 2048 x 512 50 and 57, x 2048 149 and 187; 3000 x 1024 x 1152, 752
// tiles, 89 and 87); beyond from 24 (42120 x 512 x 768 336 and 366, an input of
// zeros only 72 and 52; x 512 243 and 254, zeros only 70 and 51).
// Measured without commit words (`direct`), each work-group's two atomics on
// the counters take their turn, 28 ns: above 80 work-groups, 128 from 3 chunks
// and 192 from 9, a layer whose K the 64-row tiles do not split runs in those,
// about a quarter as many (M x N x K, us: 3136 x 128 x 128 14.7 in 392 of the
// few-tile kernel, 7.9 in 98; 784 x 512 x 128 16.0 in 400, 9.2 in 104; 3136 x 64
// x 512 10.1 in 196, 8.6 in 49; 49 x 256 x 512 5.8 in 64, 7.7 in 4; 196 x 128 x
// 1152 7.1 in 104, 9.2 in 8).  Where they split K, and a reduction follows, the
// few-tile kernel stays ahead (196 x 512 x 4608 11.8 in 208, 15.2).
LkTile lk_choose(const sparoa_conv_desc &d, const Shape &s, const GemmTileChoice &t, bool bitmap,
                 bool direct) {
  LkTile l;
  const bool f32 = d.dtype == SPAROA_F32;
  const int64_t c = f32 ? kBK : kBK2, chunks = d.kh * d.kw * cdiv(d.c_in, c);
  if (f32) {   // byte offsets below 2^31; the indices and lists as in ig_eligible
    if (t.cfg || t.pointwise || t.small_c || d.groups != 1 || d.c_in % c) return l;
    if (d.n * d.h * d.w * d.c_in >= ((int64_t)1 << 29) || s.N * s.K >= ((int64_t)1 << 29)) return l;
    if (s.M >= ((int64_t)1 << 24) || d.kw > 32 || d.kh > 32 || chunks > kMaxChunks2) return l;
    if (d.kh * d.kw * (d.c_in / 8) > (int64_t)kMaxVecWords * 32) return l;
    if (cdiv(s.M, 64) * cdiv(s.N, 64) >= (int64_t)1 << 24) return l;
  } else if (!t.cfg || chunks > 512) {
    return l;
  }
  auto take = [&](int cfg, int bm, int bn) {
    if (direct && t.split_k == 1 &&
        cdiv(s.M, bm) * cdiv(s.N, bn) > (chunks < 3 ? 80 : chunks < 9 ? 128 : 192))
      return LkTile{};
    l.cfg = cfg;
    l.bm = bm;
    l.bn = bn;
    return bitmap ? lk_bitmap_tile(l, s) : l;
  };
  auto tiles = [&](int bm, int bn) { return cdiv(s.M, bm) * cdiv(s.N, bn); };
  const bool deep = chunks >= 18;
  if (tiles(16, 16) <= 256) return take(deep ? kLk16x16Long : kLk16x16, 16, 16);
  if (tiles(16, 32) <= 256) return take(deep ? kLk16x32Long : kLk16x32, 16, 32);
  if (tiles(16, 64) <= 256) return take(kLk16x64, 16, 64);
  if (tiles(32, 64) <= 256)
    return chunks < 4 ? take(kLk32x32, 32, 32) : take(kLk32x64, 32, 64);
  if (f32) {
    const int64_t t64 = tiles(64, 64);
    if (t64 <= 256)
      return chunks >= (s.N % 8 == 0 ? 2 : 16) ? take(kLk64x64, 64, 64) : l;
    const bool many = t64 <= 512    ? chunks >= 2
                      : t64 <= 1024 ? chunks >= 12 && cdiv(t64, 256) % 2 == 0
                                    : chunks >= 24;
    if (many && s.N % 8 == 0) return take(kLk64x64Many, 64, 64);
  }
  return l;
}

// Rows of the first launch of a layer in 128 x 256 tiles.  One such tile
// fills a CU, so a few tiles beyond whole rounds of 256 cost a round of their
// own; where few enough are left, their rows go to a second launch in the
// tiles that suit so many rows.  The first launch takes whole rows of tiles
// within the whole rounds, so what is left is more than tiles % 256 where the
// columns' tiles do not divide 256, and everything where one row has more
// tiles than the rounds hold.  The line lies at up to 128 left, without 65 to
// 79 (these take 260 to 316 128 x 64 tiles, more than one a CU).  One launch
// and two, bf16, M x N x K in us, with the tiles left: 3328 x 3072 x 2304 60
// 59.9 and 53.4; 384 x 22016 x 4096 86 93.1 and 82.1; 6528 x 3072 x 1024 108
// 57.5 and 56.7; 512 x 18944 x 1024 74 34.9 and 36.5; 1024 x 11008 x 768 129
// 30.9 and 35.1; 256 x 43520 x 4096 170 134 and 192.
int64_t ig_head_rows(const Shape &s, const GemmTileChoice &t) {
  if (t.cfg != kIg128x256) return s.M;
  const int64_t ntn = cdiv(s.N, t.bn), tiles = cdiv(s.M, t.bm) * ntn;
  const int64_t head = (tiles - tiles % 256) / ntn, left = tiles - head * ntn;
  const bool few = left <= 64 || (left >= 80 && left <= 128);
  return head > 0 && left > 0 && few ? head * t.bm : s.M;
}
}  // namespace

bool gemm_skip_supported(const sparoa_conv_desc &d) {
  const Shape s = shape_of(d);
  if (ig_eligible(d) || small_c_eligible(d)) return true;
  const int64_t bits = d.kh * d.kw * cdiv(d.c_in, 8);
  return cdiv(s.K, kBK) <= kMaxChunks && bits <= (int64_t)kMaxVecWords * 32;
}


bool conv_skip_reads_mask(const sparoa_conv_desc &d, sparoa_path path) {
  if (!(path & 1) || d.groups != 1 || !gemm_skip_supported(d)) return false;
  const GemmTileChoice t = gemm_choose(d, path);
  return !(t.pointwise || t.small_c);
}

GemmTileChoice gemm_choose(const sparoa_conv_desc &d, sparoa_path path) {
  const Shape s = shape_of(d);
  GemmTileChoice t;
  if ((path & 2) && pw_eligible(d)) {   // bandwidth path, 1x1: weights in LDS, x read once
    t.cfg = 0;
    t.bm = 16;      // skip unit: 16-pixel x 32-channel activation blocks
    t.bn = 16;
    t.kchunk = 32;
    t.split_k = 1;
    t.pointwise = true;
    return t;
  }
  if (ig_eligible(d)) return ig_choose(s, d.c_in);
  if (small_c_eligible(d)) {   // up to four output rows per work-group, 16-pixel row blocks
    t.cfg = 0;
    t.bm = 16;
    t.bn = 16;
    t.kchunk = 32;
    t.split_k = 1;
    t.small_c = true;
    return t;
  }
  t.cfg = 0;
  t.kchunk = kBK;
  if (d.dtype == SPAROA_F32) {
    t.bm = 64;
    t.bn = 64;
  } else {
    t.bn = s.N <= 64 ? 64 : 128;
    t.bm = 128;
    if (cdiv(s.M, t.bm) * cdiv(s.N, t.bn) < 256) t.bm = 64;
    if (cdiv(s.M, t.bm) * cdiv(s.N, t.bn) < 256) t.bn = 64;
  }
  const int64_t tiles = cdiv(s.M, t.bm) * cdiv(s.N, t.bn);
  const int64_t nchunks = cdiv(s.K, kBK);
  int64_t split = 1;
  if (tiles < 192) {
    split = cdiv(512, tiles);
    if (split > 8) split = 8;
    if (split > nchunks / 8) split = nchunks / 8;
    if (split < 1) split = 1;
  }
  t.split_k = (int)split;
  return t;
}

bool gemm_fuses_out_measure(const sparoa_conv_desc &d, sparoa_path path, bool bitmap) {
  const GemmTileChoice t = gemm_choose(d, path);
  // the pointwise kernel measures whole tiles of one weight slice
  if (t.pointwise) return pw_fuses_out_measure(d);
  // the small-channel kernel counts (no bitmap)
  if (t.small_c) return !bitmap;
  // every tile writes whole bitmap bytes, or sets its bits, when C_out % 64 ==
  // 0.  Else the layers whose K the 64-row tiles split, at any C_out % 8 == 0:
  // the reduction measures 16-byte vectors (a wave's 64 vectors are two whole
  // bitmap words), and the few-tile kernel, which takes most of these layers
  // without a split, its 8-channel blocks.  (It could measure its unsplit
  // layers as well; the 64-column tiles, which take them when they are measured
  // without commit words, could not.)
  if (t.cfg == 0 || elem_size(d.dtype) != 2) return false;
  if (d.c_out % 64 == 0) return true;
  // the K splits of the 64-row tiles (as launch_gemm_conv counts them)
  const int64_t nchunks = d.kh * d.kw * cdiv(d.c_in, t.kchunk);
  const int64_t gz = cdiv(nchunks, cdiv(nchunks, t.split_k));
  return gz > 1 && d.c_out % 8 == 0;
}

size_t gemm_workspace_required(const sparoa_conv_desc &d, sparoa_path path) {
  const GemmTileChoice t = gemm_choose(d, path);
  if (t.split_k <= 1) return 0;
  const Shape s = shape_of(d);
  return (size_t)t.split_k * (size_t)s.M * (size_t)s.N * sizeof(float);
}


sparoa_status launch_gemm_conv(const sparoa_conv_desc &d, sparoa_path path, const void *x,
                               const void *w, const void *bias, const void *residual,
                               sparoa_act act, const uint32_t *mask, void *y, void *ws,
                               size_t ws_bytes, uint64_t *executed, hipStream_t stream,
                               const DeviceRoute *route, SplitReduceJob *defer,
                               const OutMeasure *om) {
  const Shape s = shape_of(d);
  const GemmTileChoice t = gemm_choose(d, path);
  if (om && !gemm_fuses_out_measure(d, path, om->mask != nullptr))
    return fail(SPAROA_ERR_UNSUPPORTED, "GEMM: no fused output measurement for this shape");
  const int epv = d.dtype == SPAROA_F32 ? 4 : 8;
  const bool vec = d.c_in % epv == 0;
  // the skip form: x's bitmap given, or a skip path on a kernel that tests x
  // itself (the pointwise and small-channel kernels read no bitmap)
  const bool skip = mask != nullptr || ((path & 1) && (t.pointwise || t.small_c));
  // (the second-generation kernel's chunks are per tap: whole or partial
  // 64-channel blocks)
  const int64_t nchunks =
      t.cfg ? d.kh * d.kw * cdiv(d.c_in, t.kchunk) : cdiv(s.K, t.kchunk);
  if (skip && !gemm_skip_supported(d))
    return fail(SPAROA_ERR_UNSUPPORTED, "zero-skip conv: K above the skip kernel's 65536");
  if (s.M > INT32_MAX || s.N > INT32_MAX) return fail(SPAROA_ERR_UNSUPPORTED, "GEMM too large");

  GemmArgs a;
  a.x = static_cast<const char *>(x);
  a.w = static_cast<const char *>(w);
  a.bias = static_cast<const char *>(bias);
  a.residual = static_cast<const char *>(residual);
  a.y = static_cast<char *>(y);
  a.partial = static_cast<float *>(ws);
  a.mask = skip ? mask : nullptr;
  a.executed = reinterpret_cast<unsigned long long *>(skip ? executed : nullptr);
  a.M = s.M; a.N = s.N; a.K = s.K;
  a.H = d.h; a.W = d.w; a.Cin = d.c_in; a.Ho = s.ho; a.Wo = s.wo; a.Kw = d.kw;
  a.sh = d.sh; a.sw = d.sw; a.ph = d.ph; a.pw = d.pw; a.dh = d.dh; a.dw = d.dw;
  a.taps = d.kh * d.kw;
  a.x_bytes = d.n * d.h * d.w * d.c_in * elem_size(d.dtype);
  a.w_bytes = s.N * s.K * elem_size(d.dtype);
  a.inv_wo = 1.0f / (float)s.wo;
  a.inv_ho = 1.0f / (float)s.ho;
  a.nchunks = nchunks;
  a.kh32 = (int)d.kh;
  a.inv_kw = 1.0f / (float)d.kw;
  a.inv_dh = 1.0f / (float)d.dh;
  a.inv_dw = 1.0f / (float)d.dw;
  a.split = t.split_k;
  a.chunks_per_split = cdiv(nchunks, t.split_k);
  a.act = act;
  a.route = route ? *route : DeviceRoute{nullptr, 0.0, 0, 0, nullptr};
  if (!skip) a.route.counts = nullptr;   // no skip form to route to
  // the few-tile kernel splits K inside a work-group; the workspace that the
  // query names is asked for all the same
  const bool bitmap = om && om->mask;
  const bool direct = om && !om->words;
  const LkTile lk = lk_choose(d, s, t, bitmap, direct);
  const int64_t splits = cdiv(nchunks, a.chunks_per_split), gz = lk.cfg ? 1 : splits;
  a.split = (int)gz;
  // the epilogue measures y when it writes y; with split-K the reduction does
  a.om_counts = om && gz == 1 ? om->counts : nullptr;
  a.om_mask = om && gz == 1 ? om->mask : nullptr;
  // grouped count commit when the caller gives the words
  unsigned long long *om_words = om ? om->words : nullptr;
  a.om_words = gz == 1 ? om_words : nullptr;
  if (splits > 1 && ws_bytes < (size_t)splits * s.M * s.N * sizeof(float))
    return fail(SPAROA_ERR_WORKSPACE, "GEMM split-K workspace too small");

  if (executed) {
    hipLaunchKernelGGL(set_u64, dim3(1), dim3(1), 0, stream,
                       reinterpret_cast<unsigned long long *>(executed), 0ull);
    SPAROA_LAUNCH_CHECK("set_u64");
  }
  if (t.small_c) {
    if (defer) *defer = SplitReduceJob{d.dtype, nullptr, 0, s.M, s.N, bias, residual, act, y,
                                       nullptr, nullptr, nullptr};
    return launch_small_c(d, x, w, bias, residual, act, y, skip, executed, stream, route, om);
  }
  if (t.pointwise) {
    if (defer) *defer = SplitReduceJob{d.dtype, nullptr, 0, s.M, s.N, bias, residual, act, y,
                                       nullptr, nullptr, nullptr};
    return launch_pointwise(d, x, w, bias, residual, act, y, skip, executed, stream, route, om);
  }
  bool ok = false;
  if (t.cfg || lk.cfg) {
    const bool part = d.c_in % kBK2 != 0;   // a tap's last chunk is partial
    a.cpt32 = (int)cdiv(d.c_in, t.kchunk);
    a.inv_cpt = 1.0f / (float)a.cpt32;
    a.skip_rows = t.bm;
    // rows [row0, row0 + rows) in tiles of the few-tile kernel or of u.cfg
    unsigned long long *const words = a.om_words;
    auto launch_rows = [&](int64_t row0, int64_t rows, const LkTile &l, const GemmTileChoice &u) {
      const int64_t ntn = cdiv(s.N, l.cfg ? l.bn : u.bn);
      const int64_t ntmn = cdiv(rows, l.cfg ? l.bm : u.bm) * ntn;
      if (ntmn * gz >= (int64_t)1 << 24) return false;   // refused below
      const dim3 grid((unsigned)(ntmn * gz));
      a.row0 = (int)row0;
      a.om_words = om_words_for(words, s.M * s.N, ntmn);
      const int64_t gw = cdiv(ntn, ig_column_groups(ntn, a.x_bytes, a.w_bytes));
      const int64_t gt = ntmn / ntn * gw, lastw = ntn - (cdiv(ntn, gw) - 1) * gw;
      a.ntn32 = (int)ntn;
      a.ntmn32 = (int)ntmn;
      a.gw32 = (int)gw;
      a.gt32 = (int)gt;
      a.lastw32 = (int)lastw;
      a.inv_ntmn = 1.0f / (float)ntmn;
      a.inv_gt = 1.0f / (float)gt;
      a.inv_gw = 1.0f / (float)gw;
      a.inv_lastw = 1.0f / (float)lastw;
      switch (d.dtype) {
        case SPAROA_BF16:
          return l.cfg ? dispatch_lk<SPAROA_BF16>(l.cfg, part, grid, stream, a)
                       : dispatch_ig<SPAROA_BF16>(u.cfg, part, grid, stream, a);
        case SPAROA_F16:
          return l.cfg ? dispatch_lk<SPAROA_F16>(l.cfg, part, grid, stream, a)
                       : dispatch_ig<SPAROA_F16>(u.cfg, part, grid, stream, a);
        default:
          return l.cfg != 0 && dispatch_lk<SPAROA_F32>(l.cfg, part, grid, stream, a);
      }
    };
    const int64_t head = lk.cfg || gz > 1 ? s.M : ig_head_rows(s, t);
    ok = launch_rows(0, head, lk, t);
    if (ok && head < s.M) {
      Shape rest = s;
      rest.M = s.M - head;
      const GemmTileChoice u = ig_choose(rest, d.c_in);
      ok = launch_rows(head, rest.M, lk_choose(d, rest, u, bitmap, direct), u);
    }
  } else {
    const dim3 grid((unsigned)cdiv(s.M, t.bm), (unsigned)cdiv(s.N, t.bn), (unsigned)gz);
    switch (d.dtype) {
      case SPAROA_BF16: ok = dispatch<SPAROA_BF16>(t.bm, t.bn, vec, skip, grid, stream, a); break;
      case SPAROA_F16: ok = dispatch<SPAROA_F16>(t.bm, t.bn, vec, skip, grid, stream, a); break;
      case SPAROA_F32: ok = dispatch<SPAROA_F32>(t.bm, t.bn, vec, skip, grid, stream, a); break;
    }
  }
  if (!ok) return fail(SPAROA_ERR_UNSUPPORTED, "GEMM tile shape, or 2^24 tiles or more");
  SPAROA_LAUNCH_CHECK("gemm_kernel");
  const SplitReduceJob job{d.dtype, a.partial, gz > 1 ? (int)gz : 0, s.M, s.N, bias, residual,
                           act, y, om && gz > 1 ? om->counts : nullptr,
                           om && gz > 1 ? om->mask : nullptr, gz > 1 ? om_words : nullptr};
  if (defer) {
    *defer = job;
    return SPAROA_OK;
  }
  if (gz > 1) return launch_split_reduce(job, stream);
  return SPAROA_OK;
}

}  // namespace sparoa
