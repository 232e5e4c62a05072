// dam_mask_build: attention statistics at the pattern capture length -> per-head sparse mask.
//
// Paper (arXiv 2506.11104): Sec. 4.2.2 (mean, clamp, Box-Cox, global-min shift), Sec. 4.2.3 (true
// mask by threshold tau), Sec. 4.2.4 (diagonal / vertical pattern pool, match score gamma against
// mu), Sec. 4.3 (mask of a length-S problem: true mask inside the L x L block, matched patterns
// continued elsewhere). The tile pooling, block index and kept lists are this library's own data
// structures for the sparse attention kernels.
//
// Everything here is streaming bit work bounded by HBM bandwidth: A is read once (lower triangle
// only for a single causal capture), one wave turns 64 keys into one mask word with a ballot, and
// the S x S mask is never materialised: any 64-key word of any row is recomputed on the fly from
// the true bits, the column bitset and a bit-reversed diagonal bitset (one funnel shift).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "dam_internal.h"
#include "dam_slices.h"
#include "dam_turns.h"

#pragma clang fp contract(off)

namespace {
using namespace dam;

// Workgroups of a launch whose items are short: enough to fill the chip twice (256 CUs x 8 workgroups of
// 256 threads); each takes several items in turn.
constexpr int kGridTarget = 4096;
constexpr int kHeadSub = 16;  // partial sums per head of the listed-tile counts
// Query tiles of a head up to which k_pattern_prep scans them itself, a wave each, and the scan launch is saved. Whole layers,
// launch / this, us: 2 fp32 heads x 4 tiles 23.6 / 22.1, 8 x 10 37.4 / 35.1, 6 x 16 36.5 / 34.6, 32 heads x 16 (2048 tokens of
// patterns) 53.7 / 52.8, 64 x 16 (captured at 256) 67.8 / 66.8; builds in the plain layout 32 x 8 (1000 tokens) 18.9 / 17.2, 32 x 16
// 22.4 / 21.9. Two tiles per wave, on one CU per head: 32 x 32 (captured at 1024) 103.8 / 107.0, builds 8 x 32 21.2 / 25.9.
constexpr int kScanInPrep = 16;

struct Geom {
  int H, L, S, P;            // P: length of the pattern flag arrays (L from a map, S when given)
  int tile_m, tile_n, nQt, nKt, wpr;
  int tbw;                   // words per true_bits row, ceil(L / 64)
  int pw;                    // words per pattern bitset, ceil(P / 64)
  int occw;                  // occupancy words per query tile, ceil(nKt / 64)
};

// ------------------------------------------------------------------------------------------------
// Sec. 4.2.2 in the fixed fp32 sequence (each op rounded to nearest, nothing contracted: this file
// is compiled with contraction off and with correctly rounded fp32 divide and square root; the
// __fsqrt_rn / __fdiv_rn intrinsics are NOT used because they map to the approximate forms).
__host__ __device__ __forceinline__ float clamp_mean(float a, float c, float eps) {
  const float denom = c + eps;
  const float abar = a / denom;
  return fmaxf(abar, eps);
}

template <int LAMBDA2>  // 2 * lambda: 1 -> lambda 0.5, 2 -> lambda 1
__host__ __device__ __forceinline__ float box_cox(float x) {
  if (LAMBDA2 == 1) {
    const float root = sqrtf(x);
    const float num = root - 1.0f;
    return num / 0.5f;
  }
  return x - 1.0f;
}

__global__ void k_copy_f32(float *dst, const float *src) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = *src;
}

// General case: min over every stored entry. min B = B(min X) because every step after X is
// non-decreasing; X > 0, so its bit pattern orders like an unsigned integer.
__global__ void k_min_x(const float *__restrict__ A, const float *__restrict__ C, int64_t n, int L,
                        float eps, unsigned *xmin_bits) {
  float m = INFINITY;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    float a, c;
    if (C) {
      a = A[e];
      c = C[e];
    } else {  // only reached for L == 1 (a single valid pair per map)
      a = A[e];
      c = 1.0f;
    }
    m = fminf(m, clamp_mean(a, c, eps));
  }
  for (int off = 32; off; off >>= 1) m = fminf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) atomicMin(xmin_bits, __float_as_uint(m));
}

template <int LAMBDA2>
__global__ void k_bmin_from_x(const unsigned *xmin_bits, float *bmin) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *bmin = box_cox<LAMBDA2>(__uint_as_float(*xmin_bits));
}

__global__ void k_fill_u32(unsigned *p, int64_t n, unsigned v) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    p[e] = v;
}

// ------------------------------------------------------------------------------------------------
// Sec. 4.2.3: m[i][j] = (B - bmin >= tau) and j <= i. One wave = 4 rows x 4 words (256 keys); each
// lane owns one key per word so every load is a fully coalesced 256-byte row segment, and the
// 16 loads of a lane are independent. Entries above the diagonal are never kept, so never read.
constexpr int kTmRows = 64;  // rows per block (4 passes of 4 rows per wave)

// Every operation of the fixed fp32 sequence (divide by a positive constant, max, square root,
// subtract, compare) is rounded to nearest and therefore non-decreasing in its input, so the keep
// decision (Sec. 4.2.3) is a step function of the mean attention abar (of A itself when no count
// matrix is given: then abar = A / (1 + eps)): keep <=> value >= theta for one fp32 number theta.
// k_threshold finds theta by bisection over the ordered bit patterns of fp32, evaluating the exact
// sequence at each probe; k_true_mask then needs one comparison per element and stays bit-exact.
// Ordered key: increasing with the value over [-inf, +inf]; a NaN is treated as -inf, which is what
// the sequence does with it (fmaxf(NaN, eps) = eps, the smallest clamped value).
__host__ __device__ __forceinline__ unsigned key_of(float x) {
  const unsigned b = __builtin_bit_cast(unsigned, x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__host__ __device__ __forceinline__ float value_of(unsigned k) {
  return __builtin_bit_cast(float, (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}
constexpr unsigned kKeyNegInf = 0x007FFFFFu, kKeyPosInf = 0xFF800000u;
constexpr unsigned kKeepAll = 0u, kKeepNone = 0xFFFFFFFFu;

template <int LAMBDA2, bool FROM_A>
__host__ __device__ __forceinline__ bool keep_at(float v, float eps, float tau, float bmin) {
  const float x = FROM_A ? clamp_mean(v, 1.0f, eps) : fmaxf(v, eps);
  const float bstar = box_cox<LAMBDA2>(x) - bmin;
  return bstar >= tau;
}

// (host and device: the sequence is correctly rounded IEEE arithmetic on both, so when the minimum is known
// without looking at the data -- an override, or the closed form of a single causal capture -- the bisection runs
// on the host and the first kernel of the chain takes the key by value)
template <int LAMBDA2, bool FROM_A>
__host__ __device__ unsigned threshold_key(float eps, float tau, float bmin) {
  unsigned lo = kKeyNegInf, hi = kKeyPosInf;
  if (!keep_at<LAMBDA2, FROM_A>(value_of(hi), eps, tau, bmin)) return kKeepNone;
  if (keep_at<LAMBDA2, FROM_A>(value_of(lo), eps, tau, bmin)) return kKeepAll;
  while (hi - lo > 1u) {  // keep(lo) false, keep(hi) true
    const unsigned mid = lo + (hi - lo) / 2u;
    if (keep_at<LAMBDA2, FROM_A>(value_of(mid), eps, tau, bmin)) hi = mid;
    else lo = mid;
  }
  return hi;
}

template <int LAMBDA2, bool FROM_A>
__global__ void k_threshold(float eps, float tau, const float *__restrict__ bmin_p, unsigned *__restrict__ theta_key) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  *theta_key = threshold_key<LAMBDA2, FROM_A>(eps, tau, *bmin_p);
}

// ------------------------------------------------------------------------------------------------
// App. B: the alternative transforms between the mean map and the threshold (dam_transform other
// than Box-Cox). Every one of them is non-decreasing in the mean (raw sum: in the sum), so the same
// scheme applies: the statistics the transform needs are reduced over every stored entry, the
// minimum of the transformed map is the transform of the smallest input, and one thread bisects for
// the smallest input value that is kept. raw sum, average, min-max and square root are exact fp32
// sequences; log, Yeo-Johnson, arcsinh use the device's library functions and z-score sums in fp64
// with atomics, so their decisions can differ from another implementation's within rounding of the
// threshold.
struct TransformStats {
  unsigned xmin_bits, xmax_bits;  // X > 0: its bit pattern orders like an unsigned integer
  unsigned amin_key, abarmin_key; // ordered keys (see key_of) of the smallest sum and the smallest mean
  double sum, sumsq;              // of X
};

struct TransformCtx {
  int kind;
  float lambda, eps, tau, tmin, p0, p1;  // p0, p1: (mu, sigma) for z-score, (min X, max X) for min-max
};

__global__ void k_stats_init(TransformStats *st) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->xmin_bits = 0x7F800000u;
    st->xmax_bits = 0u;
    st->amin_key = kKeyPosInf;
    st->abarmin_key = kKeyPosInf;
    st->sum = 0.0;
    st->sumsq = 0.0;
  }
}

__global__ __launch_bounds__(256) void k_stats(const float *__restrict__ A, const float *__restrict__ C, int64_t n, int L,
                                               float eps, TransformStats *st) {
  float xmin = INFINITY, xmax = 0.0f;
  unsigned amin = kKeyPosInf, abarmin = kKeyPosInf;
  double sum = 0.0, sumsq = 0.0;
  const int64_t LL = (int64_t)L * L;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    float a, c;
    if (C) {
      a = A[e];
      c = C[e];
    } else {
      const int64_t r = e % LL;
      const bool causal = r % L <= r / L;
      a = causal ? A[e] : 0.0f;
      c = causal ? 1.0f : 0.0f;
    }
    const float denom = c + eps;
    const float abar = a / denom;
    const float x = fmaxf(abar, eps);
    xmin = fminf(xmin, x);
    xmax = fmaxf(xmax, x);
    amin = min(amin, key_of(a != a ? -INFINITY : a));
    abarmin = min(abarmin, key_of(abar != abar ? -INFINITY : abar));
    sum += (double)x;
    sumsq += (double)x * (double)x;
  }
  for (int off = 32; off; off >>= 1) {
    xmin = fminf(xmin, __shfl_xor(xmin, off));
    xmax = fmaxf(xmax, __shfl_xor(xmax, off));
    amin = min(amin, (unsigned)__shfl_xor((int)amin, off));
    abarmin = min(abarmin, (unsigned)__shfl_xor((int)abarmin, off));
    sum += __shfl_xor(sum, off);
    sumsq += __shfl_xor(sumsq, off);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMin(&st->xmin_bits, __float_as_uint(xmin));
    atomicMax(&st->xmax_bits, __float_as_uint(xmax));
    atomicMin(&st->amin_key, amin);
    atomicMin(&st->abarmin_key, abarmin);
    atomicAdd(&st->sum, sum);
    atomicAdd(&st->sumsq, sumsq);
  }
}

// The transform of a mean value abar (raw sum: of a sum) in the fixed fp32 sequence.
__device__ float transform_of(const TransformCtx &c, float v) {
  if (c.kind == DAM_T_RAW_SUM || c.kind == DAM_T_AVERAGE) return v;
  const float x = fmaxf(v, c.eps);
  switch (c.kind) {
    case DAM_T_LOG:
      return logf(x);
    case DAM_T_YEO_JOHNSON: {
      const float x1 = x + 1.0f;
      if (c.lambda == 0.0f) return logf(x1);
      const float p = powf(x1, c.lambda);
      const float num = p - 1.0f;
      return num / c.lambda;
    }
    case DAM_T_ZSCORE: {
      const float num = x - c.p0;
      const float den = c.p1 + c.eps;
      return num / den;
    }
    case DAM_T_MINMAX: {
      const float num = x - c.p0;
      const float range = c.p1 - c.p0;
      const float den = range + c.eps;
      return num / den;
    }
    case DAM_T_SQRT:
      return sqrtf(x);
    default:  // DAM_T_ARCSINH
      return asinhf(x);
  }
}

// Context of the transform and the threshold key. from_a: the compared value is the sum of a single
// capture (the mean is sum / (1 + eps)); otherwise it is the mean itself (raw sum: always the sum).
__global__ void k_transform_threshold(int kind, float lambda, float eps, float tau, float tmin_override,
                                      const TransformStats *__restrict__ st, bool from_a, float n_entries,
                                      double n_exact, float *__restrict__ bmin, unsigned *__restrict__ theta_key) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  TransformCtx c;
  c.kind = kind; c.lambda = lambda; c.eps = eps; c.tau = tau; c.p0 = 0.0f; c.p1 = 0.0f;
  const float xmin = __uint_as_float(st->xmin_bits), xmax = __uint_as_float(st->xmax_bits);
  if (kind == DAM_T_ZSCORE) {
    const double mean = st->sum / n_exact;
    double var = st->sumsq / n_exact - mean * mean;
    if (var < 0.0) var = 0.0;
    c.p0 = (float)mean;
    c.p1 = (float)sqrt(var);
  } else if (kind == DAM_T_MINMAX) {
    c.p0 = xmin;
    c.p1 = xmax;
  }
  // every transform is non-decreasing: the minimum of the map is the transform of the smallest input
  float tmin;
  if (kind == DAM_T_RAW_SUM) tmin = value_of(st->amin_key);
  else if (kind == DAM_T_AVERAGE) tmin = value_of(st->abarmin_key);
  else tmin = transform_of(c, xmin);
  if (tmin_override == tmin_override) tmin = tmin_override;
  c.tmin = tmin;
  *bmin = tmin;
  auto keep = [&](float v) {
    if (kind != DAM_T_RAW_SUM && from_a) {
      const float denom = 1.0f + eps;
      v = v / denom;
    }
    const float t = transform_of(c, v);
    return t - c.tmin >= tau;
  };
  unsigned lo = kKeyNegInf, hi = kKeyPosInf;
  if (!keep(value_of(hi))) {
    *theta_key = kKeepNone;
    return;
  }
  if (keep(value_of(lo))) {
    *theta_key = kKeepAll;
    return;
  }
  while (hi - lo > 1u) {
    const unsigned mid = lo + (hi - lo) / 2u;
    if (keep(value_of(mid))) hi = mid;
    else lo = mid;
  }
  *theta_key = hi;
}

// The threshold key comes from the workspace (theta_key) or, when the host found it, by value (theta_key == nullptr:
// theta_val, and bmin_val goes to the caller's bmin from here, this being the first kernel of the chain).
struct Threshold {
  const unsigned *theta_key = nullptr;
  unsigned theta_val = 0;
  float bmin_val = 0.0f;
  float *bmin_out = nullptr;
};

__device__ __forceinline__ unsigned take_threshold(const Threshold &t) {
  if (t.theta_key) return *t.theta_key;
  if (t.bmin_out && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) *t.bmin_out = t.bmin_val;
  return t.theta_val;
}

template <bool FROM_A, bool RAW = false>
__global__ __launch_bounds__(256) void k_true_mask(const float *__restrict__ A, const float *__restrict__ C, int L,
                                                   int tbw, float eps, Threshold thr,
                                                   uint64_t *__restrict__ true_bits) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = blockIdx.z;
  const int w0 = blockIdx.x * 4;
  const unsigned theta = take_threshold(thr);
  const float *Ah = A + (int64_t)h * L * L;
  const float *Ch = FROM_A ? nullptr : C + (int64_t)h * L * L;
  constexpr int kIter = kTmRows / 16;  // passes of 4 rows per wave
#pragma unroll 2
  for (int it = 0; it < kIter; ++it) {
    const int r0 = blockIdx.y * kTmRows + (it * 4 + wave) * 4;
    float a[4][4], c[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = r0 + r, j = (w0 + k) * 64 + lane;
        const bool live = i < L && j <= i;
        a[r][k] = live ? Ah[(int64_t)i * L + j] : 0.0f;
        if (!FROM_A) c[r][k] = live ? Ch[(int64_t)i * L + j] : 0.0f;
      }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int i = r0 + r, j = (w0 + k) * 64 + lane;
        const bool live = i < L && j <= i;
        float v = a[r][k];
        if (!FROM_A && !RAW) v = v / (c[r][k] + eps);
        if (v != v) v = -INFINITY;
        const uint64_t word = __ballot(live && key_of(v) >= theta);
        if (lane == 0 && i < L && w0 + k < tbw) true_bits[((int64_t)h * L + i) * tbw + w0 + k] = word;
      }
  }
}

// The same for the common case (no count matrix, L a multiple of 4) at streaming speed: one wave per
// row, 16-byte loads, the live 256-key segments of a 2048-key span in flight at once (of the last one what lies up to the
// diagonal), and the row's bits gathered into lanes so that they leave as one coalesced store (single 8-byte stores from one
// lane made the store path the bottleneck).
// Bound by the reads where the maps are long, by instructions too where they are short; us, with the last segment read whole and
// its bits gathered by a ballot for each component and word / this: 32 maps of 1024 21.8 / 16.8, 64 of 4096 437 / 411 (5.2 TB/s);
// layers of 4000 tokens captured at 512 73.4 / 69.9, 64 heads x 2000 at 256 65.6 / 62.7.
__device__ __forceinline__ float4 load_once(const float4 *p) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
  return make_float4(t.x, t.y, t.z, t.w);
}

// FAST: theta is the key of a normal positive number (or keeps nothing, a NaN once decoded), and then
// key_of(v) >= theta is the plain comparison v >= value_of(theta): zeros, denormals and negative values
// lie below theta in either order, a NaN fails both. Segments that end before the diagonal then cost one
// comparison per element (0.490 -> 0.475 ms for 64 maps of 4096 x 4096).
template <bool FAST>
__device__ __forceinline__ void true_mask_row(const float *__restrict__ A, int L, int tbw, int h, int i_any, unsigned theta,
                                              uint64_t *__restrict__ true_bits, int lane) {
  const int i = __builtin_amdgcn_readfirstlane(i_any);
  const float4 *row = reinterpret_cast<const float4 *>(A + ((int64_t)h * L + i) * L);
  unsigned *out = reinterpret_cast<unsigned *>(true_bits + ((int64_t)h * L + i) * tbw);
  const int nseg = i / 256 + 1;  // segments with a key <= i
  const float theta_f = value_of(theta);
  const unsigned place = 1u << (4 * (lane & 7));  // of the lane's first key among those of its eight lanes
  constexpr int kSeg = 8;  // 256-key segments in flight per pass
  for (int s0 = 0; s0 * 4 < tbw; s0 += kSeg) {
    float4 v[kSeg];
#pragma unroll
    for (int u = 0; u < kSeg; ++u) {
      const int j0 = (s0 + u) * 256 + lane * 4;
      v[u] = (s0 + u < nseg && j0 <= i) ? load_once(row + (s0 + u) * 64 + lane) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // Eight lanes' 32 keys are 32 bits next to each other: put together by their places, OR over the eight lanes. Of the eight
    // lanes, lane u keeps segment u's.
    unsigned mine = 0;
#pragma unroll
    for (int u = 0; u < kSeg; ++u) {
      if (s0 + u < nseg) {  // wave-uniform
        const int j0 = (s0 + u) * 256 + lane * 4;
        const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
        unsigned bits = 0;
        if (FAST && s0 + u < nseg - 1) {  // every key of the segment is <= i
#pragma unroll
          for (int e = 0; e < 4; ++e) bits |= x[e] >= theta_f ? place << e : 0u;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float val = x[e] != x[e] ? -INFINITY : x[e];
            bits |= j0 + e <= i && key_of(val) >= theta ? place << e : 0u;
          }
        }
        bits |= __builtin_amdgcn_update_dpp(0, bits, 0xB1, 0xF, 0xF, false);   // the other lane of two
        bits |= __builtin_amdgcn_update_dpp(0, bits, 0x4E, 0xF, 0xF, false);   // the other two of four
        bits |= __builtin_amdgcn_update_dpp(0, bits, 0x141, 0xF, 0xF, false);  // the other four of eight
        if ((lane & 7) == u) mine = bits;
      }
    }
    mine = __builtin_amdgcn_ds_bpermute(4 * ((lane & 7) * 8 + (lane >> 3)), mine);  // lane 8 u + d: 32 keys d of segment u
    if (s0 * 8 + lane < 2 * tbw) out[s0 * 8 + lane] = mine;
  }
}

// Rows are taken in quads (one row per wave); quad 2 p holds rows 4 p .. 4 p + 3, quad 2 p + 1 the rows
// that complement them, L - 1 - (4 p .. 4 p + 3), so that a pair of quads is the same work whatever p.
// A workgroup takes several pairs in turn (a little faster than a workgroup per quad: 0.60 -> 0.59 ms for
// 64 maps of 4096 x 4096).
template <bool FAST>
__device__ __forceinline__ void true_mask_pairs(const float *__restrict__ A, int L, int tbw, int n_pairs, unsigned theta,
                                                uint64_t *__restrict__ true_bits) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = blockIdx.y;
  const int half = (L + 1) / 2;
  for (int pair = blockIdx.x; pair < n_pairs; pair += gridDim.x) {
    const int lo = pair * 4 + wave, hi = L - 1 - lo;
    if (lo >= half) continue;
    true_mask_row<FAST>(A, L, tbw, h, lo, theta, true_bits, lane);
    if (hi >= half) true_mask_row<FAST>(A, L, tbw, h, hi, theta, true_bits, lane);
  }
}

__global__ __launch_bounds__(256) void k_true_mask_rows(const float *__restrict__ A, int L, int tbw, int n_pairs,
                                                        Threshold thr, uint64_t *__restrict__ true_bits) {
  const unsigned theta = take_threshold(thr);
  if (theta >= 0x80800000u) true_mask_pairs<true>(A, L, tbw, n_pairs, theta, true_bits);  // key of FLT_MIN
  else true_mask_pairs<false>(A, L, tbw, n_pairs, theta, true_bits);
}

// Sec. 4.2.4 numerators (see dam_slices.h).
// Form for rows of more than 128 words (capture lengths above 8192): two waves per chunk and 64 words, 64 rows each, added up
// through LDS; every word fetched from global memory by the lane that owns it (one launch for both pattern kinds: the
// upper half of the grid's x range counts diagonals). Bound by the chain of a wave's loads, eight rows at a time: whole builds with
// a wave per chunk / two, 1 map of 8256 tokens 98 / 75 us, 4 of 8256 187 / 163, 1 of 16384 183 / 161, 2 of 20000 400 / 378.
__global__ __launch_bounds__(256) void k_pattern_slices_wide(const uint64_t *__restrict__ true_bits, int L, int tbw,
                                                        int n_chunks, uint64_t *__restrict__ vslices,
                                                        uint64_t *__restrict__ dslices) {
  constexpr int kHalf = kChunkRows / 2;
  __shared__ uint64_t second[2][kThreadSlices][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = wave & 1;
  const int h = blockIdx.z;
  const int chunk = blockIdx.y * 2 + (wave >> 1);
  const int xw = gridDim.x / 2;
  const bool DIAG = (int)blockIdx.x >= xw;  // block-uniform
  uint64_t *slices = DIAG ? dslices : vslices;
  const int wl = ((int)blockIdx.x - (DIAG ? xw : 0)) * 64 + lane;  // word of columns (or of diagonal offsets) owned by this lane
  const int i0 = chunk * kChunkRows + half * kHalf;
  const uint64_t *tb = true_bits + (int64_t)h * L * tbw;
  uint64_t s[kThreadSlices];
#pragma unroll
  for (int k = 0; k < kThreadSlices; ++k) s[k] = 0;
  // a column (offset) block that starts beyond the last of the rows holds no kept entry
  if (wl < tbw && 64 * wl <= i0 + kHalf - 1) {
    for (int g = 0; g < kHalf; g += 8) {
      uint64_t w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + g + u;
        uint64_t x = 0;
        if (i < L) {
          if (!DIAG) {
            x = tb[(int64_t)i * tbw + wl];
          } else {
            const int jhi = i - 64 * wl;  // the column of offset r = 64 wl in this row
            if (jhi >= 0) {
              const int wj = jhi >> 6, sh = (jhi & 63) + 1;  // window = bits jhi-63 .. jhi of the row
              const uint64_t hi = tb[(int64_t)i * tbw + wj];
              const uint64_t lo = wj > 0 ? tb[(int64_t)i * tbw + wj - 1] : 0;
              const uint64_t win = sh == 64 ? hi : ((hi << (64 - sh)) | (lo >> sh));
              x = __brevll(win);                             // offset r = 64 wl + t at bit t
            }
          }
        }
        w[u] = x;
      }
      add_eight(s, w);
    }
  }
  if (half) {
#pragma unroll
    for (int k = 0; k < kThreadSlices; ++k) second[wave >> 1][k][lane] = s[k];
  }
  __syncthreads();
  if (half || chunk >= n_chunks || wl >= tbw) return;
  uint64_t *out = slices + (((int64_t)h * n_chunks + chunk) * tbw + wl) * kSlices;
  uint64_t carry = 0;
#pragma unroll
  for (int k = 0; k < kThreadSlices; ++k) {
    csa(carry, s[k], s[k], second[wave >> 1][k][lane], carry);
    out[k] = s[k];
  }
  out[kThreadSlices] = carry;
}
static_assert(kSlices == kThreadSlices + 1, "two waves' counts");

// Form for rows of up to 128 words: one workgroup per (head, chunk).
__global__ __launch_bounds__(256) void k_pattern_slices(const uint64_t *__restrict__ true_bits, int L, int tbw, int n_chunks,
                                                        uint64_t *__restrict__ vslices, uint64_t *__restrict__ dslices) {
  __shared__ uint64_t sm[kSliceLds / sizeof(uint64_t)];
  const int chunk = gridDim.x - 1 - blockIdx.x, h = blockIdx.y, i0 = chunk * kChunkRows;  // the long rows first
  const int64_t at = ((int64_t)h * n_chunks + chunk) * kSlices * tbw;
  count_chunk(true_bits + ((int64_t)h * L + i0) * tbw, min(kChunkRows, L - i0), tbw, chunk, sm, vslices + at, dslices + at);
}

// Transpose of the 64 x 64 bit matrix whose row l is the word x of lane l: lane r returns the word whose
// bit l is bit r of lane l's x. Six exchange steps on blocks of 32, 16, ... 1 bits, all in the vector registers (lane
// swaps, row rotations, byte permutes: some 45 instructions; exchanges through LDS waited for it six times).
__device__ __forceinline__ uint64_t transpose64(uint64_t x, int lane) {
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  // blocks of 32: the upper halves of lanes 0 .. 31 against the lower halves of lanes 32 .. 63
  u32x2 v = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)(x >> 32), false, false);
  const unsigned sel16 = lane & 16 ? 0x07060302u : 0x05040100u, sel8 = lane & 8 ? 0x03070105u : 0x06020400u;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    unsigned w = v[k];
    // 16: even rows' values and odd rows' values, in all lanes
    const u32x2 rows = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    w = __builtin_amdgcn_perm(rows[1], rows[0], sel16);
    // 8: lane ^ 8 is the row turned by eight
    unsigned other = __builtin_amdgcn_update_dpp(0, w, 0x128, 0xF, 0xF, false);
    w = __builtin_amdgcn_perm(other, w, sel8);
    auto step = [&](unsigned from, int j, unsigned low) {  // low: the lower j bits of every 2 j
      const bool up = (lane & j) != 0;
      const unsigned turned = __builtin_amdgcn_alignbit(from, from, up ? j : 32 - j), take = up ? low : ~low;
      return (turned & take) | (w & ~take);
    };
    other = __builtin_amdgcn_update_dpp(0, w, 0x141, 0xF, 0xF, false);      // lane ^ 7, and
    other = __builtin_amdgcn_update_dpp(0, other, 0x1B, 0xF, 0xF, false);   // ^ 3: lane ^ 4
    w = step(other, 4, 0x0F0F0F0Fu);
    w = step(__builtin_amdgcn_update_dpp(0, w, 0x4E, 0xF, 0xF, false), 2, 0x33333333u);
    v[k] = step(__builtin_amdgcn_update_dpp(0, w, 0xB1, 0xF, 0xF, false), 1, 0x55555555u);
  }
  return (uint64_t)v[1] << 32 | v[0];
}

// gamma = count / size >= mu for pattern p of head h (Sec. 4.2.4), counts summed over the row chunks: a wave per word of 64
// patterns. A lane fetches one slice of one chunk, eight chunks to a fetch; the fetches of a batch, whose lanes hold slices of the
// same weight, are added up bit by bit (seven to three words), and each of the three turned around is, in the lane of a pattern,
// eight counts of a byte. blockIdx.z: 0 vertical, 1 diagonal patterns.
// (Thread by thread through bit-sliced sums of 17 slices and a tree of sixteen in LDS this
// launch took 12 us at 64 heads x 4096, now 6.6; capture of 4096 tokens 332 -> 326 us, 64 x 2048 103.4 -> 99.1, 32 x 1024 37.1 -> 32.1.)
constexpr int kMaxCountBits = 17;  // counts below 2^17: pcl is limited accordingly
__global__ __launch_bounds__(256) void k_pattern_finish(const uint64_t *__restrict__ vslices,
                                                        const uint64_t *__restrict__ dslices, int L, int tbw,
                                                        int n_chunks, float mu, int *__restrict__ vert_cnt,
                                                        int *__restrict__ diag_cnt, uint8_t *__restrict__ vert_flag,
                                                        uint8_t *__restrict__ diag_flag) {
  static_assert(kSlices == 8, "a count is a byte");
  constexpr int kEach = 7;
  const int lane = threadIdx.x & 63, word = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), h = blockIdx.y;
  if (word >= tbw) return;
  const bool diag = blockIdx.z == 1;
  const uint64_t *slices = (diag ? dslices : vslices) + ((int64_t)h * n_chunks * tbw + word) * kSlices + (lane & 7);
  int n = 0;
  // rows above pattern p hold nothing of it: start at the chunk of the word's first
  for (int c0 = word * 64 / kChunkRows; c0 < n_chunks; c0 += 8 * kEach) {
    uint64_t w[kEach];
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int chunk = c0 + 8 * u + (lane >> 3);
      w[u] = 0;
      if (c0 + 8 * u < n_chunks) {  // wave-uniform
        const uint64_t v = slices[(int64_t)min(chunk, n_chunks - 1) * tbw * kSlices];
        w[u] = chunk < n_chunks ? v : 0;
      }
    }
    uint64_t s[3], t0, t1;
    csa(t0, s[0], w[0], w[1], w[2]);
    csa(t1, s[0], s[0], w[3], w[4]);
    uint64_t t2;
    csa(t2, s[0], s[0], w[5], w[6]);
    csa(s[2], s[1], t0, t1, t2);
#pragma unroll
    for (int y = 0; y < 3; ++y)
      if (y == 0 || c0 + 8 * ((1 << y) - 1) < n_chunks) {  // (2 and 4 at once take that many fetches; wave-uniform)
        const uint64_t counts = transpose64(s[y], lane);
        const unsigned sum = __builtin_amdgcn_udot4((unsigned)(counts >> 32), 0x01010101u,
                                                    __builtin_amdgcn_udot4((unsigned)counts, 0x01010101u, 0u, false), false);
        n += (int)(sum << y);
      }
  }
  const int p = 64 * word + lane;
  if (p >= L) return;
  const int64_t e = (int64_t)h * L + p;
  if (int *out = diag ? diag_cnt : vert_cnt) out[e] = n;
  (diag ? diag_flag : vert_flag)[e] = (uint8_t)((float)n / (float)(L - p) >= mu);
}

// Eight flag bytes, four to a word, as eight bits: each byte's top bit is set where the byte is not zero, and a dot product with
// the bits' places adds them up (128 times the result). The multiplications that gather such bits otherwise run at a quarter of
// the rate.
__device__ __forceinline__ unsigned bits_of_8(unsigned lo, unsigned hi) {
  auto not_zero = [](unsigned x) { return (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u; };
  return __builtin_amdgcn_udot4(not_zero(hi), 0x80402010u, __builtin_amdgcn_udot4(not_zero(lo), 0x08040201u, 0, false), false) >> 7;
}
__device__ __forceinline__ unsigned bits_of_16(const uint4 &v) { return bits_of_8(v.x, v.y) | bits_of_8(v.z, v.w) << 8; }

// Flags -> bitsets. cbits bit c = column c matched. rrev bit q = diagonal (pw*64 - 1 - q) matched,
// i.e. the diagonal set reversed, so that the 64 offsets i-j, i-j-1, ... of one mask word are 64
// consecutive ascending bits. Four lanes build one word, 16 flag bytes each. (every thread of the workgroup calls this; 512 words
// per pass)
// A piece is read where it lies, at any alignment, and one that the row's end cuts from 16 bytes before that end and shifted:
// no lane is asked, so all of a pass's loads are under way together. (Aligned rows by 16 bytes with a branch around the last
// piece, others byte by byte: 4.2 us of the prep kernel at 32 heads x 32768 tokens, now 2.7.)
__device__ __forceinline__ void pattern_bitsets_of_head(const uint8_t *__restrict__ diag_flag,
                                                        const uint8_t *__restrict__ vert_flag, int P, int pw, int h,
                                                        uint64_t *__restrict__ cbits, uint64_t *__restrict__ rrev,
                                                        uint64_t *lds_copy) {  // both sets again, [2 pw], or nullptr
  const int part = threadIdx.x & 3;
  const uint8_t *rows[2] = {vert_flag + (int64_t)h * P, diag_flag + (int64_t)h * P};
  const int each = blockDim.x / 4;
  constexpr int kWords = 2;
  for (int w0 = 0; w0 < pw; w0 += kWords * each) {
    unsigned piece[kWords][2];
    if (P >= 16) {
      uint4 v[kWords][2];
      int past[kWords][2];
#pragma unroll
      for (int u = 0; u < kWords; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int w = w0 + u * each + (int)(threadIdx.x >> 2);
          const int first = (k ? pw - 1 - w : w) * 64 + part * 16;  // ascending offsets in a reversed word
          const int at = min(max(first, 0), P - 16);
          past[u][k] = min(first - at, 16);  // (below 0 only for a word that does not exist)
          __builtin_memcpy(&v[u][k], rows[k] + at, 16);
        }
#pragma unroll
      for (int u = 0; u < kWords; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) piece[u][k] = bits_of_16(v[u][k]) >> max(past[u][k], 0);
    } else {
#pragma unroll
      for (int u = 0; u < kWords; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          piece[u][k] = 0;
          const int w = w0 + u * each + (int)(threadIdx.x >> 2);
          if (w == 0 && part == 0)
            for (int y = 0; y < P; ++y) piece[u][k] |= (rows[k][y] != 0 ? 1u : 0u) << y;
        }
    }
#pragma unroll
    for (int u = 0; u < kWords; ++u) {
      const int w = w0 + u * each + (int)(threadIdx.x >> 2);
      uint64_t cw = (uint64_t)piece[u][0] << (16 * part), rw = (uint64_t)piece[u][1] << (16 * part);
      cw |= __shfl_xor(cw, 1);
      cw |= __shfl_xor(cw, 2);
      rw |= __shfl_xor(rw, 1);
      rw |= __shfl_xor(rw, 2);
      if (w < pw && part == 0) {
        const uint64_t rev = __brevll(rw);  // bit q of the word <- offset (pw*64 - 1) - (64 w + q)
        cbits[(int64_t)h * pw + w] = cw;
        rrev[(int64_t)h * pw + w] = rev;
        if (lds_copy) {
          lds_copy[w] = cw;
          lds_copy[pw + w] = rev;
        }
      }
    }
  }
}

// Word w of a bitset of pw words, 0 outside it. The index is clamped before the address is formed: the
// set may live in LDS, and an address formed below the start of the LDS window is not an LDS address
// any more, even if an instruction offset would bring it back inside.
__device__ __forceinline__ uint64_t set_word(const uint64_t *__restrict__ bs, int w, int pw) {
  const bool ok = (unsigned)w < (unsigned)pw;
  const uint64_t v = bs[ok ? w : 0];
  return ok ? v : 0;
}

// ------------------------------------------------------------------------------------------------
// Sec. 4.3: the 64 mask bits of row i, keys [64 wj, 64 wj + 64) of one head.
__device__ __forceinline__ uint64_t diag_window(const uint64_t *__restrict__ rrev, int pw, int64_t u) {
  // bit t <- diagonal offset u - t; in the reversed set that is position s0 + t.
  const int64_t Q = (int64_t)pw * 64 - 1;
  const int64_t s0 = Q - u;
  if (s0 > Q || s0 + 63 < 0) return 0;
  const int64_t w0 = s0 >> 6;
  const int sh = (int)(s0 & 63);
  const uint64_t lo = set_word(rrev, (int)w0, pw);
  if (sh == 0) return lo;
  const uint64_t hi = set_word(rrev, (int)w0 + 1, pw);
  return (lo >> sh) | (hi << (64 - sh));
}

// Keys of [64 wj, 64 wj + 64) that row i < L may keep in the true-mask block: causal, and columns below L.
__device__ __forceinline__ uint64_t in_true_block(const Geom &g, int i, int wj) {
  const int64_t u = (int64_t)i - (int64_t)wj * 64, left = (int64_t)g.L - (int64_t)wj * 64;
  const uint64_t causal = u < 0 ? 0ull : u >= 63 ? ~0ull : ((2ull << u) - 1);
  return left >= 64 ? causal : left <= 0 ? 0ull : causal & ((1ull << left) - 1);
}

__device__ __forceinline__ uint64_t mask_word(const Geom &g, const uint64_t *__restrict__ tb_h,
                                              const uint64_t *__restrict__ cb_h,
                                              const uint64_t *__restrict__ rr_h, int i, int wj) {
  if (i >= g.S) return 0;
  const int64_t u = (int64_t)i - (int64_t)wj * 64;
  if (u < 0) return 0;
  const uint64_t causal = u >= 63 ? ~0ull : ((2ull << u) - 1);
  if (i < g.L) {  // top-left block (and the whole mask when S <= L): the true mask
    const int64_t left = (int64_t)g.L - (int64_t)wj * 64;  // > 0 because j <= i < L
    const uint64_t inside = left >= 64 ? ~0ull : ((1ull << left) - 1);
    return tb_h[(int64_t)i * g.tbw + wj] & causal & inside;
  }
  uint64_t pat = cb_h ? set_word(cb_h, wj, g.pw) : 0;  // cb_h == nullptr: the diagonal part alone
  pat |= diag_window(rr_h, g.pw, u);
  return pat & causal;
}

// Any set bit among positions [lo, hi] of a bitset of nw words (positions outside it read as 0).
__device__ __forceinline__ bool range_any(const uint64_t *__restrict__ bs, int nw, int64_t lo, int64_t hi) {
  lo = max(lo, (int64_t)0);
  hi = min(hi, (int64_t)nw * 64 - 1);
  if (lo > hi) return false;
  for (int64_t w = lo >> 6; w <= (hi >> 6); ++w) {
    uint64_t m = bs[w];
    if (w == (lo >> 6)) m &= ~0ull << (lo & 63);
    if (w == (hi >> 6)) m &= ~0ull >> (63 - (hi & 63));
    if (m) return true;
  }
  return false;
}

// A tile strictly below the diagonal and outside the true-mask block holds only pattern entries:
// (i, j) is kept iff column j is matched or offset i - j is. Rows [i0, i1], columns [j0, j1]: some column of the tile is matched,
// or some offset in [i0 - j1, i1 - j0] is. (cb == nullptr: no columns.)
__device__ __forceinline__ bool pattern_tile_any(const uint64_t *__restrict__ cb, const uint64_t *__restrict__ rr, int pw, int i0, int i1,
                                                 int j0, int j1) {
  const int64_t Q = (int64_t)pw * 64 - 1;  // offset u sits at position Q - u of the reversed set
  return (cb && range_any(cb, pw, j0, j1)) || range_any(rr, pw, Q - (i1 - j0), Q - (i0 - j1));
}

// Every entry of row i in the words [w0, w0 + W) is kept, the columns' part as above.
__device__ __forceinline__ bool pattern_row_full(const uint64_t *__restrict__ cb, const uint64_t *__restrict__ rr, int pw, int i, int w0, int W) {
  uint64_t all = ~0ull;
  for (int w = w0; w < w0 + W; ++w) all &= (cb ? set_word(cb, w, pw) : 0) | diag_window(rr, pw, (int64_t)i - (int64_t)w * 64);
  return all == ~0ull;
}

// Every column of the tile of row i0 and words [w0, w0 + wpr) is matched, or every offset that it meets. (Tiles begin at multiples of
// 64: the offsets are (tile_m + tile_n) / 64 whole words but for the last bit, as in the classes below.)
__device__ __forceinline__ bool pattern_tile_all(const Geom &g, const uint64_t *__restrict__ cb, const uint64_t *__restrict__ rr, int i0, int w0) {
  uint64_t columns = cb ? ~0ull : 0, offsets = ~0ull;
  for (int y = 0; cb && y < g.wpr; ++y) columns &= set_word(cb, w0 + y, g.pw);
  const int end = g.pw - i0 / 64 + w0 + g.wpr;
  for (int y = 1; y <= (g.tile_m + g.tile_n) / 64; ++y) offsets &= set_word(rr, end - y, g.pw) | (y == 1 ? 1ull << 63 : 0);
  return columns == ~0ull || offsets == ~0ull;
}

// Classes of whole tiles for square tiles of width T, per head (pattern region, tile strictly below
// the diagonal): the entries of tile (qt, kt) have the columns of key tile kt and exactly the offsets
// T d - (T - 1) .. T d + (T - 1), d = qt - kt. So "some column matched" / "all columns matched" is a
// property of kt alone and "some offset matched" / "all offsets matched" of d alone. The d classes
// are stored reversed (d at position 64 dw - 1 - d), like the diagonal set, so that the 64 key tiles
// of an occupancy word are 64 consecutive bits.
// A head's words lie together: [some columns, all columns, some offsets, all offsets][occw].
enum { kColAny = 0, kColAll = 1, kOffAny = 2, kOffAll = 3 };
__device__ __forceinline__ void tile_classes_of_head(const Geom &g, const uint64_t *__restrict__ cb,  // the head's sets
                                                     const uint64_t *__restrict__ rr, uint64_t *__restrict__ classes,
                                                     uint64_t *lds_copy) {  // or nullptr
  // Tiles are whole words wide: the columns of a key tile are W = T / 64 words of the column set, the offsets of distance d
  // the 2 W words from pw - W (d + 1) on of the reversed diagonal set, but for the last bit (offset T (d - 1), which the tile
  // does not meet). So a lane reads its words side by side and waits once; a wave per word of either kind.
  const int lane = threadIdx.x & 63, W = g.tile_n / 64;
  for (int x = threadIdx.x >> 6; x < 2 * g.occw; x += blockDim.x >> 6) {
    const int w = x >> 1;
    uint64_t any = 0, all = ~0ull;
    bool live;
    if (x & 1) {
      const int kt = w * 64 + lane;
      live = kt < g.nKt;
#pragma unroll
      for (int y = 0; y < 4; ++y)
        if (y < W) {
          const uint64_t v = set_word(cb, kt * W + y, g.pw);
          any |= v;
          all &= v;
        }
    } else {
      const int d = g.occw * 64 - 1 - (w * 64 + lane), first = g.pw - W * (d + 1);
      live = d >= 1 && d < g.nQt;
#pragma unroll
      for (int y = 0; y < 8; ++y)
        if (y < 2 * W) {
          const uint64_t v = set_word(rr, first + y, g.pw), spare = y == 2 * W - 1 ? 1ull << 63 : 0;
          any |= v & ~spare;
          all &= v | spare;
        }
    }
    const uint64_t wa = __ballot(live && any != 0), wf = __ballot(live && all == ~0ull);
    if (lane == 0) {
      const int at = (x & 1 ? kColAny : kOffAny) * g.occw + w;
      classes[at] = wa;
      classes[at + g.occw] = wf;
      if (lds_copy) {
        lds_copy[at] = wa;
        lds_copy[at + g.occw] = wf;
      }
    }
  }
}

// The column bitset and the reversed diagonal bitset of one head, copied into LDS by the whole
// workgroup when they fit (lds_words = 2 pw, else 0): every mask word then costs LDS reads instead
// of dependent global loads. Contains a barrier. The callers then run their body on the
// LDS array itself, in a call of its own: only then does the compiler know the address space of the sets and read
// them with LDS instructions (a pointer that may be either is read through the flat path, with waits on both counters).
constexpr size_t kMaxStagedBytes = 48 * 1024;
constexpr int kGuardFront = 4, kGuardBack = 2;

inline size_t staged_bytes(const Geom &g) {
  const size_t b = ((size_t)g.pw * 2 + kGuardFront + kGuardBack) * sizeof(uint64_t);
  return b <= kMaxStagedBytes ? b : 0;
}
inline size_t class_bytes(const Geom &g) { return (size_t)g.occw * 4 * sizeof(uint64_t); }
constexpr size_t kMaxWithClasses = 56 * 1024;  // (64 KiB less what the kernels hold besides)

// Layout: the column set (pw words), kGuardFront zero words, the reversed diagonal set (pw words), kGuardBack zero
// words: words -kGuardFront .. -1 and pw, pw + 1 of the staged diagonal set read as empty without a test; behind them the
// head's class words, where they are wanted (n_classes).
__device__ __forceinline__ void stage_sets(uint64_t *lds_sets, int pw, const uint64_t *cb, const uint64_t *rr,
                                           const uint64_t *classes = nullptr, int n_classes = 0) {
  for (int x = threadIdx.x; x < n_classes; x += blockDim.x) lds_sets[2 * pw + kGuardFront + kGuardBack + x] = classes[x];
  for (int x = threadIdx.x; x < pw; x += blockDim.x) {
    lds_sets[x] = cb[x];
    lds_sets[pw + kGuardFront + x] = rr[x];
  }
  if (threadIdx.x < kGuardFront + kGuardBack)
    lds_sets[threadIdx.x < kGuardFront ? pw + threadIdx.x : 2 * pw + threadIdx.x] = 0;
  __syncthreads();
}

// ------------------------------------------------------------------------------------------------
// Gathered column tiles (flag DAM_MASK_GATHER_COLUMNS). The mask is unchanged; its entries in query
// tiles of the pattern region are split into a diagonal part, listed in ordinary tiles, and a column
// part, listed in tiles whose 128 (tile_n) "keys" are matched columns taken in ascending order:
// gathered tile v of head h holds columns gidx[h][v tile_n ..], and row i keeps slot s iff
// c = gidx[s] <= i and i - c is not a matched diagonal (those entries belong to the diagonal part).
// A vertical stripe then costs its share of one dense tile per query tile instead of a whole tile.

// The matched columns below S of one head, ascending, padded with -1 up to the stride. One workgroup of 16 waves per
// head, a word of the column set per lane and pass; the words with more than two columns (sinks, the last columns of a
// capture) are then written by the whole wave, a lane per bit. (Bit by bit in the word's own lane, 64 dependent steps for a
// full word, this and the classes took 5.5 us of the prep kernel's 8 at 32 heads x 4096 tokens captured at 1024.)
__device__ __forceinline__ void gather_columns_of_head(const Geom &g, const uint64_t *__restrict__ cb,  // the head's column set
                                                       int stride, int h, int *__restrict__ gidx, int *__restrict__ gcnt) {
  __shared__ int s_wave[2][16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int *out = gidx + (int64_t)h * stride;
  const int n_cols = min(g.P, g.S), n_words = (n_cols + 63) / 64;
  int base = 0;  // the same value in every thread
  for (int w0 = 0, pass = 0; w0 < n_words; w0 += 1024, ++pass) {
    const int each = (min(n_words - w0, 1024) + 15) / 16;  // words per wave
    const int w = w0 + wave * each + lane;
    uint64_t m = lane < each && w < n_words ? cb[w] : 0;
    if (w * 64 + 64 > n_cols && w * 64 < n_cols) m &= ~0ull >> (64 - (n_cols - w * 64));
    const int v = __popcll(m), incl = wave_prefix(v);
    if (lane == 63) s_wave[pass & 1][wave] = incl;
    __syncthreads();  // one per pass: the totals of consecutive passes lie in alternating words
    const int totals = wave_prefix(lane < 16 ? s_wave[pass & 1][lane] : 0);
    const int before = base + (wave > 0 ? __builtin_amdgcn_readlane(totals, (wave - 1) & 15) : 0), at = before + incl - v;
    base += __builtin_amdgcn_readlane(totals, 15);
    if (v == 1 || v == 2) {
      out[at] = w * 64 + __ffsll((unsigned long long)m) - 1;
      if (v == 2) out[at + 1] = w * 64 + 63 - __clzll((long long)m);
    }
    for (uint64_t many = __ballot(v > 2); many; many &= many - 1) {
      const int from = __ffsll((unsigned long long)many) - 1;
      const unsigned lo = __builtin_amdgcn_readlane((int)m, from), hi = __builtin_amdgcn_readlane((int)(m >> 32), from);
      const int to = __builtin_amdgcn_readlane(at, from) + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
      if ((lane < 32 ? lo >> lane : hi >> (lane - 32)) & 1) out[to] = (w0 + wave * each + from) * 64 + lane;
    }
  }
  if (threadIdx.x == 0) gcnt[h] = base;
  // the empty slots: 16 bytes per store where the row allows it (rows are `stride` ints apart, a multiple of 64)
  const int first4 = (base + 3) & ~3;
  if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    if (base + (int)threadIdx.x < min(first4, stride)) out[base + threadIdx.x] = -1;
    for (int x = first4 + 4 * (int)threadIdx.x; x + 4 <= stride; x += 4 * blockDim.x)
      *reinterpret_cast<int4 *>(out + x) = make_int4(-1, -1, -1, -1);
    if ((int)threadIdx.x < (stride & 3)) out[(stride & ~3) + threadIdx.x] = -1;
  } else {
    for (int x = base + threadIdx.x; x < stride; x += blockDim.x) out[x] = -1;
  }
}

// a3 for short captures, inside the kernel that needs the flags: match counts of one head from its true bits, gamma >= mu,
// flags and bitsets, by the 16 waves of one workgroup. A job is one word (64 patterns) of one kind over one chunk of 64 rows:
// a lane per row, the 64 x 64 bits turned around, and a lane per pattern then counts its word. The jobs of the causal
// triangle go round the waves and add into LDS.
// In place of the launches that longer captures take (k_pattern_slices, and k_pattern_finish or sum_slices_of_head), which
// cost 5 us each however short they are. The jobs grow with the square of the capture and run on one CU per head, so the line
// lies where the gain ends; whole layers of 4000 tokens, the launches / this, us: 8 heads captured at 576 61.0 / 57.3, 768 61.5 / 60.0,
// 832 70.3 / 69.5, 1024 68.7 / 72.2; 32 heads 85.2 / 81.3, 93.3 / 91.2, 101.1 / 100.0, 105.4 / 108.6; 64 heads 131.3 / 127.2, 138.7 / 136.7,
// 157.2 / 155.1, 170.2 / 172.2. Patterns alone, where the launches are two and this is one: 1 head x 832 17.8 / 17.1, 96 x 832
// 57.9 / 56.1; 1 x 896 18.1 / 18.8, 32 x 896 30.4 / 31.6, 96 x 896 61.8 / 61.6.
constexpr int kDirectL = 832;
template <int MOST>
__device__ __forceinline__ void count_patterns_of_head(const Geom &g, const uint64_t *__restrict__ tb,  // the head's true bits
                                                       float mu, int h, int *cnt,                       // LDS [2][MOST]
                                                       int *__restrict__ vert_cnt, int *__restrict__ diag_cnt,
                                                       uint8_t *__restrict__ vert_flag, uint8_t *__restrict__ diag_flag,
                                                       uint64_t *__restrict__ cbits, uint64_t *__restrict__ rrev,
                                                       uint64_t *lds_copy) {  // both sets again, [2 pw], or nullptr
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  for (int x = threadIdx.x; x < 2 * MOST; x += blockDim.x) cnt[x] = 0;
  __syncthreads();
  const bool diag = wave & 1;
  int chunk = 0, w = wave >> 1;  // the pair (chunk, word <= chunk) of this wave; both kinds take every n_waves / 2-th
  auto settle = [&] {
    while (w > chunk) w -= ++chunk;
  };
  uint64_t hi = 0, lo = 0;
  auto fetch = [&] {
    const int i = 64 * chunk + lane, wj = diag ? chunk - w : w;
    const uint64_t *row = tb + (int64_t)min(i, g.L - 1) * g.tbw;
    hi = lo = 0;
    if (i < g.L) {
      hi = row[wj];
      if (diag && wj > 0) lo = row[wj - 1];
    }
  };
  settle();
  if (chunk < g.tbw) fetch();
  while (chunk < g.tbw) {  // wave-uniform
    // diagonals: the window of the row that ends at column i - 64 w, reversed: offset 64 w + t at bit t
    uint64_t x = hi;
    if (diag) x = __brevll(lane == 63 ? hi : (hi << (63 - lane)) | (lo >> (lane + 1)));
    const int at = (diag ? MOST : 0) + 64 * w + lane;
    w += n_waves / 2;
    settle();
    if (chunk < g.tbw) fetch();
    atomicAdd(&cnt[at], __popcll(transpose64(x, lane)));
  }
  __syncthreads();
  for (int x = wave; x < 2 * g.tbw; x += n_waves) {
    const int word = x >> 1, p = 64 * word + lane, n = cnt[(x & 1) * MOST + p];
    const bool hit = p < g.L && (float)n / (float)(g.L - p) >= mu;
    const uint64_t set = __ballot(hit);
    const int64_t e = (int64_t)h * g.L + p;
    if (p < g.L) {
      if (int *out = x & 1 ? diag_cnt : vert_cnt) out[e] = n;
      (x & 1 ? diag_flag : vert_flag)[e] = (uint8_t)hit;
    }
    if (lane == 0) {
      const int to = x & 1 ? g.pw - 1 - word : word;
      const uint64_t v = x & 1 ? __brevll(set) : set;
      (x & 1 ? rrev : cbits)[(int64_t)h * g.pw + to] = v;
      if (lds_copy) lds_copy[(x & 1 ? g.pw : 0) + to] = v;
    }
  }
}

// The same from the chunk counts of k_pattern_slices (kSlicesInPrep), a wave per word of patterns: a lane fetches one of the
// eight slices of one chunk, and the 64 x 64 bits of eight chunks turned around are, in the lane of a pattern, its eight
// counts, a byte each. Bound by one trip to memory per job, so the next job's slices are under way.
// Saves the launch of k_pattern_finish, but on one CU per head, so the line lies where the two meet. Whole builds of twice the
// captured length, the launch / this, us: 2 heads captured at 1792 42.6 / 42.8, 1984 60.3 / 61.1, 2048 44.5 / 45.3; 8 heads at 1600 57.8 /
// 57.5, 2048 52.1 / 52.9; 32 heads at 1600 86.5 / 86.2, 1792 83.3 / 83.2, 2048 97.3 / 98.1; 64 heads at 1600 132.0 / 131.6, 1792 137.2 /
// 136.8, 2048 176.5 / 177.1.
// (Each slice a wave-uniform load of its own / this, layers of 32 heads: 4096 tokens captured at 1024 111.9 / 108.4, 6000 at 1536
// 187.1 / 180.2.)
constexpr int kSlicesInPrep = 1792;
__device__ __forceinline__ void sum_slices_of_head(const Geom &g, const uint64_t *__restrict__ vslices, const uint64_t *__restrict__ dslices,
                                                   float mu, int h, int *__restrict__ vert_cnt, int *__restrict__ diag_cnt,
                                                   uint8_t *__restrict__ vert_flag, uint8_t *__restrict__ diag_flag,
                                                   uint64_t *__restrict__ cbits, uint64_t *__restrict__ rrev, uint64_t *lds_copy) {
  static_assert(kSlices == 8, "a count is a byte");
  constexpr int kEach = (kSlicesInPrep / kChunkRows + 7) / 8;  // fetches per lane and job
  const int lane = threadIdx.x & 63, n_waves = blockDim.x >> 6;
  const int n_chunks = (g.L + kChunkRows - 1) / kChunkRows;
  uint64_t next[kEach];
  // rows above pattern p hold nothing of it: start at the chunk of the word's first
  auto fetch = [&](int x) {
    const int word = x >> 1, from = word * 64 / kChunkRows;
    const uint64_t *slices = (x & 1 ? dslices : vslices) + ((int64_t)h * n_chunks * g.tbw + word) * kSlices + (lane & 7);
#pragma unroll
    for (int u = 0; u < kEach; ++u) {
      const int chunk = from + 8 * u + (lane >> 3);
      next[u] = 0;
      if (from + 8 * u < n_chunks) {  // wave-uniform
        const uint64_t v = slices[(int64_t)min(chunk, n_chunks - 1) * g.tbw * kSlices];
        next[u] = chunk < n_chunks ? v : 0;
      }
    }
  };
  int x = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (x < 2 * g.tbw) fetch(x);
  for (; x < 2 * g.tbw; x += n_waves) {
    uint64_t w[kEach];
#pragma unroll
    for (int u = 0; u < kEach; ++u) w[u] = next[u];
    if (x + n_waves < 2 * g.tbw) fetch(x + n_waves);
    const int word = x >> 1, p = 64 * word + lane;
    int n = 0;
#pragma unroll
    for (int u = 0; u < kEach; ++u)
      if (word * 64 / kChunkRows + 8 * u < n_chunks) {  // wave-uniform
        const uint64_t counts = transpose64(w[u], lane);
        n = __builtin_amdgcn_udot4((unsigned)counts, 0x01010101u, n, false);
        n = __builtin_amdgcn_udot4((unsigned)(counts >> 32), 0x01010101u, n, false);
      }
    const bool hit = p < g.L && (float)n / (float)(g.L - p) >= mu;
    const uint64_t set = __ballot(hit);
    const int64_t e = (int64_t)h * g.L + p;
    if (p < g.L) {
      if (int *out = x & 1 ? diag_cnt : vert_cnt) out[e] = n;
      (x & 1 ? diag_flag : vert_flag)[e] = (uint8_t)hit;
    }
    if (lane == 0) {
      const int to = x & 1 ? g.pw - 1 - word : word;
      const uint64_t v = x & 1 ? __brevll(set) : set;
      (x & 1 ? rrev : cbits)[(int64_t)h * g.pw + to] = v;
      if (lds_copy) lds_copy[(x & 1 ? g.pw : 0) + to] = v;
    }
  }
}

// Row bitmap of one gathered slot for the rows of query tile qt: bit r of word k is row 64 k + r of the
// tile. c < 0: an empty slot.
__device__ __forceinline__ void slot_rows(const Geom &g, const uint64_t *__restrict__ rr, int i0, int c,
                                          uint64_t (&keep)[4]) {
  const int row_words = g.tile_m / 64;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    keep[k] = 0;
    if (k < row_words && c >= 0) {
      const int r0 = 64 * k;                       // first row of the word
      const int first = c - i0 - r0;               // rows of the word from `first` on are causal
      uint64_t m = first <= 0 ? ~0ull : (first >= 64 ? 0ull : ~0ull << first);
      const int live = g.S - i0 - r0;              // rows of the word below `live` exist
      m &= live >= 64 ? ~0ull : (live <= 0 ? 0ull : ~0ull >> (64 - live));
      // offsets i - c of the word's rows, highest first, are 64 consecutive bits of the reversed set
      const uint64_t diag = __brevll(diag_window(rr, g.pw, (int64_t)i0 + r0 + 63 - c));
      keep[k] = m & ~diag;
    }
  }
}

// The largest tile distance with a matched offset, 0 if there is none: the first set bit of the head's reversed class words.
// By a whole wave.
__device__ __forceinline__ int64_t farthest_tile(const uint64_t *__restrict__ off_any_h, int occw, int lane) {
  for (int w0 = 0; w0 < occw; w0 += 64) {
    const uint64_t word = w0 + lane < occw ? off_any_h[w0 + lane] : 0;
    const uint64_t nz = __ballot(word != 0);
    if (nz) {
      const int wl = __ffsll((unsigned long long)nz) - 1;
      const unsigned hi = __builtin_amdgcn_readlane((int)(word >> 32), wl), lo = __builtin_amdgcn_readlane((int)word, wl);
      return (int64_t)(occw - w0 - wl) * 64 - __ffsll((unsigned long long)((uint64_t)hi << 32 | lo));
    }
  }
  return 0;
}

// Pass 1 of the block index: which key tiles of query tile (h, qt) hold a kept entry / are full.
// One wave per query tile, 64 key tiles (one occupancy word) at a time, one lane per key tile. Tiles
// strictly below the diagonal and outside the true-mask block are decided by their lane alone (from
// the class bitsets, or from its first and last row), and so is the diagonal tile of a query tile that lies wholly in the pattern
// region (square tiles); the other tiles on the diagonal and those inside the true-mask block are then evaluated word by word
// by the whole wave. No LDS, no barrier.
// (What a row needs of the gathered columns, fetched in front of everything else: a load issued behind the stores below waits for
// them. The first 64 gathered tiles' first and last columns; slots past the count hold -1.)
struct RowColumns {
  int n_cols, first, last;
};
__device__ __forceinline__ RowColumns fetch_columns(const Geom &g, const int *__restrict__ gidx, const int *__restrict__ gcnt, int gstride,
                                                    int h, int qt, int lane) {
  RowColumns c{0, -1, -1};
  if (gidx != nullptr && qt * g.tile_m >= g.L) {
    const int *gi = gidx + (int64_t)h * gstride;
    c.n_cols = gcnt[h];
    if ((lane + 1) * g.tile_n <= gstride) {
      c.first = gi[lane * g.tile_n];
      c.last = gi[lane * g.tile_n + g.tile_n - 1];
    }
  }
  return c;
}
// TRUE_BLOCK: there is a true-mask block (L > 0). SQUARE: tile_m == tile_n, so that there are classes; tiles of other shapes are a
// form of their own, which leaves the square ones' code as it was (with what they need in one form, and with the test of the two
// widths left out, the compiler's choice of registers cost layers of 4096 tokens up to 0.5 %).
template <bool TRUE_BLOCK, bool SQUARE>
__device__ __forceinline__ int tile_scan_row(const Geom &g, const uint64_t *__restrict__ tb, const uint64_t *__restrict__ cb,
                                              const uint64_t *__restrict__ rr, const uint64_t *__restrict__ classes,  // of the head
                                              uint64_t *__restrict__ occ,
                                              uint64_t *__restrict__ full, int *__restrict__ cnt, const int *__restrict__ gidx,
                                              const RowColumns &columns, int gstride, uint64_t *__restrict__ vocc,
                                              uint64_t *__restrict__ vfull, int h, int qt, int lane) {
  const int i0 = qt * g.tile_m;
  const int i_last = min(g.S - 1, i0 + g.tile_m - 1);
  const int kmax = i_last / g.tile_n;
  // Square tiles, a whole row of tiles in the pattern region: 64 tiles at a time from the per-head
  // class bitsets. Only a tile that has matched and unmatched columns AND matched and unmatched
  // offsets needs the exact one-lane test for "full".
  const bool by_class = SQUARE && g.tile_m == g.tile_n && i0 >= g.L && i0 + g.tile_m <= g.S;
  // gathered columns: in a query tile of the pattern region the ordinary tiles hold the diagonal part only
  const bool split = gidx != nullptr && i0 >= g.L;
  const int n_cols = columns.n_cols, g_first = columns.first, g_last = columns.last;
  const int *gi = split ? gidx + (int64_t)h * gstride : nullptr;
  const uint64_t *cbw = split ? nullptr : cb;
  const uint64_t *ca = classes + kColAny * g.occw, *cf = classes + kColAll * g.occw;
  const uint64_t *da = classes + kOffAny * g.occw, *df = classes + kOffAll * g.occw;
  const int words = g.tile_m * g.wpr;
  const bool inner = TRUE_BLOCK && i0 + g.tile_m <= min(g.L, g.S) && words <= 256;  // (words: 64 per lane and step, 4 steps)
  // This lane's words of a tile, divided by a multiplication (four divisions by a variable cost every wave of the launch
  // about a microsecond, also where it looks at no tile of the true-mask block): a row has 1 to 4 words, x is below 256.
  const int inv_wpr = g.wpr == 1 ? 65537 : g.wpr == 2 ? 32769 : g.wpr == 3 ? 21846 : 16385;
  int word_row[4], word_col[4];
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    word_row[y] = ((lane + 64 * y) * inv_wpr) >> 16;
    word_col[y] = lane + 64 * y - word_row[y] * g.wpr;
  }
  // Occupancy words whose 64 tiles all lie further above the query tile than any matched diagonal reaches, and hold no
  // matched column (or leave those to the gathered tiles), are empty: a lane per word finds that out, and the walk, whose
  // steps wait for memory one after the other, takes the other words only. (64 heads x 128k tokens, captured at 4096, 16 words
  // a row at most: scan 281 -> 226 us; with the diagonal and the incomplete gathered tile decided by bounds, 191.) From two
  // words in front of the diagonal's on, or where the gathered tiles want the bound anyway: below that it saves nothing.
  const int n_words = (kmax >> 6) + 1;
  const int64_t dmax = by_class && (n_words > 2 || split) ? farthest_tile(da, g.occw, lane) : INT64_MAX;
  int total = 0;
  for (int wb = 0; wb < n_words; wb += 64) {  // (the words past the diagonal tile's are neither written nor read)
    const int mine = wb + lane;
    const bool empty = dmax != INT64_MAX && mine < n_words && qt - (mine * 64 + 63) > dmax && (split || ca[mine] == 0);
    if (empty) {
      occ[((int64_t)h * g.nQt + qt) * g.occw + mine] = 0;
      full[((int64_t)h * g.nQt + qt) * g.occw + mine] = 0;
    }
    uint64_t todo = __ballot(mine < n_words && !empty);
    // (from a line of the instruction cache on, as the words' loop below, whatever code stands in front: 64 heads x 8192 tokens
    // captured at 4096 scan 46.8 us, 48.3 from elsewhere in a line)
    asm volatile(".p2align 6" ::: "memory");
    while (todo) {
      const int w = wb + __ffsll((unsigned long long)todo) - 1;
      todo &= todo - 1;
      const int kt = w * 64 + lane;
      int f = 0;
      if (kt <= kmax) {
        const int j0 = kt * g.tile_n, j1 = min(j0 + g.tile_n - 1, g.S - 1);
        f = 4;  // evaluate word by word
        if (i0 >= g.L && j1 <= i0) {
          bool exact = true;
          if (by_class) {
            const int d = qt - kt;  // >= 1 here
            const int64_t pos = (int64_t)g.occw * 64 - 1 - d;
            const bool c_any = !split && ((ca[w] >> lane) & 1), c_all = !split && ((cf[w] >> lane) & 1);
            const bool d_any = (da[pos >> 6] >> (pos & 63)) & 1, d_all = (df[pos >> 6] >> (pos & 63)) & 1;
            if (!(c_any && !c_all && d_any && !d_all)) {
              exact = false;
              f = ((c_any || d_any) ? 1 : 0) | ((c_all || d_all) ? 3 : 0);
            }
          }
          if (exact) {
            f = pattern_tile_any(cbw, rr, g.pw, i0, i_last, j0, j1) ? 1 : 0;
            // Full only if its first and its last row are, which few are: those are evaluated by the whole wave. (A tile cut
            // by the end of the sequence never is, its bits past S are zero.) A lane that went through the unmatched offsets
            // itself, each with the columns it meets, held the wave for as long as the longest took: 6 heads x 1000 tokens,
            // captured at 256, in the plain layout, whole layer 50.9 -> 36.5 us; builds of 32 heads of patterns there, 1024 tokens 29.7 ->
            // 14.3, 8000 57.4 -> 36.5, 32768 140 -> 121.
            // Tiles that are not square have no classes: those of matched columns or offsets alone, all of a dense mask and of a
            // window, are looked for here, and tall ones are asked for the last row of every tile_n (an unmatched offset meets
            // one of those or the first). Builds of 32 heads with windows of 4096 at 32768 tokens, 64 x 128 / 128 x 64 / 256 x 128
            // tiles, 200 / 205 / 204 us with their full tiles evaluated by the whole wave, 69 / 64 / 56 so.
            if constexpr (SQUARE) {
              if (f && j0 + g.tile_n <= g.S && i0 + g.tile_m <= g.S && pattern_row_full(cbw, rr, g.pw, i0, kt * g.wpr, g.wpr) &&
                  pattern_row_full(cbw, rr, g.pw, i_last, kt * g.wpr, g.wpr))
                f = 4;
            } else if (f && j0 + g.tile_n <= g.S && i0 + g.tile_m <= g.S) {
              if (pattern_tile_all(g, cbw, rr, i0, kt * g.wpr)) f = 3;
              else f = 4;
              for (int i = i0; f == 4; i = i == i0 ? i0 + min(g.tile_m, g.tile_n) - 1 : min(i + g.tile_n, i_last)) {
                if (!pattern_row_full(cbw, rr, g.pw, i, kt * g.wpr, g.wpr)) f = 1;
                if (i == i_last) break;
              }
            }
          }
        } else if (by_class && kt == qt) {
          // the diagonal tile of a row of the pattern region, never full: it meets the offsets 0 .. T - 1, each in its last
          // row too, and a matched column at least in the column's own row
          const int64_t Q = (int64_t)g.pw * 64 - 1;
          f = range_any(rr, g.pw, Q - (g.tile_n - 1), Q) || (!split && ((ca[w] >> lane) & 1)) ? 1 : 0;
        }
      }
      uint64_t ow = __ballot(f & 1), fw = __ballot(f & 2);
      uint64_t need = __ballot(f & 4);
      // A query tile inside the true-mask block: four tiles' words are fetched before the first is looked at (a word is one
      // load from global memory; one tile after the other made a row of eight tiles wait eight times, and set the time of
      // the launch: 32 heads x 4096 tokens, captured at 1024, whole build 73.7 -> 69.6 us).
      while (inner && need) {  // wave-uniform
        int b[4];
        uint64_t m[4][4];
  #pragma unroll
        for (int u = 0; u < 4; ++u) {
          b[u] = need ? __ffsll((unsigned long long)need) - 1 : b[u > 0 ? u - 1 : 0];  // (the last of them again)
          need &= need - 1;
  #pragma unroll
          for (int y = 0; y < 4; ++y) {
            if (64 * y >= words) break;
            m[u][y] = tb[(int64_t)(i0 + word_row[y]) * g.tbw + min((w * 64 + b[u]) * g.wpr + word_col[y], g.tbw - 1)];
          }
        }
  #pragma unroll
        for (int u = 0; u < 4; ++u) {
          bool any = false, all = true;
  #pragma unroll
          for (int y = 0; y < 4; ++y) {
            if (64 * y >= words) break;
            const int wj = (w * 64 + b[u]) * g.wpr + word_col[y];
            const uint64_t x = m[u][y] & in_true_block(g, i0 + word_row[y], wj);
            any |= x != 0;
            all &= x == ~0ull;
          }
          if (__ballot(any) != 0) ow |= 1ull << b[u];
          if (__ballot(!all) == 0) fw |= 1ull << b[u];
        }
      }
      while (need) {  // wave-uniform
        const int b = __ffsll((unsigned long long)need) - 1;
        need &= need - 1;
        bool any = false, all = true;
        asm volatile(".p2align 6" ::: "memory");
        for (int x = lane; x < words; x += 64) {
          const uint64_t m = mask_word(g, tb, cbw, rr, i0 + x / g.wpr, (w * 64 + b) * g.wpr + x % g.wpr);
          any |= m != 0;
          all &= m == ~0ull;
          // (listed and not full, which the first words mostly tell: wave-uniform. 32 heads x 4096 tokens, 256 x 128 tiles with an
          // unmatched offset here and there 45.2 -> 38.6 us. Of square tiles few come here: 2 heads x 454 tokens, 64 x 64 tiles,
          // captured at 224, whole layer 28.1 us without it, 28.4 with.)
          if (!SQUARE && __ballot(any) != 0 && __ballot(!all) != 0) break;
        }
        if (__ballot(any) != 0) ow |= 1ull << b;
        if (__ballot(!all) == 0) fw |= 1ull << b;
      }
      if (lane == 0) {
        occ[((int64_t)h * g.nQt + qt) * g.occw + w] = ow;
        full[((int64_t)h * g.nQt + qt) * g.occw + w] = fw;
      }
      total += __popcll(ow);
    }
  }
  if (gidx) {
    // the gathered tiles of this query tile: one lane per slot, the rows of the tile as a bitmap
    const int n_gt = (n_cols + g.tile_n - 1) / g.tile_n;
    const int row_words = g.tile_m / 64;
    // No matched diagonal lies beyond r_bound: the largest tile distance with a matched offset covers offsets up to
    // T d + T - 1. (Square tiles only: the classes are theirs.)
    const int64_t r_bound = dmax != INT64_MAX ? dmax * g.tile_n + g.tile_n - 1 : INT64_MAX;
    for (int w = 0; w * 64 < n_gt; ++w) {  // (only the words that hold a gathered tile are written, and read)
      // A gathered tile whose columns all lie further above this query tile than any matched diagonal reaches keeps
      // every row of every filled slot: every row is causal for it and no offset i - c is a matched one. It is full
      // if it is complete. A tile whose first column lies below the query tile's last row holds nothing (its columns
      // ascend). One lane per tile; the other tiles are evaluated slot by slot.
      bool certain = false, nothing = false, complete = false;
      {
        const int v = w * 64 + lane;
        if (v < n_gt) {
          nothing = (w == 0 ? g_first : gi[v * g.tile_n]) > i_last;
          complete = (v + 1) * g.tile_n <= n_cols;
          if (r_bound != INT64_MAX) {
            const int cmax = w == 0 && complete ? g_last : gi[min((v + 1) * g.tile_n, n_cols) - 1];
            certain = (int64_t)i0 - cmax > r_bound;
          }
        }
      }
      const uint64_t sure = __ballot(certain), skip = sure | __ballot(nothing);
      uint64_t ow = sure, fw = __ballot(certain && complete);
      for (int v = w * 64; v < min(n_gt, w * 64 + 64); ++v) {
        if ((skip >> (v & 63)) & 1) continue;  // wave-uniform
        bool any = false, all = true;
        for (int wg = 0; wg < g.wpr; ++wg) {
          const int c = gi[v * g.tile_n + wg * 64 + lane];
          uint64_t keep[4];
          slot_rows(g, rr, i0, c, keep);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (k < row_words) {
              any |= keep[k] != 0;
              all &= keep[k] == ~0ull;
            }
        }
        if (__ballot(any) != 0) ow |= 1ull << (v & 63);
        if (__ballot(!all) == 0) fw |= 1ull << (v & 63);
      }
      if (lane == 0) {
        vocc[((int64_t)h * g.nQt + qt) * g.occw + w] = ow;
        vfull[((int64_t)h * g.nQt + qt) * g.occw + w] = fw;
      }
      total += __popcll(ow);
    }
  }
  if (lane == 0) cnt[(int64_t)h * g.nQt + qt] = total;
  return total;
}

// Everything the block index needs from the pattern flags of one head, in one launch (one workgroup of 1024
// per head: the three steps are short chains of dependent work, and as separate kernels each paid a launch):
// the two bitsets, the tile classes, the gathered column list.
// SOURCE says where the flags come from: they are given; the patterns are counted here, from the true mask, or from the
// attention map itself, whose true mask is made first; or the chunks' counts are added up. (A kernel for each, because their LDS
// arrays differ, up to 6.5 KiB; all hold the registers of the scan, 126 or 127.)
enum PrepSource { kFlagsGiven, kFromTrueBits, kFromMap, kFromSlices };
struct CountArgs {
  PrepSource source = kFlagsGiven;
  const float *map = nullptr;  // kFromMap, with its threshold
  Threshold thr{};
  uint64_t *true_bits = nullptr;
  const uint64_t *vslices = nullptr, *dslices = nullptr;
  float mu = 0.0f;
  int *vert_cnt = nullptr, *diag_cnt = nullptr;
  uint8_t *vert_flag = nullptr, *diag_flag = nullptr;
};

// a2 of one short map by the 16 waves of its workgroup: a lane per key and a ballot per word, every word up to the diagonal
// under way at once, into LDS (which the counts and the scan read) and from there, with the zero words above the diagonal, to
// memory as whole lines. In place of a launch of k_true_mask_rows. The map is read by one CU per head, so the line is low; whole
// layers, launch / this, us: 2 fp32 heads x 256 tokens captured at 64 22.2 / 19.7, 8 x 400 at 128 25.7 / 23.9, 8 x 600 at 192 34.8 /
// 35.5, 6 x 1000 at 256 34.1 / 37.6 (64 x 2000 at 256 66.0 / 63.3).
constexpr int kMapInPrep = 128;
__device__ __forceinline__ void true_mask_of_head(const Geom &g, const float *__restrict__ map, unsigned theta, uint64_t *words,  // LDS
                                                  uint64_t *__restrict__ true_bits) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kWords = kMapInPrep / 64;
  float v[kWords][4 * kWords];
  // word w of rows 64 w + wave + 16 k
  auto each = [&](auto f) {
#pragma unroll
    for (int w = 0; w < kWords; ++w)
#pragma unroll
      for (int k = 0; k < 4 * (kWords - w); ++k)
        if (64 * w + wave + 16 * k < g.L) f(w, k, 64 * w + wave + 16 * k, 64 * w + lane);  // wave-uniform
  };
  each([&](int w, int k, int i, int j) { v[w][k] = map[(int64_t)i * g.L + min(j, i)]; });
  each([&](int w, int k, int i, int j) {
    const float x = v[w][k] != v[w][k] ? -INFINITY : v[w][k];
    const uint64_t word = __ballot(j <= i && key_of(x) >= theta);
    if (lane == 0) words[i * g.tbw + w] = word;
  });
  __syncthreads();
  for (int x = threadIdx.x; x < g.L * g.tbw; x += blockDim.x) {
    const int i = x / g.tbw, w = x - i * g.tbw;
    const uint64_t word = 64 * w <= i ? words[x] : 0;
    if (64 * w > i) words[x] = 0;  // (the scan reads them)
    true_bits[x] = word;
  }
}
// scan.on: and pass 1 of the block index (tile_scan_row, below as a kernel of its own), a wave per query tile, which saves that
// launch where the query tiles of a head are few (see scans_in_prep).
struct ScanArgs {
  bool on;
  uint64_t *occ, *full, *vocc, *vfull;
  int *cnt;
  const uint64_t *true_bits;
};
template <PrepSource SOURCE, bool SQUARE>  // (SQUARE: of tile_scan_row)
__global__ __launch_bounds__(1024) void k_pattern_prep(Geom g, CountArgs ca, ScanArgs scan, const uint8_t *__restrict__ diag_flag,
                                                       const uint8_t *__restrict__ vert_flag, uint64_t *__restrict__ cbits,
                                                       uint64_t *__restrict__ rrev, bool want_classes, uint64_t *__restrict__ classes,
                                                       int gstride, int *__restrict__ gidx, int *__restrict__ gcnt,
                                                       int *__restrict__ head_cnt, bool in_lds) {
  extern __shared__ uint64_t prep_sets[];  // in_lds: the head's two sets, [2 pw], and its class words, [4 occw]
  const int h = blockIdx.x;
  if (threadIdx.x < kHeadSub) head_cnt[h * kHeadSub + threadIdx.x] = 0;  // the head's number of listed tiles: summed by k_tile_scan
  uint64_t *copy = in_lds && want_classes ? prep_sets : nullptr;
  __shared__ int cnt[SOURCE == kFromTrueBits ? 2 * kDirectL : SOURCE == kFromMap ? 2 * kMapInPrep : 1];
  __shared__ uint64_t true_words[SOURCE == kFromMap ? kMapInPrep * kMapInPrep / 64 : 1];
  if constexpr (SOURCE == kFromTrueBits) {
    count_patterns_of_head<kDirectL>(g, ca.true_bits + (int64_t)h * g.L * g.tbw, ca.mu, h, cnt, ca.vert_cnt, ca.diag_cnt, ca.vert_flag,
                                     ca.diag_flag, cbits, rrev, copy);
  } else if constexpr (SOURCE == kFromMap) {
    true_mask_of_head(g, ca.map + (int64_t)h * g.L * g.L, take_threshold(ca.thr), true_words, ca.true_bits + (int64_t)h * g.L * g.tbw);
    __syncthreads();
    count_patterns_of_head<kMapInPrep>(g, true_words, ca.mu, h, cnt, ca.vert_cnt, ca.diag_cnt, ca.vert_flag, ca.diag_flag, cbits, rrev, copy);
  } else if constexpr (SOURCE == kFromSlices) {
    sum_slices_of_head(g, ca.vslices, ca.dslices, ca.mu, h, ca.vert_cnt, ca.diag_cnt, ca.vert_flag, ca.diag_flag, cbits, rrev, copy);
  } else {
    pattern_bitsets_of_head(diag_flag, vert_flag, g.P, g.pw, h, cbits, rrev, copy);
  }
  if (!want_classes) return;  // uniform over the grid
  __syncthreads();       // the sets are read back by other threads of this workgroup
  // (from the LDS copy when they fit: the steps below are chains of dependent reads. One call per address space,
  // so that the compiler knows which kind of read to use.)
  uint64_t *classes_h = classes + (int64_t)h * 4 * g.occw;
  if (in_lds) {
    tile_classes_of_head(g, prep_sets, prep_sets + g.pw, classes_h, prep_sets + 2 * g.pw);
    if (gidx) gather_columns_of_head(g, prep_sets, gstride, h, gidx, gcnt);
  } else {
    tile_classes_of_head(g, cbits + (int64_t)h * g.pw, rrev + (int64_t)h * g.pw, classes_h, nullptr);
    if (gidx) gather_columns_of_head(g, cbits + (int64_t)h * g.pw, gstride, h, gidx, gcnt);
  }
  if (!scan.on) return;  // uniform over the grid
  __syncthreads();  // classes and columns are read back by other threads of this workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t *tb = SOURCE == kFromMap ? true_words : scan.true_bits ? scan.true_bits + (int64_t)h * g.L * g.tbw : nullptr;
  int mine = 0;
  for (int qt = wave; qt < g.nQt; qt += blockDim.x >> 6)
    mine += tile_scan_row<true, SQUARE>(g, tb, prep_sets, prep_sets + g.pw, prep_sets + 2 * g.pw, scan.occ, scan.full, scan.cnt, gidx,
                          fetch_columns(g, gidx, gcnt, gstride, h, qt, lane), gstride, scan.vocc, scan.vfull, h, qt, lane);
  if (lane == 0) head_cnt[h * kHeadSub + wave] = mine;
}

// Exclusive scan of n counts by one block. group > 0: the result is laid out as [n / group]
// rows of group + 1 offsets (row r ends where row r + 1 begins); group == 0: plain [n + 1].
// Offsets are written as min(offset, clamp): with clamp = the capacity of the buffers the offsets point
// into, an index that does not fit is truncated to its first `capacity` entries and stays consistent
// with what the fill kernels wrote; *total is the unclamped sum.
// Every thread takes kScanItems consecutive counts per pass, so that the block-wide part (a wave
// scan, one exchange of the wave totals) is paid once per 8192 counts.
constexpr int kScanItems = 8;

// The scan itself, run by every thread of one workgroup of THREADS threads (a multiple of 64, at most 1024).
template <int THREADS>
__device__ __forceinline__ void block_exclusive_scan(const int *__restrict__ cnt, int64_t n, int group, int *__restrict__ ptr,
                                                     int64_t *__restrict__ total, int64_t clamp) {
  __shared__ int64_t wave_sum[2][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t carry = 0;  // the same value in every thread
  int pass = 0;
  for (int64_t base = 0; base < n; base += THREADS * kScanItems, ++pass) {
    const int64_t e0 = base + (int64_t)threadIdx.x * kScanItems;
    int v[kScanItems];
#pragma unroll
    for (int x = 0; x < kScanItems; ++x) v[x] = e0 + x < n ? cnt[e0 + x] : 0;
    int64_t mine = 0;
#pragma unroll
    for (int x = 0; x < kScanItems; ++x) mine += v[x];
    int64_t incl = mine;
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t up = __shfl_up(incl, off);
      if (lane >= off) incl += up;
    }
    if (lane == 63) wave_sum[pass & 1][wave] = incl;
    __syncthreads();  // one barrier per pass: the totals of consecutive passes live in alternating buffers
    int64_t before = carry, all = 0;
    for (int w = 0; w < THREADS / 64; ++w) {
      const int64_t ws = wave_sum[pass & 1][w];
      if (w < wave) before += ws;
      all += ws;
    }
    int64_t excl = before + incl - mine;
    int64_t r = 0;
    int q = 0;
#pragma unroll
    for (int x = 0; x < kScanItems; ++x) {
      const int64_t e = e0 + x;
      if (e < n) {
        if (group > 0) {
          // row and position of count e: divided once per thread and pass (x == 0), stepped after that
          if (x == 0) {
            r = e / group;
            q = (int)(e - r * group);
          }
          ptr[r * (group + 1) + q] = (int)min(excl, clamp);
          if (q == 0 && r > 0) ptr[(r - 1) * (group + 1) + group] = (int)min(excl, clamp);
          if (++q == group) {
            q = 0;
            ++r;
          }
        } else {
          ptr[e] = (int)min(excl, clamp);
        }
      }
      excl += v[x];
    }
    carry += all;
  }
  if (threadIdx.x == 0) {
    if (group > 0) {
      if (n > 0) ptr[(n / group - 1) * (group + 1) + group] = (int)min(carry, clamp);
    } else {
      ptr[n] = (int)min(carry, clamp);
    }
    if (total) *total = carry;
  }
}

__global__ __launch_bounds__(1024) void k_exclusive_scan(const int *__restrict__ cnt, int64_t n,
                                                         int group, int *__restrict__ ptr,
                                                         int64_t *__restrict__ total, int64_t clamp) {
  block_exclusive_scan<1024>(cnt, n, group, ptr, total, clamp);
}

// This workgroup's turn among the query tiles, `each` of a head at a time (dam_turns.h).
__device__ __forceinline__ QueryTiles my_query_tiles(const Geom &g, int each, bool by_heads) {
  const int n = (g.nQt + each - 1) / each, rows = each * g.tile_m;
  const int inside = g.L > 0 ? min(n, (min(g.L, g.S) + rows - 1) / rows) : 0;
  return query_tiles_of(g.H, n, inside, blockIdx.y * kGridRow + blockIdx.x, by_heads);  // (a second row follows a full one)
}

// Pass 1 as a kernel: a wave per query tile; the workgroup adds its four counts to the head's total. The CSR offsets
// need no launch of their own: every wave of the fill kernel adds up the totals of the heads before its own and the
// counts of the query tiles before its own. (Folding a scan into the last workgroup to finish was measured and
// dropped: it needs a device-wide release fence in every workgroup, which on this chip writes back the L2 of its
// XCD each time: 20 -> 190 us at S = 32768.)
template <bool TRUE_BLOCK, bool STAGED, bool SQUARE>
__global__ __launch_bounds__(256) void k_tile_scan(Geom g, const uint64_t *__restrict__ true_bits,
                                                   const uint64_t *__restrict__ cbits,
                                                   const uint64_t *__restrict__ rrev,
                                                   const uint64_t *__restrict__ classes,
                                                   uint64_t *__restrict__ occ,
                                                   uint64_t *__restrict__ full, int *__restrict__ cnt,
                                                   const int *__restrict__ gidx, const int *__restrict__ gcnt,
                                                   int gstride, uint64_t *__restrict__ vocc,
                                                   uint64_t *__restrict__ vfull, int *__restrict__ head_cnt) {
  extern __shared__ uint64_t lds_sets[];
  __shared__ int wave_cnt[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const QueryTiles my = my_query_tiles(g, 4, false);
  const int h = my.h, qt = my.at * 4 + wave;
  const uint64_t *tb = true_bits ? true_bits + (int64_t)h * g.L * g.tbw : nullptr;
  const uint64_t *cb = cbits + (int64_t)h * g.pw;
  const uint64_t *rr = rrev + (int64_t)h * g.pw;
  const uint64_t *classes_h = classes + (int64_t)h * 4 * g.occw;
  int mine = 0;
  const RowColumns columns = fetch_columns(g, gidx, gcnt, gstride, h, min(qt, g.nQt - 1), lane);
  if constexpr (STAGED) {
    stage_sets(lds_sets, g.pw, cb, rr, classes_h, 4 * g.occw);
    if (qt < g.nQt)
      mine = tile_scan_row<TRUE_BLOCK, SQUARE>(g, tb, lds_sets, lds_sets + g.pw + kGuardFront, lds_sets + 2 * g.pw + kGuardFront + kGuardBack, occ, full, cnt,
                           gidx, columns, gstride, vocc, vfull, h, qt, lane);
  } else if (qt < g.nQt) {
    mine = tile_scan_row<TRUE_BLOCK, SQUARE>(g, tb, cb, rr, classes_h, occ, full, cnt, gidx, columns, gstride, vocc, vfull, h, qt, lane);
  }
  // the head's total, for the offsets that the fill kernel derives itself (plain atomics, read by the next kernel
  // only; spread over kHeadSub words per head, because atomics on one address are served one after the other)
  if (lane == 0) wave_cnt[wave] = mine;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // (not the library's barrier, which waits for the stores above)
  if (threadIdx.x == 0)
    atomicAdd(head_cnt + h * kHeadSub + (my.at & (kHeadSub - 1)), wave_cnt[0] + wave_cnt[1] + wave_cnt[2] + wave_cnt[3]);
}

// Pass 2: write column, kind and the tile's element bits for every listed tile (below capacity). A wave per
// query tile (the four of a workgroup belong to one head and share its staged sets): the wave walks its own row
// of the index and writes every listed tile itself, a lane per tile row. With few query tiles in all (share = 4) the
// four waves of a workgroup share one query tile instead, each walking the whole row and taking every fourth
// tile: more waves, but the walk is then three quarters of the instructions.
// STAGED: the head's pattern sets are staged in LDS (they fit), or read from global memory. PATTERNS: tiles of 128 x 128 and no
// true-mask block, known to the compiler: 80 registers and none spilled instead of 96 and 68 scalar ones, and the last row of
// tiles of a ragged length goes the way of the others. Builds of 32 heads in the gathered layout 57.3 -> 51.0 us at 32768 tokens, 46.0 ->
// 33.1 at 12345.
template <bool STAGED, bool PATTERNS>
__global__ __launch_bounds__(256) void k_tile_fill(Geom g, const uint64_t *__restrict__ true_bits,
                                                   const uint64_t *__restrict__ cbits,
                                                   const uint64_t *__restrict__ rrev,
                                                   const uint64_t *__restrict__ occ,
                                                   const uint64_t *__restrict__ full,
                                                   const int *__restrict__ tile_cnt, const int *__restrict__ head_cnt,
                                                   int *__restrict__ row_ptr, int64_t *__restrict__ blk_total,
                                                   int *__restrict__ blk_col,
                                                   uint8_t *__restrict__ blk_kind,
                                                   uint64_t *__restrict__ tile_bits, int64_t capacity,
                                                   bool skip_full_bits,
                                                   const int *__restrict__ gidx, const int *__restrict__ gcnt,
                                                   int gstride, const uint64_t *__restrict__ vocc,
                                                   const uint64_t *__restrict__ vfull, const uint64_t *__restrict__ classes,
                                                   int share) {
  extern __shared__ uint64_t lds_sets[];
  const int tile_m = PATTERNS ? 128 : g.tile_m, tile_n = PATTERNS ? 128 : g.tile_n, wpr = PATTERNS ? 2 : g.wpr, L = PATTERNS ? 0 : g.L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const QueryTiles my = my_query_tiles(g, share == 4 ? 1 : 4, true);
  const int h = my.h;
  const int my_qt = share == 4 ? my.at : my.at * 4 + wave, my_turn = share == 4 ? wave : 0;
  const bool live = my_qt < g.nQt;
  const int qt = live ? my_qt : g.nQt - 1;  // (a spare wave reads a valid row and writes nothing)
  const uint64_t *tb = !PATTERNS && true_bits ? true_bits + (int64_t)h * L * g.tbw : nullptr;
  const uint64_t *cb = cbits + (int64_t)h * g.pw;
  const uint64_t *rr = rrev + (int64_t)h * g.pw;
  const uint64_t *oc = occ + ((int64_t)h * g.nQt + qt) * g.occw;
  const uint64_t *fl = full + ((int64_t)h * g.nQt + qt) * g.occw;
  const int i_last = min(g.S - 1, qt * tile_m + tile_m - 1);
  const int kmax = i_last / tile_n, n_words = (kmax >> 6) + 1;
  // where this query tile's entries start: the listed tiles of the heads before h and of the query tiles before
  // qt (no scan kernel between the two passes: the counts are few enough for every wave to add up its own prefix)
  int64_t part = 0;
  // (Both as one list, dealt out over the workgroup's waves, which share all of it but the query tiles of the workgroup itself; a
  // wave's loads travel together, places past the end repeated and left out. Each wave by itself, in batches of eight, four and
  // one and list by list, the waits were up to nine, at 32 heads x 32 query tiles 2.6 us of the kernel's 11.)
  __shared__ int64_t s_before[4];
  const int each = share == 4 ? 1 : 4, at0 = my.at * each;  // the workgroup's first query tile
  const int n_head = h * kHeadSub, n_before = n_head + at0;
  const int *cnt_h = tile_cnt + (int64_t)h * g.nQt;
  for (int x0 = wave * 64; x0 < n_before; x0 += 1024) {
    int v[4];
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int x = min(x0 + 256 * y + lane, n_before - 1);
      v[y] = *(x < n_head ? head_cnt + x : cnt_h + (x - n_head));
    }
#pragma unroll
    for (int y = 0; y < 4; ++y) part += x0 + 256 * y + lane < n_before ? v[y] : 0;
  }
  const int mine4 = cnt_h[min(at0 + min(lane, each - 1), g.nQt - 1)];  // the workgroup's own counts, one per lane
  const int my_cnt = __builtin_amdgcn_readlane(mine4, qt - at0);
  // the walk's index words, a word of 64 tiles per lane, the first 64 of them before the sets are staged
  uint64_t ow_mine = lane < n_words ? oc[lane] : 0, fw_mine = lane < n_words ? fl[lane] : 0;
  // gathered columns: the ordinary tiles of a query tile of the pattern region hold the diagonal part only
  const bool split = gidx != nullptr && qt * tile_m >= L;
  // (their first index word too: a load issued behind the stores of the ordinary tiles waits for them)
  const uint64_t *voc = split ? vocc + ((int64_t)h * g.nQt + qt) * g.occw : nullptr;
  const uint64_t *vfl = split ? vfull + ((int64_t)h * g.nQt + qt) * g.occw : nullptr;
  const int n_gt = split ? (gcnt[h] + tile_n - 1) / tile_n : 0;
  // no matched diagonal lies beyond r_bound (as in tile_scan_row)
  int64_t r_bound = INT64_MAX;
  if (split && tile_m == tile_n && (qt + 1) * tile_m <= g.S)
    r_bound = farthest_tile(classes + ((int64_t)h * 4 + kOffAny) * g.occw, g.occw, lane) * tile_n + tile_n - 1;
  const uint64_t vow0 = split ? voc[0] : 0, vfw0 = split ? vfl[0] : 0;  // (not written where there is no gathered tile)
  {
    const int low = wave_total((int)(part & 0xFFFFFF)), high = wave_total((int)(part >> 24));  // (64 lanes' sums fit 32 bits each)
    if (lane == 0) s_before[wave] = ((int64_t)high << 24) + low;
  }
  if (STAGED) stage_sets(lds_sets, g.pw, cb, rr);
  else __syncthreads();
  if (!live) return;
  int64_t first = s_before[0] + s_before[1] + s_before[2] + s_before[3];
  for (int y = 0; y < qt - at0; ++y) first += __builtin_amdgcn_readlane(mine4, y);
  if (lane == 0 && my_turn == 0) {  // the CSR offsets, cut to the capacity like everything they point into
    int *rp = row_ptr + (int64_t)h * (g.nQt + 1);
    rp[qt] = (int)min(first, capacity);
    if (qt == g.nQt - 1) {
      rp[g.nQt] = (int)min(first + my_cnt, capacity);
      if (h == g.H - 1 && blk_total) *blk_total = first + my_cnt;
    }
  }
  const int words = tile_m * wpr;
  const int qw = tile_n / 4;  // quarter width in keys, a multiple of 16
  // the walk, once for sets in LDS and once for sets in global memory (see stage_sets)
  auto walk = [&](const uint64_t *cb, const uint64_t *rr, auto in_lds) __attribute__((always_inline)) {
  constexpr bool IN_LDS = decltype(in_lds)::value;
  if (split) cb = nullptr;
  // walk the listed tiles of this query tile in ascending order
  int rank = 0;
  uint64_t todo = __ballot(ow_mine != 0);  // (empty words are passed over: 446 -> 432 us at 64 heads x 128k)
  for (int wb = 0; wb < n_words;) {
    if (!todo) {
      wb += 64;
      if (wb >= n_words) break;
      ow_mine = wb + lane < n_words ? oc[wb + lane] : 0;
      fw_mine = wb + lane < n_words ? fl[wb + lane] : 0;
      todo = __ballot(ow_mine != 0);
      continue;
    }
    const int from = __ffsll((unsigned long long)todo) - 1, ow_i = wb + from;
    todo &= todo - 1;
    auto word_of = [&](uint64_t x) {
      return (uint64_t)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), from) << 32 |
             (unsigned)__builtin_amdgcn_readlane((int)x, from);
    };
    uint64_t ow = word_of(ow_mine);
    const uint64_t fw = word_of(fw_mine);
    const uint64_t listed = ow;
    if (skip_full_bits) {
      // full tiles get a column and a kind only: all of the word's at once, lane j takes tile 64 ow_i + j
      const uint64_t below = (1ull << lane) - 1;
      const int r = rank + __popcll(listed & below);
      if (((listed & fw) >> lane) & 1) {
        const int64_t t = first + r;
        if (r % share == my_turn && t < capacity) {
          if (blk_col) blk_col[t] = ow_i * 64 + lane;
          if (blk_kind) blk_kind[t] = (uint8_t)31;
        }
      }
      ow &= ~fw;
    }
    const int rank0 = rank;
    rank += __popcll(listed);
    while (ow) {
      const int bit = __ffsll((unsigned long long)ow) - 1;
      const int kt = ow_i * 64 + bit;
      ow &= ow - 1;
      const int rk = rank0 + __popcll(listed & ((1ull << bit) - 1));
      const int64_t t = first + rk;
      const bool mine = rk % share == my_turn;
      if (!mine || t >= capacity) continue;
      // element words, and which key quarters of the tile hold a kept entry
      const bool is_full = (fw >> (kt & 63)) & 1;
      int quarters = 0, kind_q = 0;  // occupied key quarters: per lane (summed up by ballots below), or for the wave
      const bool by_rows = PATTERNS || (words == 256 && wpr == 2 && qt * 128 >= L && qt * 128 + 128 <= g.S);
      if (by_rows) {
        // 128 x 128 tile with every row in the pattern region: a lane takes rows lane and lane + 64 whole
        // (128 keys = two words). The offsets i - j of a row's 128 keys are 128 consecutive positions of the
        // reversed diagonal set, starting at Q - (i - 128 kt); row lane + 64 starts 64 positions below row lane,
        // so both rows come out of four consecutive words of the set: 256 bits, of which row lane + 64 takes
        // bits [sh, sh + 128) and row lane bits [64 + sh, 64 + sh + 128), as 32-bit funnel shifts.
        const int Q = g.pw * 64 - 1;
        const uint64_t c0 = cb ? set_word(cb, 2 * kt, g.pw) : 0, c1 = cb ? set_word(cb, 2 * kt + 1, g.pw) : 0;
        const int u_lane = (qt - kt) * 128 + lane;  // offset of the tile's first key in row lane, >= 0
        const int s0 = Q - u_lane;                  // (negative where the row's offsets lie beyond the pattern length)
        const int w0 = max(s0 >> 6, -3);            // from word -3 down all four words are outside the set
        // (staged sets carry four zero words in front and two behind: words -4 .. -1, pw and pw + 1 read as nothing)
        // (written out value by value: arrays indexed in unrolled loops end up in scratch memory here, because the
        // choice between neighbours below is turned into an index first)
        auto word = [&](int w) { return IN_LDS ? rr[w] : set_word(rr, w, g.pw); };
        const uint64_t wd0 = word(w0 - 1), wd1 = word(w0), wd2 = word(w0 + 1), wd3 = word(w0 + 2);
        const uint32_t e0 = (uint32_t)wd0, e1 = (uint32_t)(wd0 >> 32), e2 = (uint32_t)wd1, e3 = (uint32_t)(wd1 >> 32);
        const uint32_t e4 = (uint32_t)wd2, e5 = (uint32_t)(wd2 >> 32), e6 = (uint32_t)wd3, e7 = (uint32_t)(wd3 >> 32);
        const bool odd = (s0 & 32) != 0;
        const int r = s0 & 31;
        const uint32_t f0 = odd ? e1 : e0, f1 = odd ? e2 : e1, f2 = odd ? e3 : e2, f3 = odd ? e4 : e3;
        const uint32_t f4 = odd ? e5 : e4, f5 = odd ? e6 : e5, f6 = odd ? e7 : e6;
        uint32_t row[2][4];  // [u][dword]: row lane + 64 u
        row[1][0] = __builtin_amdgcn_alignbit(f1, f0, r);
        row[1][1] = __builtin_amdgcn_alignbit(f2, f1, r);
        row[1][2] = __builtin_amdgcn_alignbit(f3, f2, r);
        row[1][3] = __builtin_amdgcn_alignbit(f4, f3, r);
        row[0][0] = row[1][2];
        row[0][1] = row[1][3];
        row[0][2] = __builtin_amdgcn_alignbit(f5, f4, r);
        row[0][3] = __builtin_amdgcn_alignbit(f6, f5, r);
        const uint32_t cd[4] = {(uint32_t)c0, (uint32_t)(c0 >> 32), (uint32_t)c1, (uint32_t)(c1 >> 32)};
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k) row[u][k] = is_full ? ~0u : (row[u][k] | cd[k]);
        if (kt == qt) {  // the diagonal tile (wave-uniform): keys up to the row's own only
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int u0 = u_lane + 64 * u;  // = the row's index inside the tile
            const uint64_t lo = u0 >= 63 ? ~0ull : ((2ull << u0) - 1);
            const uint64_t hi = u0 >= 127 ? ~0ull : (u0 < 64 ? 0ull : ((2ull << (u0 - 64)) - 1));
            row[u][0] &= (uint32_t)lo; row[u][1] &= (uint32_t)(lo >> 32);
            row[u][2] &= (uint32_t)hi; row[u][3] &= (uint32_t)(hi >> 32);
          }
        }
        if (PATTERNS && qt * 128 + 128 > g.S) {  // the last query tile of a ragged length: no row past the end
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (qt * 128 + lane + 64 * u >= g.S) row[u][0] = row[u][1] = row[u][2] = row[u][3] = 0;
        }
        if (tile_bits) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            uint4 st;
            st.x = row[u][0]; st.y = row[u][1]; st.z = row[u][2]; st.w = row[u][3];
            *reinterpret_cast<uint4 *>(tile_bits + t * 256 + 2 * (lane + 64 * u)) = st;
          }
        }
        // a key quarter is 32 keys: one of the four 32-bit words of a row
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (__ballot((row[0][k] | row[1][k]) != 0)) kind_q |= 2 << k;
      } else if (!PATTERNS && words == 256 && wpr == 2) {
        // 128 x 128 tiles: four words per lane, evaluated together so that their loads overlap
        uint64_t m[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int w = lane + 64 * u;
          m[u] = is_full ? ~0ull : mask_word(g, tb, cb, rr, qt * 128 + (w >> 1), kt * 2 + (w & 1));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (tile_bits) tile_bits[t * 256 + lane + 64 * u] = m[u];
          if ((uint32_t)m[u]) quarters |= 1 << (2 * (lane & 1));
          if (m[u] >> 32) quarters |= 2 << (2 * (lane & 1));
        }
      } else if (!PATTERNS)
      for (int w = lane; w < words; w += 64) {
        const int wi = w % wpr;
        const uint64_t m = is_full ? ~0ull : mask_word(g, tb, cb, rr, qt * tile_m + w / wpr, kt * wpr + wi);
        if (tile_bits) tile_bits[t * words + w] = m;
        if (qw == 32) {  // 128-key tiles: a quarter is half a word
          if ((uint32_t)m) quarters |= 1 << (2 * wi);
          if (m >> 32) quarters |= 2 << (2 * wi);
        } else {
          for (int q = 0; q < 4; ++q) {
            // bits of this word that fall into quarter q: keys [q qw, (q + 1) qw) minus the word base
            const int lo = max(q * qw - wi * 64, 0), hi = min((q + 1) * qw - wi * 64, 64);
            if (hi > lo) {
              const uint64_t span = (hi - lo == 64 ? ~0ull : ((1ull << (hi - lo)) - 1)) << lo;
              if (m & span) quarters |= 1 << q;
            }
          }
        }
      }
      int kind = (is_full ? 1 : 0) | kind_q;
      if (!by_rows)
        for (int q = 0; q < 4; ++q)
          if (__ballot(quarters & (1 << q))) kind |= 2 << q;
      if (lane == 0) {
        if (blk_col) blk_col[t] = kt;
        if (blk_kind) blk_kind[t] = (uint8_t)kind;
      }
    }
  }
  if (!split) return;
  // the gathered tiles, after the ordinary ones: tile index nKt + v
  const int *gi = gidx + (int64_t)h * gstride;
  const int i0 = qt * tile_m;
  // (a tile's columns are fetched while the tile before it is written: a load issued behind stores waits for them)
  int v_pre = -1, c_pre[4] = {-1, -1, -1, -1};  // (tiles are at most 256 wide: four groups of 64 slots)
  for (int ow_i = 0; ow_i * 64 < n_gt; ++ow_i) {
    uint64_t ow = ow_i == 0 ? vow0 : voc[ow_i];
    const uint64_t vfw = ow_i == 0 ? vfw0 : vfl[ow_i];
    if (skip_full_bits) {
      // full tiles get a column and a kind only: all of the word's at once, lane j takes gathered tile 64 ow_i + j
      const uint64_t listed = ow;
      const int r = rank + __popcll(listed & ((1ull << lane) - 1));
      if (((listed & vfw) >> lane) & 1) {
        const int64_t t = first + r;
        if (r % share == my_turn && t < capacity) {
          if (blk_col) blk_col[t] = g.nKt + ow_i * 64 + lane;
          if (blk_kind) blk_kind[t] = (uint8_t)31;
        }
      }
    }
    const uint64_t listed_v = ow;
    const int rank0_v = rank;
    rank += __popcll(listed_v);
    if (skip_full_bits) ow &= ~vfw;
    while (ow) {
      const int bit = __ffsll((unsigned long long)ow) - 1;
      const int v = ow_i * 64 + bit;
      ow &= ow - 1;
      const int rk = rank0_v + __popcll(listed_v & ((1ull << bit) - 1));
      const int64_t t = first + rk;
      const bool mine = rk % share == my_turn;
      if (!mine || t >= capacity) continue;
      const bool is_full = (vfw >> (v & 63)) & 1;
      int c_all[4];
#pragma unroll
      for (int wg = 0; wg < 4; ++wg)
        if (wg < wpr) c_all[wg] = v == v_pre ? c_pre[wg] : gi[v * tile_n + wg * 64 + lane];
      if (ow) {  // the next listed tile of this word (if it turns out not to be this wave's, the fetch is wasted)
        v_pre = ow_i * 64 + __ffsll((unsigned long long)ow) - 1;
#pragma unroll
        for (int wg = 0; wg < 4; ++wg)
          if (wg < wpr) c_pre[wg] = gi[v_pre * tile_n + wg * 64 + lane];
      }
      int kind = 0;
#pragma unroll
      for (int wg = 0; wg < 4; ++wg) {  // the tile's slots, 64 at a time: lane = slot
        if (wg >= wpr) break;
        const int c = c_all[wg];
        uint64_t keep[4];
        // (filled slots above every matched diagonal keep every row)
        const bool far = r_bound != INT64_MAX && __ballot(c >= 0 && (int64_t)i0 - c <= r_bound) == 0;
        if (far) keep[0] = keep[1] = keep[2] = keep[3] = c >= 0 ? ~0ull : 0ull;
        else slot_rows(g, rr, i0, c, keep);
        const bool any = (keep[0] | keep[1] | keep[2] | keep[3]) != 0;
        const uint64_t lanes_any = __ballot(any);
        for (int q = 0; q < 4; ++q) {  // quarter q: slots [q qw, (q + 1) qw)
          const int lo = q * qw - wg * 64, hi = lo + qw;
          if (hi > 0 && lo < 64) {
            const int a = max(lo, 0), b = min(hi, 64);
            const uint64_t span = (b - a == 64 ? ~0ull : ((1ull << (b - a)) - 1)) << a;
            if (lanes_any & span) kind |= 2 << q;
          }
        }
        if (tile_bits) {
          const uint64_t filled = __ballot(c >= 0);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (k < tile_m / 64) {
              // rows 64 k .. 64 k + 63 of the group: lane r gets the word (row 64 k + r, group wg), whose bit l is
              // slot l. Where every filled slot keeps all 64 rows (no row above a column, no matched offset met:
              // the usual case away from the diagonal) every row's word is the set of filled slots; otherwise the
              // 64 x 64 bits are transposed.
              const bool plain = far || __ballot(keep[k] != (c >= 0 ? ~0ull : 0ull)) == 0;  // wave-uniform
              tile_bits[t * words + (int64_t)(64 * k + lane) * wpr + wg] = plain ? filled : transpose64(keep[k], lane);
            }
        }
      }
      if (lane == 0) {
        if (blk_col) blk_col[t] = g.nKt + v;
        if (blk_kind) blk_kind[t] = (uint8_t)((is_full ? 1 : 0) | kind);
      }
    }
  }
  };
  if constexpr (STAGED)
    walk(lds_sets, lds_sets + g.pw + kGuardFront, std::true_type{});
  else
    walk(cb, rr, std::false_type{});
}

__global__ void k_dense_bits(Geom g, const uint64_t *__restrict__ true_bits,
                             const uint64_t *__restrict__ cbits, const uint64_t *__restrict__ rrev,
                             int sw, uint64_t *__restrict__ dense) {
  const int h = blockIdx.z, i = blockIdx.y;
  const int w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= sw) return;
  const uint64_t *tb = true_bits ? true_bits + (int64_t)h * g.L * g.tbw : nullptr;
  dense[((int64_t)h * g.S + i) * sw + w] =
      mask_word(g, tb, cbits + (int64_t)h * g.pw, rrev + (int64_t)h * g.pw, i, w);
}

// Kept-key lists of rows [row_begin, row_end): count, scan, fill (ascending).
__global__ __launch_bounds__(256) void k_row_count(Geom g, const uint64_t *__restrict__ true_bits,
                                                   const uint64_t *__restrict__ cbits,
                                                   const uint64_t *__restrict__ rrev, int row_begin,
                                                   int nrows, int *__restrict__ cnt) {
  __shared__ int total;
  const int h = blockIdx.y, i = row_begin + blockIdx.x;
  const uint64_t *tb = true_bits ? true_bits + (int64_t)h * g.L * g.tbw : nullptr;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  int mine = 0;
  for (int w = threadIdx.x; w <= (i >> 6); w += blockDim.x)
    mine += __popcll(mask_word(g, tb, cbits + (int64_t)h * g.pw, rrev + (int64_t)h * g.pw, i, w));
  for (int off = 32; off; off >>= 1) mine += __shfl_xor(mine, off);
  if ((threadIdx.x & 63) == 0 && mine) atomicAdd(&total, mine);
  __syncthreads();
  if (threadIdx.x == 0) cnt[(int64_t)h * nrows + blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_row_fill(Geom g, const uint64_t *__restrict__ true_bits,
                                                  const uint64_t *__restrict__ cbits,
                                                  const uint64_t *__restrict__ rrev, int row_begin,
                                                  int nrows, const int *__restrict__ kept_ptr,
                                                  int *__restrict__ kept_idx, int64_t capacity) {
  __shared__ int wave_sum[4];
  __shared__ int carry;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = blockIdx.y, i = row_begin + blockIdx.x;
  const uint64_t *tb = true_bits ? true_bits + (int64_t)h * g.L * g.tbw : nullptr;
  const int64_t first = kept_ptr[(int64_t)h * nrows + blockIdx.x];
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int nw = (i >> 6) + 1;
  for (int base = 0; base < nw; base += 256) {
    const int w = base + threadIdx.x;
    uint64_t m = w < nw ? mask_word(g, tb, cbits + (int64_t)h * g.pw, rrev + (int64_t)h * g.pw, i, w) : 0;
    const int v = __popcll(m);
    int incl = v;
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(incl, off);
      if (lane >= off) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = carry;
    for (int x = 0; x < wave; ++x) before += wave_sum[x];
    int64_t at = first + before + incl - v;
    while (m) {
      const int b = __ffsll((unsigned long long)m) - 1;
      if (at < capacity) kept_idx[at] = w * 64 + b;
      ++at;
      m &= m - 1;
    }
    __syncthreads();
    if (threadIdx.x == 255) carry = before + incl;
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------------
// Kept lists of one row, as a decode step needs them: one list per group of G consecutive maps (DAM_MASK_GROUP_LISTS;
// a list per map is groups of one), holding each key some map of the group keeps once, in G + 1 runs (kept by two or
// more maps; by map 0 alone; by map 1 alone; ...), each ascending, with a byte of member bits per entry. A lane owns
// kPieceBits consecutive keys, a workgroup kListSpan; the work is spread thin on purpose: the lists are short, so the
// time is launches and the latency of the longest chain of dependent steps, not throughput.
//
// Two launches, count per (group, run, span) and fill, both straight from the flags (from the true bits for a row above
// pcl): a piece is eight flag bytes of the columns and eight of the diagonals, and turning whole flag rows into
// bitsets first is a launch of its own for twice the reading. The fill kernel adds up the counts before its own
// itself, so there is no scan launch either up to kAddedCounts of them. 8 KV heads of 4 maps at row 20000: 21 us
// in four launches (bitsets, count, scan, fill) -> 13 us; 16 maps at row 4095: 13 -> 8 us.
constexpr int kMaxGroup = 8;
constexpr int kPieceBits = 8;
constexpr int kPiecesPerWord = 64 / kPieceBits;
constexpr int kChunkWords = 64 / kPiecesPerWord;  // mask words per wave
constexpr int kListSpan = 256 * kPieceBits;       // keys per workgroup
// Beyond this many counts a scan launch between the two is cheaper than every workgroup adding up what lies before it,
// which grows with the square of (lists x spans). Time of the whole build, us, added / scanned: 32 maps at 20000 in groups
// of four (400 counts) 12.0 / 14.5; 64 maps at 262144 in groups of four (10240) 32.5 / 34.2, one by one (16384) 50.9 /
// 44.6; 64 maps at 2^20 one by one (65536) 377 / 156.
constexpr int64_t kAddedCounts = 12288;

// This lane's pieces of row i, keys [key0, key0 + 8), for the maps of group kv (m[x], zero for x >= G), and the bits set in at least
// two of them. Flags are read eight at a time, all maps' together and none behind a test: a piece that the row's or the flags' end
// cuts is read from inside and shifted. (Flag by flag, the one piece at the row's end held both launches unless the row ends with a
// whole one, seven in eight do not: 8 lists of four maps at 20004 18.2 -> 9.0 us, at 20007 9.9 -> 9.0; of eight at 17000 27.2 -> 11.4.)
__device__ __forceinline__ void row_pieces(const Geom &g, const uint64_t *__restrict__ true_bits,
                                           const uint8_t *__restrict__ dflag, const uint8_t *__restrict__ vflag, int kv, int G, int i,
                                           int key0, unsigned (&m)[kMaxGroup], unsigned &shared) {
  const int u = i - key0;  // offset of the first key; key k of the piece has offset u - k
  const unsigned causal = u >= 7 ? 0xFFu : u < 0 ? 0u : (2u << u) - 1;
  if (i < g.L) {  // uniform
#pragma unroll
    for (int x = 0; x < kMaxGroup; ++x) {
      m[x] = 0;
      if (x < G && u >= 0) {
        m[x] = (unsigned)(true_bits[((int64_t)(kv * G + x) * g.L + i) * g.tbw + (key0 >> 6)] >> (key0 & 63)) & causal;
        if (key0 + 8 > g.L) m[x] &= (1u << (g.L - key0)) - 1;
      }
    }
  } else if (g.P >= 8) {  // uniform
    const int at_v = min(key0, g.P - 8), at_d = min(max(u - 7, 0), g.P - 8);
    const int cut_v = min(key0 - at_v, 8), cut_d = 7 - u + at_d;  // (cut_d < 0: offsets past the flags' end)
    uint64_t v[kMaxGroup], d[kMaxGroup];
#pragma unroll
    for (int x = 0; x < kMaxGroup; ++x)
      if (x < G) {  // uniform
        const int64_t row = (int64_t)(kv * G + x) * g.P;
        __builtin_memcpy(&v[x], vflag + row + at_v, 8);
        __builtin_memcpy(&d[x], dflag + row + at_d, 8);
      }
#pragma unroll
    for (int x = 0; x < kMaxGroup; ++x) {
      m[x] = 0;
      if (x < G) {
        const unsigned off = __brev(bits_of_8((unsigned)d[x], (unsigned)(d[x] >> 32))) >> 24;
        m[x] = (bits_of_8((unsigned)v[x], (unsigned)(v[x] >> 32)) >> cut_v | (cut_d >= 0 ? off >> min(cut_d, 8) : off << min(-cut_d, 8))) & causal;
      }
    }
  } else {
#pragma unroll
    for (int x = 0; x < kMaxGroup; ++x) {
      m[x] = 0;
      for (int k = 0; k < 8 && x < G; ++k) {
        const int64_t row = (int64_t)(kv * G + x) * g.P;
        const bool col = key0 + k < g.P && vflag[row + key0 + k] != 0;
        const bool off = u - k >= 0 && u - k < g.P && dflag[row + u - k] != 0;
        m[x] |= ((col || off) && k <= u ? 1u : 0u) << k;
      }
    }
  }
  unsigned any = 0;
  shared = 0;
#pragma unroll
  for (int x = 0; x < kMaxGroup; ++x) {
    shared |= any & m[x];
    any |= m[x];
  }
}

// cnt[(kv * (G + 1) + run) * spans + span]
__global__ __launch_bounds__(256) void k_list_count(Geom g, const uint64_t *__restrict__ true_bits,
                                                    const uint8_t *__restrict__ dflag, const uint8_t *__restrict__ vflag, int row,
                                                    int G, int *__restrict__ cnt) {
  __shared__ int part[4][kMaxGroup + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kv = blockIdx.y, spans = gridDim.x;
  unsigned m[kMaxGroup], shared;
  row_pieces(g, true_bits, dflag, vflag, kv, G, row, (blockIdx.x * 256 + threadIdx.x) * kPieceBits, m, shared);
#pragma unroll
  for (int r = 0; r <= kMaxGroup; ++r)
    if (r <= G) {
      const int c = wave_total(__popc(r == 0 ? shared : m[r - 1] & ~shared));
      if (lane == 0) part[wave][r] = c;
    }
  __syncthreads();
  if (threadIdx.x <= G)
    cnt[((int64_t)kv * (G + 1) + threadIdx.x) * spans + blockIdx.x] =
        part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] + part[3][threadIdx.x];
}

// SCANNED: cnt is the exclusive scan of the counts, with the total behind it.
template <bool SCANNED>
__global__ __launch_bounds__(256) void k_list_fill(Geom g, const uint64_t *__restrict__ true_bits,
                                                   const uint8_t *__restrict__ dflag, const uint8_t *__restrict__ vflag, int row,
                                                   int G, const int *__restrict__ cnt, int *__restrict__ kept_ptr,
                                                   int64_t *__restrict__ kept_total, int *__restrict__ kept_idx,
                                                   uint8_t *__restrict__ kept_member, int64_t capacity) {
  // [r <= G]: entries before run r of this span, counted from the end of what lies before run r - 1's; [G + 1]: the rest
  __shared__ unsigned long long before[kMaxGroup + 2];
  __shared__ int part[4][kMaxGroup + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kv = blockIdx.y, n_groups = gridDim.y, span = blockIdx.x, spans = gridDim.x;
  if (threadIdx.x < kMaxGroup + 2) before[threadIdx.x] = 0;
  const int key0 = (span * 256 + (int)threadIdx.x) * kPieceBits;
  unsigned m[kMaxGroup], shared;
  row_pieces(g, true_bits, dflag, vflag, kv, G, row, key0, m, shared);
  __syncthreads();
  const int64_t at0 = (int64_t)kv * (G + 1) * spans + span, last = (int64_t)n_groups * (G + 1) * spans;
  if (SCANNED) {
    if (threadIdx.x <= G + 1) {
      const int64_t to = threadIdx.x <= G ? at0 + (int64_t)threadIdx.x * spans : last;
      before[threadIdx.x] = (unsigned long long)(cnt[to] - (threadIdx.x > 0 ? cnt[at0 + (int64_t)(threadIdx.x - 1) * spans] : 0));
    }
  } else {
    unsigned long long sum = 0;
    for (int64_t e = threadIdx.x; e < at0; e += 256) sum += cnt[e];
    for (int off = 32; off; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0 && sum) atomicAdd(&before[0], sum);
    for (int e = threadIdx.x; e < G * spans; e += 256) atomicAdd(&before[1 + e / spans], (unsigned long long)cnt[at0 + e]);
    if (kv == n_groups - 1 && span == 0)  // the workgroup that reports the total adds up the counts from its last run on
      for (int64_t e = at0 + (int64_t)G * spans + threadIdx.x; e < last; e += 256)
        atomicAdd(&before[G + 1], (unsigned long long)cnt[e]);
  }
  int incl[kMaxGroup + 1];
#pragma unroll
  for (int r = 0; r <= kMaxGroup; ++r)
    if (r <= G) {
      incl[r] = wave_prefix(__popc(r == 0 ? shared : m[r - 1] & ~shared));
      if (lane == 63) part[wave][r] = incl[r];
    }
  __syncthreads();
  if (threadIdx.x == 0 && span == 0) {  // (offsets past the capacity of the list buffers are cut to it, like the block index')
    const unsigned long long clamp = kept_idx ? (unsigned long long)capacity : (unsigned long long)INT64_MAX;
    kept_ptr[kv] = (int)min(before[0], clamp);
    if (kv == n_groups - 1) {
      unsigned long long total = 0;
      for (int r = 0; r <= G + 1; ++r) total += before[r];
      kept_ptr[n_groups] = (int)min(total, clamp);
      if (kept_total && !SCANNED) *kept_total = (int64_t)total;  // (the scan has written it)
    }
  }
  if (!kept_idx) return;
  int64_t base = 0;
#pragma unroll
  for (int r = 0; r <= kMaxGroup; ++r) {
    if (r <= G) {
      unsigned left = r == 0 ? shared : m[r - 1] & ~shared;  // lane's piece of run r
      base += (int64_t)before[r];
      int64_t at = base + incl[r] - __popc(left);
      for (int x = 0; x < wave; ++x) at += part[x][r];
      while (left) {
        const int bit = __ffs(left) - 1;
        left &= left - 1;
        unsigned who = r == 0 ? 0u : 1u << (r - 1);
        if (r == 0) {
#pragma unroll
          for (int y = 0; y < kMaxGroup; ++y) who |= ((m[y] >> bit) & 1u) << y;  // m[y] = 0 for y >= G
        }
        if (at < capacity) {
          kept_idx[at] = key0 + bit;
          if (kept_member) kept_member[at] = (uint8_t)who;
        }
        ++at;
      }
    }
  }
}

// The same in one launch, a workgroup per list, for rows of up to 1024 W keys and up to 64 lists. What a list needs of the
// others is how many entries lie in front of its own, the totals of the lists before it: every workgroup says its total where
// the others can read it past their L2 (two words that only this call's number makes a total of: nothing has to be cleared, and a
// captured launch, whose number would be the same at every replay, takes the two launches above) and looks at those in front.
// Nobody waits for longer than `polls` looks: a total that is not there by then is counted again from the flags.
// Bound by the chain flags -> counts -> totals -> entries of one workgroup per list, and its instructions: a lane owns W keys next
// to each other, so that a run takes one prefix sum whatever the row's length. Lists with
// the decode behind them, us, two launches / this: 8 sequences at 20000, merged lists of 32 heads 29.5 / 28.0, 2 at 32700 32.5 / 23.0,
// 4 at 8000 (16 heads) 19.6 / 15.7; a list per head 4 fp32 sequences at 4096, 16 heads 12.2 / 10.6, 2 at 30000, 32 heads 20.4 / 18.0.
constexpr int kOneLists = 64, kOnePolls = 64;
// Where a lane owns 128 bytes of flags of either kind (four maps above 16384 keys, eight above 8192), flags off a multiple of
// eight bytes cost this launch 2 us and the other two nothing, so up to 32 lists of such rows take those; lists alone, two
// launches / this, us: 8 lists of four maps at 24575, windows, 9.1 / 11.3, in place 9.1 / 7.5, 5 % of the keys one by one 9.7 /
// 13.4, in place 10.4 / 9.8; 64 lists 13.6 / 12.1. 8 of four maps at 16383, 64 bytes, off 9.1 / 8.1. (Bound by its instructions, it
// grows with the keys that it lists, the two launches hardly do: with a fifth of the keys kept one by one they are faster from
// some 16000 keys on, 8 lists of one map at 20007 6.7 / 8.0, of four at 16383 9.9 / 14.3. The host does not know that.)
constexpr int kOneWide = 128, kOneWideLists = 32;

// m[x]: bit k is key W * lane of the workgroup + k of the map x of group kv, of row i >= L whose patterns all exist (i < P, P >= W).
// All flags are under way together, none of them behind a test: a piece that the row's or the flags' end cuts is read from inside
// and shifted.
template <int W, int GM>
__device__ __forceinline__ void keys_of_list(const Geom &g, const uint8_t *__restrict__ dflag, const uint8_t *__restrict__ vflag, int kv, int G,
                                             int i, unsigned (&m)[GM]) {
  constexpr int kWords = W / 8;
  uint64_t v[GM][kWords], d[GM][kWords];
  const int key0 = (int)threadIdx.x * W, left = i - key0;  // (keys behind the row's own: left < 0)
  const int at_v = min(key0, g.P - W), at_d = max(left - (W - 1), 0);  // offset of key k: left - k
#pragma unroll
  for (int x = 0; x < GM; ++x) {
    const int64_t row = (int64_t)(kv * G + min(x, G - 1)) * g.P;
    __builtin_memcpy(v[x], vflag + row + at_v, W);
    __builtin_memcpy(d[x], dflag + row + at_d, W);
  }
  const unsigned all = W == 32 ? ~0u : (1u << (W & 31)) - 1, causal = left >= W - 1 ? all : left < 0 ? 0u : (2u << left) - 1;
  const int cut_v = min(key0 - at_v, 31), cut_d = left < 0 ? 0 : max(W - 1 - left, 0);
  auto gather = [&](auto ones) {  // ones: no flag is above 1, so its byte is its bit
    constexpr bool ONES = decltype(ones)::value;
    auto eight = [](uint64_t y) -> unsigned {
      const unsigned lo = (unsigned)y, hi = (unsigned)(y >> 32);
      if (ONES) return __builtin_amdgcn_udot4(hi, 0x80402010u, __builtin_amdgcn_udot4(lo, 0x08040201u, 0, false), false);
      return bits_of_8(lo, hi);
    };
#pragma unroll
    for (int x = 0; x < GM; ++x) {
      unsigned vb = 0, db = 0;
#pragma unroll
      for (int w = 0; w < kWords; ++w) {
        vb |= eight(v[x][w]) << (8 * w);
        db |= eight(d[x][w]) << (8 * w);
      }
      m[x] = x < G ? (vb >> cut_v | __brev(db) >> (32 - W) >> cut_d) & causal : 0;
    }
  };
  uint64_t high = 0;
#pragma unroll
  for (int x = 0; x < GM; ++x)
#pragma unroll
    for (int w = 0; w < kWords; ++w) high |= v[x][w] | d[x][w];
  if (__ballot((high & 0xFEFEFEFEFEFEFEFEull) != 0) == 0) gather(std::true_type{});
  else gather(std::false_type{});
}

template <int W, int GM>
__global__ __launch_bounds__(1024) void k_list_one(Geom g, const uint8_t *__restrict__ dflag, const uint8_t *__restrict__ vflag, int row, int G,
                                                   uint64_t number, int polls, uint64_t *__restrict__ said, int *__restrict__ kept_ptr,
                                                   int64_t *__restrict__ kept_total, int *__restrict__ kept_idx,
                                                   uint8_t *__restrict__ kept_member, int64_t capacity) {
  __shared__ int part[GM + 1][16], run_total[GM + 1];
  __shared__ int s_before, s_again;
  __shared__ uint64_t s_missing;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kv = blockIdx.x, lists = gridDim.x;
  unsigned m[GM], more = 0, any = 0;  // more: keys of two maps or more
  keys_of_list<W, GM>(g, dflag, vflag, kv, G, row, m);
#pragma unroll
  for (int x = 0; x < GM; ++x) {
    more |= any & m[x];
    any |= m[x];
  }
  auto run = [&](int r) { return r == 0 ? more : m[r > 0 ? r - 1 : 0] & ~more; };
  // a run's entries in front of the lane's, in its wave; two runs to a sum (a wave has at most 2048 keys)
  int in_wave[GM + 1];
#pragma unroll
  for (int r = 0; r <= GM; r += 2)
    if (r <= G) {
      const int both = __popc(run(r)) | (r < GM ? __popc(run(r + 1)) << 16 : 0), incl = wave_prefix(both);
      in_wave[r] = (incl & 0xFFFF) - (both & 0xFFFF);
      if (lane == 63) part[r][wave] = incl & 0xFFFF;
      if (r < GM) {
        in_wave[r + 1] = (int)((unsigned)incl >> 16) - (both >> 16);
        if (lane == 63) part[r + 1][wave] = (int)((unsigned)incl >> 16);
      }
    }
  __syncthreads();
  if (wave <= G) {
    const int v = lane < 16 ? part[wave][lane] : 0, incl = wave_prefix(v);
    if (lane < 16) part[wave][lane] = incl - v;
    if (lane == 63) run_total[wave] = incl;
  }
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int r = 0; r <= GM; ++r)
    if (r <= G) total += run_total[r];
  if (wave == 0) {
    // (two words: one alone would be taken for a total with a probability of 2^-33 whatever it holds)
    const uint64_t second = number ^ (uint64_t)(unsigned)total;
    if (lane == 0)
      store_through(said + 2 * kv, __uint_as_float((unsigned)number), __uint_as_float((unsigned)(number >> 32)),
                    __uint_as_float((unsigned)second), __uint_as_float((unsigned)(second >> 32)));
    int theirs = 0;
    bool there = lane >= kv;
    for (int look = 0; look < polls && __ballot(!there) != 0; ++look)
      if (!there) {
        const uint64_t a = __hip_atomic_load(said + 2 * lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t b = __hip_atomic_load(said + 2 * lane + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ^ number;
        if (a == number && b >> 31 == 0) {
          theirs = (int)b;
          there = true;
        }
      }
    const uint64_t missing = __ballot(!there);
    const int before = wave_total(theirs);
    if (lane == 0) {
      s_before = before;
      s_missing = missing;
      s_again = 0;
    }
  }
  __syncthreads();
  uint64_t missing = s_missing;
  while (missing) {  // uniform
    const int x = __ffsll((unsigned long long)missing) - 1;
    missing &= missing - 1;
    unsigned other[GM], keys = 0;
    keys_of_list<W, GM>(g, dflag, vflag, x, G, row, other);
#pragma unroll
    for (int y = 0; y < GM; ++y) keys |= other[y];
    int n = __popc(keys);
    n = wave_total(n);
    if (lane == 0) atomicAdd(&s_again, n);
  }
  __syncthreads();
  const int64_t first = (int64_t)s_before + s_again;
  if (threadIdx.x == 0) {  // (offsets past the capacity of the list buffers are cut to it, like the block index')
    const int64_t clamp = kept_idx ? capacity : INT64_MAX;
    kept_ptr[kv] = (int)min(first, clamp);
    if (kv == lists - 1) {
      kept_ptr[lists] = (int)min(first + total, clamp);
      if (kept_total) *kept_total = first + total;
    }
  }
  if (!kept_idx) return;
  // Windows and sinks fill the pieces of a few lanes next to each other: wide pieces are dealt out again for the writing, one to
  // every wave in turn. (Written where they were counted, one wave of the sixteen took 4 us longer than the others.)
  constexpr bool kSpread = W > 8;
  constexpr int kPitch = kSpread ? 17 * 64 : 1;
  __shared__ unsigned piece[GM][kPitch];
  __shared__ unsigned short place[GM + 1][kPitch];
  int my = threadIdx.x, at_run[GM + 1];  // the piece this lane writes, and its places in the runs
#pragma unroll
  for (int r = 0; r <= GM; ++r) at_run[r] = r <= G ? part[r][wave] + in_wave[r] : 0;
  if constexpr (kSpread) {
    const int to = my + (my >> 4);  // (17 words for 16 pieces: no two lanes of a wave on one bank)
#pragma unroll
    for (int x = 0; x < GM; ++x)
      if (x < G) piece[x][to] = m[x];
#pragma unroll
    for (int r = 0; r <= GM; ++r)
      if (r <= G) place[r][to] = (unsigned short)at_run[r];
    __syncthreads();
    my = lane * 16 + wave;
    const int from = my + (my >> 4);
    more = any = 0;
#pragma unroll
    for (int x = 0; x < GM; ++x) {
      m[x] = x < G ? piece[x][from] : 0;
      more |= any & m[x];
      any |= m[x];
    }
#pragma unroll
    for (int r = 0; r <= GM; ++r)
      if (r <= G) at_run[r] = place[r][from];
  }
  auto put = [&](int at, int key, unsigned who) {  // at: place in the list
    if (first + at < capacity) {
      kept_idx[first + at] = key;
      if (kept_member) kept_member[first + at] = (uint8_t)who;
    }
  };
  int base = 0;
#pragma unroll
  for (int r = 0; r <= GM; ++r) {
    if (r <= G) {
      unsigned left = run(r);
      int at = base + at_run[r];
      // Lanes with many keys (windows, sinks): 64 / W of them at a time, a lane of the wave per key, so that the stores of
      // neighbours lie side by side. (Key by key in their own lane the launch above took 2 us more.)
      constexpr int kFew = 4, kAtOnce = 64 / W;
      if (W > 8) {
        for (uint64_t many = __ballot(__popc(left) > kFew); many;) {
          int from = 64;
#pragma unroll
          for (int y = 0; y < kAtOnce; ++y) {
            const int next = many ? __ffsll((unsigned long long)many) - 1 : 64;
            if (lane / W == y) from = next;
            many &= many - 1;
          }
          const int src = from & 63, bit = lane & (W - 1);
          const unsigned mask = (unsigned)__shfl((int)left, src);
          const int their_at = __shfl(at, src);
          unsigned who = r == 0 ? 0u : 1u << (r - 1);
          if (r == 0) {
#pragma unroll
            for (int y = 0; y < GM; ++y)
              if (y < G) who |= (((unsigned)__shfl((int)m[y], src) >> bit) & 1u) << y;
          }
          if (from < 64 && ((mask >> bit) & 1)) put(their_at + __popc(mask & ((1u << bit) - 1)), (kSpread ? from * 16 + wave : wave * 64 + from) * W + bit, who);
        }
        if (__popc(left) > kFew) left = 0;
      }
      while (left) {
        const int bit = __ffs(left) - 1;
        left &= left - 1;
        unsigned who = r == 0 ? 0u : 1u << (r - 1);
        if (r == 0) {
#pragma unroll
          for (int y = 0; y < GM; ++y) who |= ((m[y] >> bit) & 1u) << y;
        }
        put(at++, my * W + bit, who);
      }
      base += run_total[r];
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Position-independent lists for grouped-query decoding in the pattern region (DAM_MASK_PATTERN_PLAN): per
// group of G maps first every diagonal offset matched by some map of the group, then every such column, each
// part in G + 1 runs (patterns of two or more maps; of map 0 alone; ...), each run ascending in the key it
// stands for. A diagonal r is stored as -1 - r (key p - r at position p), a column c as c. The diagonal part
// is the kept list of the last row of a P x P mask that has the group's diagonals and no columns (key j of
// that row is offset P - 1 - j), counted, scanned and filled in chunks of a wave's 64 pieces; the
// column part reads the column bitset itself. cnt / first: [((kv * 2 + part) * (G + 1) + run) * nchunks + chunk].
__device__ __forceinline__ void plan_pieces(const Geom &gp, const uint64_t *__restrict__ cbits,
                                            const uint64_t *__restrict__ rrev, int kv, int G, int part, int n_cols, int chunk,
                                            int lane, unsigned (&m)[kMaxGroup], unsigned &shared) {
  const int w = chunk * kChunkWords + lane / kPiecesPerWord;
  const int shift = (lane % kPiecesPerWord) * kPieceBits;
  unsigned any = 0;
  shared = 0;
#pragma unroll
  for (int x = 0; x < kMaxGroup; ++x) {
    m[x] = 0;
    if (x < G && w < gp.pw) {
      const int h = kv * G + x;
      uint64_t word;
      if (part == 0) {
        word = mask_word(gp, nullptr, nullptr, rrev + (int64_t)h * gp.pw, gp.S - 1, w);  // gp.S == P, gp.L == 0
      } else {
        word = cbits[(int64_t)h * gp.pw + w];
        const int left = n_cols - w * 64;  // columns of this word that exist
        word &= left >= 64 ? ~0ull : (left <= 0 ? 0ull : ~0ull >> (64 - left));
      }
      m[x] = (unsigned)(word >> shift) & ((1u << kPieceBits) - 1);
    }
    shared |= any & m[x];
    any |= m[x];
  }
}

__global__ __launch_bounds__(256) void k_plan_count(Geom gp, const uint64_t *__restrict__ cbits,
                                                    const uint64_t *__restrict__ rrev, int G, int n_cols, int nchunks,
                                                    int *__restrict__ cnt) {
  const int lane = threadIdx.x & 63, chunk = blockIdx.x * 4 + (threadIdx.x >> 6), kv = blockIdx.y, part = blockIdx.z;
  if (chunk >= nchunks) return;  // whole waves
  unsigned m[kMaxGroup], shared;
  plan_pieces(gp, cbits, rrev, kv, G, part, n_cols, chunk, lane, m, shared);
  int *out = cnt + (int64_t)(kv * 2 + part) * (G + 1) * nchunks + chunk;
  const int c0 = wave_total(__popc(shared));
  if (lane == 0) out[0] = c0;
#pragma unroll
  for (int x = 0; x < kMaxGroup; ++x) {
    if (x < G) {
      const int c = wave_total(__popc(m[x] & ~shared));
      if (lane == 0) out[(int64_t)(1 + x) * nchunks] = c;
    }
  }
}

__global__ __launch_bounds__(256) void k_plan_fill(Geom gp, const uint64_t *__restrict__ cbits,
                                                   const uint64_t *__restrict__ rrev, int G, int n_cols, int nchunks,
                                                   int n_groups, const int *__restrict__ first, int *__restrict__ kept_ptr,
                                                   int *__restrict__ kept_idx, uint8_t *__restrict__ kept_member,
                                                   int64_t capacity) {
  const int lane = threadIdx.x & 63, chunk = blockIdx.x * 4 + (threadIdx.x >> 6), kv = blockIdx.y, part = blockIdx.z;
  if (chunk >= nchunks) return;  // whole waves
  const int *mine_first = first + (int64_t)(kv * 2 + part) * (G + 1) * nchunks + chunk;
  if (chunk == 0 && lane == 0 && part == 0) {
    const int64_t clamp = kept_idx ? capacity : INT64_MAX;
    kept_ptr[kv] = (int)min((int64_t)mine_first[0], clamp);
    if (kv == n_groups - 1) kept_ptr[n_groups] = (int)min((int64_t)first[(int64_t)n_groups * 2 * (G + 1) * nchunks], clamp);
  }
  if (!kept_idx) return;
  unsigned m[kMaxGroup], shared;
  plan_pieces(gp, cbits, rrev, kv, G, part, n_cols, chunk, lane, m, shared);
  const int key0 = (chunk * kChunkWords + lane / kPiecesPerWord) * 64 + (lane % kPiecesPerWord) * kPieceBits;
  const int base = part == 0 ? key0 - gp.S : key0;  // diagonal part: key j of the virtual row P - 1 is -1 - (P - 1 - j) = j - P
#pragma unroll
  for (int r = 0; r <= kMaxGroup; ++r) {
    if (r <= G) {
      unsigned left = r == 0 ? shared : m[r - 1] & ~shared;
      const int v = __popc(left);
      int incl = v;
      for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
      }
      int64_t at = (int64_t)mine_first[(int64_t)r * nchunks] + incl - v;
      while (left) {
        const int bit = __ffs(left) - 1;
        left &= left - 1;
        unsigned who = r == 0 ? 0u : 1u << (r - 1);
        if (r == 0) {
#pragma unroll
          for (int y = 0; y < kMaxGroup; ++y) who |= ((m[y] >> bit) & 1u) << y;
        }
        if (at < capacity) {
          kept_idx[at] = base + bit;
          if (kept_member) kept_member[at] = (uint8_t)who;
        }
        ++at;
      }
    }
  }
}

// table[kv][r] = which maps of group kv have diagonal r matched (bit x: map kv * G + x)
__global__ void k_plan_table(const uint8_t *__restrict__ diag_flag, int P, int G, uint8_t *__restrict__ table) {
  const int kv = blockIdx.y;
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < P; r += gridDim.x * blockDim.x) {
    unsigned who = 0;
    for (int x = 0; x < G; ++x) who |= (diag_flag[(int64_t)(kv * G + x) * P + r] ? 1u : 0u) << x;
    table[(int64_t)kv * P + r] = (uint8_t)who;
  }
}

int validate(const dam_mask_params *p, const float *attn_sum, const uint8_t *diag_in,
             const uint8_t *vert_in, const dam_mask_out *o) {
  if (!p || !o) return DAM_ERR_INVALID_ARG;
  if (p->mode != DAM_FROM_ATTN_MAP && p->mode != DAM_FROM_PATTERNS) return DAM_ERR_INVALID_ARG;
  if (p->n_maps < 1 || p->seq < 1) return DAM_ERR_INVALID_ARG;
  if (p->flags & ~(DAM_MASK_SKIP_FULL_TILE_BITS | DAM_MASK_GATHER_COLUMNS | DAM_MASK_GROUP_LISTS | DAM_MASK_PATTERN_PLAN))
    return DAM_ERR_INVALID_ARG;
  const bool plan = (p->flags & DAM_MASK_PATTERN_PLAN) != 0;
  if (plan && (!(p->flags & DAM_MASK_GROUP_LISTS) || !o->kept_ptr || !o->plan_table)) return DAM_ERR_INVALID_ARG;
  if ((p->flags & DAM_MASK_GROUP_LISTS) && o->kept_ptr) {
    if (p->group < 1 || p->group > kMaxGroup || p->n_maps % p->group) return DAM_ERR_INVALID_ARG;
    if (!plan && p->row_end != p->row_begin + 1) return DAM_ERR_UNSUPPORTED;
    if (o->kept_idx && !o->kept_member) return DAM_ERR_INVALID_ARG;
  }
  if ((p->flags & DAM_MASK_GATHER_COLUMNS) && (!o->gather_idx || !o->gather_cnt)) return DAM_ERR_INVALID_ARG;
  if (p->tile_m < 64 || p->tile_n < 64 || p->tile_m % 64 || p->tile_n % 64) return DAM_ERR_INVALID_ARG;
  if (p->tile_m > 256 || p->tile_n > 256) return DAM_ERR_UNSUPPORTED;
  if ((int64_t)(p->seq + p->tile_n - 1) / p->tile_n > 32768) return DAM_ERR_UNSUPPORTED;
  if (p->mode == DAM_FROM_ATTN_MAP) {
    if (p->pcl < 1 || !attn_sum || !o->true_bits) return DAM_ERR_INVALID_ARG;
    if (p->pcl >= (1 << kMaxCountBits)) return DAM_ERR_UNSUPPORTED;
    if (!(p->eps > 0.0f)) return DAM_ERR_INVALID_ARG;
    if (p->transform < DAM_T_BOXCOX || p->transform > DAM_T_ARCSINH) return DAM_ERR_INVALID_ARG;
    if (p->transform == DAM_T_BOXCOX && p->lambda != 0.5f && p->lambda != 1.0f) return DAM_ERR_UNSUPPORTED;
    if (isnan(p->lambda)) return DAM_ERR_INVALID_ARG;
    if (isnan(p->tau) || isnan(p->mu)) return DAM_ERR_INVALID_ARG;
  } else {
    if (p->pcl < 0 || !diag_in || !vert_in) return DAM_ERR_INVALID_ARG;
    if (p->pcl > 0 && !o->true_bits) return DAM_ERR_INVALID_ARG;
  }
  const bool blocks = o->blk_col || o->blk_kind || o->tile_bits || o->blk_total || o->blk_row_ptr;
  if (blocks && (!o->blk_row_ptr || !o->blk_total || o->blk_capacity < 0)) return DAM_ERR_INVALID_ARG;
  if ((o->blk_col || o->blk_kind || o->tile_bits) && o->blk_capacity < 1) return DAM_ERR_INVALID_ARG;
  if (o->dense_bits && p->seq > 65535) return DAM_ERR_UNSUPPORTED;
  if (o->kept_ptr || o->kept_idx || o->kept_total) {
    if (!o->kept_ptr || !o->kept_total || o->kept_capacity < 0) return DAM_ERR_INVALID_ARG;
    if (!plan && (p->row_begin < 0 || p->row_begin > p->row_end || p->row_end > p->seq)) return DAM_ERR_INVALID_ARG;
    if ((int64_t)p->n_maps * (p->row_end - p->row_begin) > (int64_t)1 << 30) return DAM_ERR_UNSUPPORTED;
  }
  return DAM_OK;
}

struct Workspace {
  float *bmin;
  unsigned *xmin_bits, *theta_key;
  TransformStats *stats;
  uint64_t *vslices, *dslices;
  uint8_t *diag_flag, *vert_flag;
  uint64_t *cbits, *rrev, *occ, *full, *classes, *vocc, *vfull;
  int *tile_cnt, *head_cnt, *row_cnt, *group_first;
  size_t bytes;
};

// Maps per list when a single row is listed: the group size with DAM_MASK_GROUP_LISTS, else 1 (a list per map is
// the same thing with groups of one: no key is shared, the only run is "map 0 alone", ascending).
int list_group(const dam_mask_params *p) {
  return (p->flags & DAM_MASK_GROUP_LISTS) && p->group >= 1 && p->group <= kMaxGroup ? p->group : 1;
}

// Counts of the lists of a single row: one per list, run and span of keys.
int64_t list_counts(const dam_mask_params *p) {
  const int group = list_group(p);
  return (int64_t)(p->n_maps / group) * (group + 1) * (p->row_begin / kListSpan + 1);
}

// Chunks of kChunkWords mask words covering keys 0..row (one wave each in the plan kernels).
int group_chunks(int row) { return ((row >> 6) + 1 + kChunkWords - 1) / kChunkWords; }

Geom geometry(const dam_mask_params *p) {
  Geom g;
  g.H = p->n_maps;
  g.L = p->pcl;
  g.S = p->seq;
  g.P = p->mode == DAM_FROM_ATTN_MAP ? p->pcl : p->seq;
  g.tile_m = p->tile_m;
  g.tile_n = p->tile_n;
  g.nQt = (g.S + g.tile_m - 1) / g.tile_m;
  g.nKt = (g.S + g.tile_n - 1) / g.tile_n;
  g.wpr = g.tile_n / 64;
  g.tbw = (g.L + 63) / 64;
  g.pw = (g.P + 63) / 64;
  g.occw = (g.nKt + 63) / 64;
  return g;
}

Workspace carve(const dam_mask_params *p, void *ws) {
  const Geom g = geometry(p);
  Carver c(ws);
  Workspace w;
  const size_t HL = (size_t)g.H * (size_t)(g.L > 0 ? g.L : 1);
  w.bmin = c.take<float>(1);
  w.xmin_bits = c.take<unsigned>(1);
  w.theta_key = c.take<unsigned>(1);
  w.stats = c.take<TransformStats>(1);
  const size_t n_slices = p->mode == DAM_FROM_ATTN_MAP
                              ? (size_t)g.H * (size_t)((g.L + kChunkRows - 1) / kChunkRows) * kSlices * (size_t)g.tbw
                              : 1;
  w.vslices = c.take<uint64_t>(n_slices);
  w.dslices = c.take<uint64_t>(n_slices);
  w.diag_flag = c.take<uint8_t>(HL);
  w.vert_flag = c.take<uint8_t>(HL);
  w.cbits = c.take<uint64_t>((size_t)g.H * g.pw);
  w.rrev = c.take<uint64_t>((size_t)g.H * g.pw);
  w.classes = c.take<uint64_t>((size_t)g.H * 4 * g.occw);
  w.occ = c.take<uint64_t>((size_t)g.H * g.nQt * g.occw);
  w.full = c.take<uint64_t>((size_t)g.H * g.nQt * g.occw);
  const bool gather = (p->flags & DAM_MASK_GATHER_COLUMNS) != 0;
  w.vocc = c.take<uint64_t>(gather ? (size_t)g.H * g.nQt * g.occw : 1);
  w.vfull = c.take<uint64_t>(gather ? (size_t)g.H * g.nQt * g.occw : 1);
  w.tile_cnt = c.take<int>((size_t)g.H * g.nQt);
  w.head_cnt = c.take<int>((size_t)g.H * kHeadSub);
  const int nrows = p->row_end > p->row_begin ? p->row_end - p->row_begin : 0;
  size_t n_cnt = (size_t)g.H * (size_t)(nrows > 0 ? nrows : 1);
  size_t n_first = 1;
  if (nrows == 1 && p->row_begin >= 0) {  // a single row: the run sizes per span
    n_cnt = std::max(n_cnt, (size_t)list_counts(p));
    if (list_counts(p) > kAddedCounts) n_first = (size_t)list_counts(p) + 1;
  }
  if (p->flags & DAM_MASK_PATTERN_PLAN) {  // two parts (diagonals, columns) over the P pattern positions
    const int group = list_group(p);
    n_first = std::max(n_first, (size_t)(g.H / group) * 2 * (size_t)group_chunks(g.P - 1) * (size_t)(group + 1) + 1);
    n_cnt = std::max(n_cnt, n_first);
  }
  w.row_cnt = c.take<int>(n_cnt);
  w.group_first = c.take<int>(n_first);
  w.bytes = c.off;
  return w;
}

// a1 and the threshold of a2. attn_sum / attn_cnt are only read in the general minimum. Returns how the
// true-mask kernel gets the key: by value when the host could find it (then that kernel also writes out_bmin),
// else from the workspace.
Threshold stage_threshold(const dam_mask_params *p, const Geom &g, const Workspace &w, const float *attn_sum,
                          const float *attn_cnt, hipStream_t stream, float *out_bmin, bool *bmin_written) {
  const Threshold from_ws{w.theta_key, 0u, 0.0f, nullptr};
  *bmin_written = false;
  if (p->transform != DAM_T_BOXCOX) {
    // App. B alternatives: one reduction pass for the statistics, then minimum and threshold together
    const int64_t n = (int64_t)g.H * g.L * g.L;
    k_stats_init<<<1, 64, 0, stream>>>(w.stats);
    const int blocks = (int)std::min<int64_t>((n + 1023) / 1024, 256 * 16);
    k_stats<<<blocks, 256, 0, stream>>>(attn_sum, attn_cnt, n, g.L, p->eps, w.stats);
    k_transform_threshold<<<1, 64, 0, stream>>>(p->transform, p->lambda, p->eps, p->tau, p->bmin_override, w.stats,
                                                attn_cnt == nullptr, (float)n, (double)n, w.bmin, w.theta_key);
    return from_ws;
  }
  const bool half = p->lambda == 0.5f;
  // a1: the global minimum of the Box-Cox map. Known without the data when the caller overrides it, and for a single
  // causal capture with L >= 2 (some pair was never computed: its X is the clamp eps, and no X is smaller)
  if (!isnan(p->bmin_override) || (!attn_cnt && g.L >= 2)) {
    const float x_min = clamp_mean(0.0f, 0.0f, p->eps);
    const float bmin = !isnan(p->bmin_override) ? p->bmin_override : (half ? box_cox<1>(x_min) : box_cox<2>(x_min));
    unsigned key;
    if (half) key = attn_cnt ? threshold_key<1, false>(p->eps, p->tau, bmin) : threshold_key<1, true>(p->eps, p->tau, bmin);
    else key = attn_cnt ? threshold_key<2, false>(p->eps, p->tau, bmin) : threshold_key<2, true>(p->eps, p->tau, bmin);
    *bmin_written = true;
    return Threshold{nullptr, key, bmin, out_bmin};
  }
  const int64_t n = (int64_t)g.H * g.L * g.L;
  k_fill_u32<<<1, 64, 0, stream>>>(w.xmin_bits, 1, 0x7F800000u);
  const int blocks = (int)std::min<int64_t>((n + 1023) / 1024, 256 * 16);
  k_min_x<<<blocks, 256, 0, stream>>>(attn_sum, attn_cnt, n, g.L, p->eps, w.xmin_bits);
  if (half) k_bmin_from_x<1><<<1, 64, 0, stream>>>(w.xmin_bits, w.bmin);
  else k_bmin_from_x<2><<<1, 64, 0, stream>>>(w.xmin_bits, w.bmin);
  // a2: the threshold, found once
  if (half) {
    if (attn_cnt) k_threshold<1, false><<<1, 64, 0, stream>>>(p->eps, p->tau, w.bmin, w.theta_key);
    else k_threshold<1, true><<<1, 64, 0, stream>>>(p->eps, p->tau, w.bmin, w.theta_key);
  } else {
    if (attn_cnt) k_threshold<2, false><<<1, 64, 0, stream>>>(p->eps, p->tau, w.bmin, w.theta_key);
    else k_threshold<2, true><<<1, 64, 0, stream>>>(p->eps, p->tau, w.bmin, w.theta_key);
  }
  return from_ws;
}

// What follows needs k_pattern_prep whether or not it counts (a single row is listed from the flags).
bool needs_prep(const dam_mask_params *p, const dam_mask_out *o) {
  const bool rows = (p->flags & DAM_MASK_PATTERN_PLAN) != 0 || p->row_end - p->row_begin > 1;
  return o->blk_row_ptr || o->dense_bits || (o->kept_ptr && rows);
}

// Whether k_pattern_prep scans the tiles too: sets in LDS, and few query tiles for a wave to take.
size_t prep_lds_bytes(const Geom &g) {
  const size_t sets = (size_t)g.pw * 16, all = sets + class_bytes(g);
  return sets <= kMaxStagedBytes && all <= kMaxWithClasses ? all : 0;
}
bool scans_in_prep(const Geom &g, const dam_mask_out *o) { return o->blk_row_ptr && prep_lds_bytes(g) > 0 && g.nQt <= kScanInPrep; }

// Whether k_pattern_prep counts the patterns itself (short captures, see count_patterns_of_head).
bool counts_in_prep(const Geom &g) { return g.L <= kDirectL; }

// a3: match scores of the true mask in o->true_bits; says where the flags are written, and (short captures) what
// k_pattern_prep has to count for that. counted: the chunks' slices are there already. map: k_pattern_prep makes the true mask
// too (maps_in_prep).
CountArgs stage_patterns(const dam_mask_params *p, const Geom &g, const Workspace &w, const dam_mask_out *o,
                    hipStream_t stream, const uint8_t **dflag, const uint8_t **vflag, bool bmin_written, bool counted,
                    const float *map = nullptr, const Threshold &thr = {}) {
  uint8_t *df = o->diag_flag ? o->diag_flag : w.diag_flag;
  uint8_t *vf = o->vert_flag ? o->vert_flag : w.vert_flag;
  *dflag = df;
  *vflag = vf;
  if (o->bmin && !bmin_written) k_copy_f32<<<1, 64, 0, stream>>>(o->bmin, w.bmin);
  if (counts_in_prep(g))
    return CountArgs{map ? kFromMap : kFromTrueBits, map, thr, o->true_bits, nullptr, nullptr, p->mu, o->vert_cnt, o->diag_cnt, vf, df};
  const int n_chunks = (g.L + kChunkRows - 1) / kChunkRows;
  if (counted) {
  } else if (g.tbw <= 128) {
    k_pattern_slices<<<dim3(n_chunks, g.H), 256, 0, stream>>>(o->true_bits, g.L, g.tbw, n_chunks, w.vslices, w.dslices);
  } else {
    const dim3 sgrid(2 * ((g.tbw + 63) / 64), (n_chunks + 1) / 2, g.H);
    k_pattern_slices_wide<<<sgrid, 256, 0, stream>>>(o->true_bits, g.L, g.tbw, n_chunks, w.vslices, w.dslices);
  }
  if (g.L <= kSlicesInPrep && needs_prep(p, o))
    return CountArgs{kFromSlices, nullptr, {}, nullptr, w.vslices, w.dslices, p->mu, o->vert_cnt, o->diag_cnt, vf, df};
  k_pattern_finish<<<dim3((g.tbw + 3) / 4, g.H, 2), 256, 0, stream>>>(w.vslices, w.dslices, g.L, g.tbw, n_chunks, p->mu, o->vert_cnt, o->diag_cnt,
                                                                     vf, df);
  return CountArgs{};
}

// Whether there is a form of k_list_one for the lists of one row.
bool one_launch_lists(const dam_mask_params *p, const Geom &g) {
  const int lists = g.H / list_group(p);
  if (lists > kOneLists || p->row_begin >= 1024 * 32 || (int64_t)g.H * g.pw < 2 * lists) return false;
  if (p->row_begin < g.L || p->row_begin >= g.P || g.P < 8) return false;  // (rows of 8192 keys and more: g.P >= 16, 32)
  return list_group(p) <= 4 || p->row_begin < 1024 * 16;                    // (eight maps' pieces of 32 keys spill registers)
}

// Whether they take it. (A stream whose state cannot be told counts as captured.)
bool lists_in_one(const dam_mask_params *p, const Geom &g, hipStream_t stream) {
  if (!one_launch_lists(p, g)) return false;
  const int keys = p->row_begin < 1024 * 8 ? 8 : p->row_begin < 1024 * 16 ? 16 : 32, G = list_group(p), maps = G > 4 ? 8 : G > 1 ? 4 : 1;
  if (maps * keys >= kOneWide && g.P % 8 != 0 && g.H / G <= kOneWideLists) return false;
  hipStreamCaptureStatus state = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &state) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return state == hipStreamCaptureStatusNone;
}

// (the totals lie where the column sets would: nothing reads those behind this launch)
void launch_list_one(const dam_mask_params *p, const Geom &g, const Workspace &w, const dam_mask_out *o, const uint8_t *dflag,
                     const uint8_t *vflag, int polls, hipStream_t stream) {
  const int G = list_group(p), w_at = p->row_begin < 1024 * 8 ? 0 : p->row_begin < 1024 * 16 ? 1 : 2;
  using Kernel = decltype(&k_list_one<8, 1>);
  static const Kernel kernels[3][3] = {{k_list_one<8, 1>, k_list_one<8, 4>, k_list_one<8, 8>},
                                       {k_list_one<16, 1>, k_list_one<16, 4>, k_list_one<16, 8>},
                                       {k_list_one<32, 1>, k_list_one<32, 4>, nullptr}};
  kernels[w_at][G > 4 ? 2 : G > 1 ? 1 : 0]<<<g.H / G, 1024, 0, stream>>>(
      g, dflag, vflag, p->row_begin, G, fresh_flag(), polls, w.cbits, o->kept_ptr, o->kept_total,
      o->kept_capacity > 0 ? o->kept_idx : nullptr, o->kept_member, o->kept_capacity);
}

// a4 + a5 and the kept lists: everything downstream of the stored artefact.
void stage_extension(const dam_mask_params *p, const Geom &g, const Workspace &w, const dam_mask_out *o,
                     const uint64_t *true_bits, const uint8_t *dflag, const uint8_t *vflag, const CountArgs &count,
                     hipStream_t stream) {
  const bool want_blocks = o->blk_row_ptr != nullptr;
  const bool want_lists = o->kept_ptr != nullptr;
  const bool gather = want_blocks && (p->flags & DAM_MASK_GATHER_COLUMNS) != 0;
  const int gstride = dam_gather_stride(p);
  const int *gidx = gather ? o->gather_idx : nullptr, *gcnt = gather ? o->gather_cnt : nullptr;
  const int nrows = p->row_end - p->row_begin;
  const bool plan = (p->flags & DAM_MASK_PATTERN_PLAN) != 0;
  if (needs_prep(p, o) || count.source != kFlagsGiven) {
    const size_t prep_lds = want_blocks ? prep_lds_bytes(g) : 0;
    const ScanArgs scan{scans_in_prep(g, o), w.occ, w.full, w.vocc, w.vfull, w.tile_cnt, true_bits};
    auto form = [&](auto square) {
      constexpr bool SQUARE = decltype(square)::value;
      return count.source == kFromMap        ? k_pattern_prep<kFromMap, SQUARE>
             : count.source == kFromTrueBits ? k_pattern_prep<kFromTrueBits, SQUARE>
             : count.source == kFromSlices   ? k_pattern_prep<kFromSlices, SQUARE>
                                             : k_pattern_prep<kFlagsGiven, SQUARE>;
    };
    auto prep = g.tile_m == g.tile_n ? form(std::true_type{}) : form(std::false_type{});
    prep<<<g.H, 1024, prep_lds, stream>>>(g, count, scan, dflag, vflag, w.cbits, w.rrev, want_blocks, w.classes, gstride, gather ? o->gather_idx : nullptr,
                                                   gather ? o->gather_cnt : nullptr, w.head_cnt, prep_lds > 0);
  }
  // a4 + a5: tile occupancy, CSR offsets, tile bits
  if (want_blocks) {
    const size_t lds_sets = staged_bytes(g);
    const bool fill = o->blk_col || o->blk_kind || o->tile_bits;
    auto grid_of = [&](int each) {
      const TurnGrid t = turn_grid((int64_t)((g.nQt + each - 1) / each) * g.H);
      return dim3(t.x, t.y);
    };
    if (!scans_in_prep(g, o)) {
      const size_t lds = lds_sets > 0 && lds_sets + class_bytes(g) <= kMaxWithClasses ? lds_sets + class_bytes(g) : 0;
      auto form = [&](auto square) {
        constexpr bool SQUARE = decltype(square)::value;
        return g.L > 0 ? (lds > 0 ? k_tile_scan<true, true, SQUARE> : k_tile_scan<true, false, SQUARE>)
                       : (lds > 0 ? k_tile_scan<false, true, SQUARE> : k_tile_scan<false, false, SQUARE>);
      };
      auto scan = g.tile_m == g.tile_n ? form(std::true_type{}) : form(std::false_type{});
      scan<<<grid_of(4), 256, lds, stream>>>(g, true_bits, w.cbits, w.rrev, w.classes, w.occ, w.full, w.tile_cnt, gidx, gcnt, gstride, w.vocc, w.vfull, w.head_cnt);
    }
    if (fill) {
      // (the CSR offsets come out of the fill kernel: no scan launch between the two passes)
      const int share = (int64_t)g.H * g.nQt >= 2048 ? 1 : 4;  // enough query tiles to give every wave its own
      const dim3 fill_grid = grid_of(share == 4 ? 1 : 4);
      const bool skip_full = (p->flags & DAM_MASK_SKIP_FULL_TILE_BITS) != 0;
      const bool patterns = g.L == 0 && g.tile_m == 128 && g.tile_n == 128;
      auto kern = lds_sets > 0 ? (patterns ? k_tile_fill<true, true> : k_tile_fill<true, false>)
                               : (patterns ? k_tile_fill<false, true> : k_tile_fill<false, false>);
      kern<<<fill_grid, 256, lds_sets, stream>>>(g, true_bits, w.cbits, w.rrev, w.occ, w.full, w.tile_cnt, w.head_cnt, o->blk_row_ptr,
                                                 o->blk_total, o->blk_col, o->blk_kind, o->tile_bits, o->blk_capacity, skip_full, gidx, gcnt,
                                                 gstride, w.vocc, w.vfull, w.classes, share);
    } else {  // the sizing call: offsets and total only
      k_exclusive_scan<<<1, 1024, 0, stream>>>(w.tile_cnt, (int64_t)g.H * g.nQt, g.nQt, o->blk_row_ptr, o->blk_total, INT64_MAX);
    }
  }
  if (o->dense_bits) {
    const int sw = (g.S + 63) / 64;
    k_dense_bits<<<dim3((sw + 255) / 256, g.S, g.H), 256, 0, stream>>>(g, true_bits, w.cbits, w.rrev, sw, o->dense_bits);
  }
  if (want_lists && plan) {
    Geom gp = g;  // the P x P pattern-only mask whose last row lists the diagonals
    gp.L = 0;
    gp.S = g.P;
    const int G = list_group(p), n_groups = g.H / G, nchunks = group_chunks(g.P - 1), n_cols = std::min(g.P, g.S);
    const dim3 grid((nchunks + 3) / 4, n_groups, 2);
    k_plan_count<<<grid, 256, 0, stream>>>(gp, w.cbits, w.rrev, G, n_cols, nchunks, w.row_cnt);
    k_exclusive_scan<<<1, 1024, 0, stream>>>(w.row_cnt, (int64_t)n_groups * 2 * (G + 1) * nchunks, 0, w.group_first, o->kept_total,
                                             INT64_MAX);
    k_plan_fill<<<grid, 256, 0, stream>>>(gp, w.cbits, w.rrev, G, n_cols, nchunks, n_groups, w.group_first, o->kept_ptr,
                                          o->kept_capacity > 0 ? o->kept_idx : nullptr, o->kept_member, o->kept_capacity);
    k_plan_table<<<dim3((g.P + 255) / 256, n_groups), 256, 0, stream>>>(dflag, g.P, G, o->plan_table);
  } else if (want_lists) {
    if (nrows == 1) {
      const int G = list_group(p);
      const dim3 grid(p->row_begin / kListSpan + 1, g.H / G);
      const int64_t counts = list_counts(p);
      const bool scan = counts > kAddedCounts;
      if (lists_in_one(p, g, stream)) {
        launch_list_one(p, g, w, o, dflag, vflag, kOnePolls, stream);
        return;
      }
      k_list_count<<<grid, 256, 0, stream>>>(g, true_bits, dflag, vflag, p->row_begin, G, w.row_cnt);
      if (scan) k_exclusive_scan<<<1, 1024, 0, stream>>>(w.row_cnt, counts, 0, w.group_first, o->kept_total, INT32_MAX);
      auto fill = scan ? k_list_fill<true> : k_list_fill<false>;
      fill<<<grid, 256, 0, stream>>>(g, true_bits, dflag, vflag, p->row_begin, G, scan ? w.group_first : w.row_cnt, o->kept_ptr,
                                     o->kept_total, o->kept_capacity > 0 ? o->kept_idx : nullptr, o->kept_member, o->kept_capacity);
    } else if (nrows > 0) {
      k_row_count<<<dim3(nrows, g.H), 256, 0, stream>>>(g, true_bits, w.cbits, w.rrev, p->row_begin, nrows, w.row_cnt);
      const bool fill_lists = o->kept_idx && o->kept_capacity > 0;
      k_exclusive_scan<<<1, 1024, 0, stream>>>(w.row_cnt, (int64_t)g.H * nrows, 0, o->kept_ptr, o->kept_total,
                                               fill_lists ? o->kept_capacity : INT64_MAX);
      if (fill_lists)
        k_row_fill<<<dim3(nrows, g.H), 256, 0, stream>>>(g, true_bits, w.cbits, w.rrev, p->row_begin, nrows, o->kept_ptr,
                                                         o->kept_idx, o->kept_capacity);
    } else {
      k_exclusive_scan<<<1, 1024, 0, stream>>>(w.row_cnt, 0, 0, o->kept_ptr, o->kept_total, INT64_MAX);
    }
  }
}

}  // namespace

extern "C" int32_t dam_gather_stride(const dam_mask_params *p) {
  if (!p || p->seq < 1 || p->tile_n < 64 || p->pcl < 0) return 0;
  const int64_t P = p->mode == DAM_FROM_ATTN_MAP ? p->pcl : p->seq;
  const int64_t n = std::min<int64_t>(P, p->seq);
  return (int32_t)((n + p->tile_n - 1) / p->tile_n * p->tile_n);
}

extern "C" size_t dam_mask_build_workspace(const dam_mask_params *p) {
  if (!p || p->n_maps < 1 || p->seq < 1 || p->pcl < 0 || p->tile_m < 64 || p->tile_n < 64 ||
      p->tile_m % 64 || p->tile_n % 64)
    return 0;
  return carve(p, nullptr).bytes;
}

extern "C" int dam_mask_build(const dam_mask_params *p, const float *attn_sum, const float *attn_cnt,
                              const uint8_t *diag_in, const uint8_t *vert_in, const dam_mask_out *o,
                              void *ws, size_t ws_bytes, void *stream_v) {
  const int bad = validate(p, attn_sum, diag_in, vert_in, o);
  if (bad != DAM_OK) return bad;
  if (!ws || ws_bytes < dam_mask_build_workspace(p)) return DAM_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const Geom g = geometry(p);
  const Workspace w = carve(p, ws);
  const uint8_t *dflag = diag_in, *vflag = vert_in;
  const uint64_t *true_bits = g.L > 0 ? o->true_bits : nullptr;
  CountArgs count{};

  if (p->mode == DAM_FROM_ATTN_MAP) {
    bool bmin_written;
    const Threshold thr = stage_threshold(p, g, w, attn_sum, attn_cnt, stream, o->bmin, &bmin_written);
    // a2: true mask, one comparison per element
    const bool in_prep = !attn_cnt && g.L <= kMapInPrep;
    dim3 grid((g.tbw + 3) / 4, (g.L + kTmRows - 1) / kTmRows, g.H);
    if (in_prep) {
    } else if (attn_cnt && p->transform == DAM_T_RAW_SUM)
      k_true_mask<false, true><<<grid, 256, 0, stream>>>(attn_sum, attn_cnt, g.L, g.tbw, p->eps, thr, o->true_bits);
    else if (attn_cnt)
      k_true_mask<false><<<grid, 256, 0, stream>>>(attn_sum, attn_cnt, g.L, g.tbw, p->eps, thr, o->true_bits);
    else if (g.L % 4 == 0 && (reinterpret_cast<uintptr_t>(attn_sum) & 15) == 0) {
      const int n_pairs = (((g.L + 1) / 2) + 3) / 4;
      const int per_map = std::max(1, std::min(n_pairs, kGridTarget / g.H));
      k_true_mask_rows<<<dim3(per_map, g.H), 256, 0, stream>>>(attn_sum, g.L, g.tbw, n_pairs, thr, o->true_bits);
    } else
      k_true_mask<true><<<grid, 256, 0, stream>>>(attn_sum, attn_cnt, g.L, g.tbw, p->eps, thr, o->true_bits);
    count = stage_patterns(p, g, w, o, stream, &dflag, &vflag, bmin_written, false, in_prep ? attn_sum : nullptr, thr);
  }
  stage_extension(p, g, w, o, true_bits, dflag, vflag, count, stream);
  return launch_status();
}

// Sec. 4.2.1 - 4.3 for one captured sequence, from its Q and K: the probabilities are thresholded
// as the capture kernels produce them (dam_capture.hip); the rest is the path above.
extern "C" size_t dam_mask_build_from_qk_workspace(const dam_mask_params *p, const dam_capture_params *cp) {
  const size_t base = dam_mask_build_workspace(p);
  if (!base || !cp || cp->hq < 1 || cp->pcl < 1) return 0;
  return base + capture_lse_bytes(cp);
}

extern "C" int dam_mask_build_from_qk(const dam_mask_params *p, const dam_capture_params *cp, const void *q,
                                      const void *k, const dam_mask_out *o, void *ws, size_t ws_bytes,
                                      void *stream_v) {
  if (!p || !o || !cp) return DAM_ERR_INVALID_ARG;
  if (p->mode != DAM_FROM_ATTN_MAP) return DAM_ERR_INVALID_ARG;
  const float dummy_map = 0.0f;  // validate() only checks that a map pointer is present
  int bad = validate(p, &dummy_map, nullptr, nullptr, o);
  if (bad != DAM_OK) return bad;
  bad = capture_validate(cp, q, k);
  if (bad != DAM_OK) return bad;
  if (p->n_maps != cp->hq || p->pcl != cp->pcl || cp->len != cp->pcl || p->pcl < 2) return DAM_ERR_INVALID_ARG;
  if (p->transform != DAM_T_BOXCOX) return DAM_ERR_UNSUPPORTED;  // the other transforms need statistics of the whole map
  if (!ws || ws_bytes < dam_mask_build_from_qk_workspace(p, cp)) return DAM_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const Geom g = geometry(p);
  const Workspace w = carve(p, ws);
  float *lse2 = reinterpret_cast<float *>(static_cast<char *>(ws) + w.bytes);
  const uint8_t *dflag = nullptr, *vflag = nullptr;
  bool bmin_written;
  // (one causal capture of two tokens or more: the minimum, and so the threshold, is known on the host)
  const Threshold thr = stage_threshold(p, g, w, nullptr, nullptr, stream, o->bmin, &bmin_written);
  const bool counted = launch_capture_true_bits(cp, q, k, lse2, thr.theta_val, thr.bmin_val, thr.bmin_out, o->true_bits,
                                                counts_in_prep(g) ? nullptr : w.vslices, w.dslices, stream);
  const CountArgs count = stage_patterns(p, g, w, o, stream, &dflag, &vflag, bmin_written, counted);
  stage_extension(p, g, w, o, o->true_bits, dflag, vflag, count, stream);
  return launch_status();
}

// The lists of one row as dam_mask_build makes them in one launch, without a look at the other workgroups' totals.
extern "C" int dam_probe_row_lists(const dam_mask_params *p, const uint8_t *diag_in, const uint8_t *vert_in, const dam_mask_out *o, void *ws,
                                   size_t ws_bytes, void *stream_v) {
  const int bad = validate(p, nullptr, diag_in, vert_in, o);
  if (bad != DAM_OK) return bad;
  if (!ws || ws_bytes < dam_mask_build_workspace(p)) return DAM_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const Geom g = geometry(p);
  if (p->mode != DAM_FROM_PATTERNS || !o->kept_ptr || (p->flags & DAM_MASK_PATTERN_PLAN) || p->row_end != p->row_begin + 1 ||
      !one_launch_lists(p, g))
    return DAM_ERR_UNSUPPORTED;
  launch_list_one(p, g, carve(p, ws), o, diag_in, vert_in, 0, stream);
  return launch_status();
}
