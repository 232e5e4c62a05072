// dam_capture_accumulate and the capture half of dam_mask_build_from_qk: full causal attention
// probabilities of a captured sequence, summed into the statistics A (and C) or thresholded on
// the fly into the true mask.
//
// Paper (arXiv 2506.11104): Sec. 4.2.1 (sequences truncated to the pattern capture length are run
// with full attention), Sec. 4.2.2 (the attention weights are summed over the captured batches and
// the valid position pairs are counted), Sec. 4.2.3 (threshold) for the fused form. The two-pass
// organisation and the kernels are this library's own.
//
// Both forms take two passes over the causal triangle of Q K^T: the first one reduces every row to
// its log-sum-exp (never materialising the logits), the second one recomputes the logits and turns
// them into probabilities p = exp2(s - lse). bf16 inputs with head_dim 128 run on the matrix
// cores: S^T = K Q^T with v_mfma_f32_32x32x16_bf16, so that the 16 accumulators of a lane belong
// to one query row and the row reductions are in-lane plus one exchange between the half-waves.
// Everything else (fp32 inputs, other head dims) goes through a plain one-row-per-workgroup kernel.
#include <hip/hip_bf16.h>
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "dam_internal.h"
#include "dam_slices.h"

namespace {
using namespace dam;

constexpr float kLog2e = 1.4426950408889634f;

struct CapArgs {
  int Hq, Hkv, n, L, d, tbw;
  int parts, chunk;  // matrix-core path: a row tile's stages of keys are shared by `parts` workgroups, `chunk` stages each
  unsigned theta_key;          // fused form: the threshold as an ordered key,
  float bmin, *out_bmin;       // and the minimum it was found against, stored by the second pass when wanted
  uint64_t *vslices, *dslices; // the patterns' chunk counts, when the second pass takes them
  float c2;  // scale * log2(e): logits in log2 units
  int64_t q_sh, q_ss, k_sh, k_ss;
};

// Ordered key of an fp32 value (increasing with the value; NaN counts as -inf): the form in which
// the true-mask threshold is handed over.
__device__ __forceinline__ unsigned key_of(float x) {
  if (x != x) x = -INFINITY;
  const unsigned b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

enum { kEmitBits = 0, kEmitSum = 1 };

// ================================================================================================
// Plain kernel: one workgroup per (row i, head h). The row's logits live in LDS between the
// reduction and the emission, so this kernel needs one pass only.
template <typename T>
__device__ __forceinline__ float dot_row(const float *__restrict__ qs, const T *__restrict__ krow, int d);

template <>
__device__ __forceinline__ float dot_row<float>(const float *__restrict__ qs, const float *__restrict__ krow, int d) {
  float acc = 0.0f;
  for (int t = 0; t < d; t += 4) {
    const float4 kv = *reinterpret_cast<const float4 *>(krow + t);
    acc = fmaf(qs[t], kv.x, acc);
    acc = fmaf(qs[t + 1], kv.y, acc);
    acc = fmaf(qs[t + 2], kv.z, acc);
    acc = fmaf(qs[t + 3], kv.w, acc);
  }
  return acc;
}

template <>
__device__ __forceinline__ float dot_row<__hip_bfloat16>(const float *__restrict__ qs, const __hip_bfloat16 *__restrict__ krow,
                                                         int d) {
  float acc = 0.0f;
  for (int t = 0; t < d; t += 8) {
    const uint4 kv = *reinterpret_cast<const uint4 *>(krow + t);
    const unsigned u[4] = {kv.x, kv.y, kv.z, kv.w};
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      acc = fmaf(qs[t + 2 * x], __uint_as_float(u[x] << 16), acc);
      acc = fmaf(qs[t + 2 * x + 1], __uint_as_float(u[x] & 0xFFFF0000u), acc);
    }
  }
  return acc;
}

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__hip_bfloat16 x) { return __bfloat162float(x); }

template <typename T, int MODE>
__global__ __launch_bounds__(256) void k_capture_rows(CapArgs a, const T *__restrict__ q, const T *__restrict__ k,
                                                      uint64_t *__restrict__ true_bits, float *__restrict__ attn_sum,
                                                      float *__restrict__ attn_cnt) {
  extern __shared__ float smem[];  // [d] query, then [i + 1] logits
  __shared__ float red[4];
  const int i = a.n - 1 - blockIdx.x, h = blockIdx.y;  // long rows first
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float *qs = smem, *sv = smem + a.d;
  const T *qrow = q + (int64_t)h * a.q_sh + (int64_t)i * a.q_ss;
  for (int t = threadIdx.x; t < a.d; t += 256) qs[t] = to_f32(qrow[t]);
  __syncthreads();
  const T *kh = k + (int64_t)(h / (a.Hq / a.Hkv)) * a.k_sh;
  float mx = -INFINITY;
  for (int j = threadIdx.x; j <= i; j += 256) {
    const float s = dot_row<T>(qs, kh + (int64_t)j * a.k_ss, a.d) * a.c2;
    sv[j] = s;
    mx = fmaxf(mx, s);
  }
  for (int off = 32; off; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sum = 0.0f;
  for (int j = threadIdx.x; j <= i; j += 256) sum += __builtin_amdgcn_exp2f(sv[j] - mx);
  for (int off = 32; off; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  sum = (red[0] + red[1]) + (red[2] + red[3]);
  const float lse2 = mx + __builtin_amdgcn_logf(sum);  // v_log_f32 is the base-2 logarithm
  if (MODE == kEmitBits) {
    const unsigned theta = a.theta_key;
    if (a.out_bmin && blockIdx.x == 0 && h == 0 && threadIdx.x == 0) *a.out_bmin = a.bmin;
    uint64_t *out = true_bits + ((int64_t)h * a.L + i) * a.tbw;
    for (int w = wave; w < a.tbw; w += 4) {
      const int j = w * 64 + lane;
      const bool keep = j <= i && key_of(__builtin_amdgcn_exp2f(sv[j <= i ? j : 0] - lse2)) >= theta;
      const uint64_t word = __ballot(keep);
      if (lane == 0) out[w] = word;
    }
  } else {
    float *arow = attn_sum + ((int64_t)h * a.L + i) * a.L;
    float *crow = attn_cnt ? attn_cnt + ((int64_t)h * a.L + i) * a.L : nullptr;
    for (int j = threadIdx.x; j <= i; j += 256) {
      arow[j] += __builtin_amdgcn_exp2f(sv[j] - lse2);
      if (crow) crow[j] += 1.0f;
    }
  }
}

// ================================================================================================
// Matrix-core kernels (bf16, head_dim 128). The two reducing passes: one workgroup of 4 waves per (head, tile of
// 128 query rows), each wave owning 32 rows; K moves through LDS in stages of 64 keys (16 KiB), double
// buffered, one barrier per stage. A K row is 16 chunks of 16 bytes; chunk c of row r is stored at
// position c ^ (r & 15), so that the 16-byte operand reads of 16 consecutive rows cover all banks.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int kRows = 128, kBlk = 32, kBlkBytes = kBlk * 256;
constexpr int kXcd = 8;
constexpr int kStageKeys = 64, kStageBytes = kStageKeys * 256;
constexpr int kMaxParts = 4;
constexpr int kPartTiles = 1024;  // row tiles times parts at most, where there is more than one part

// One wave's quarter of a stage as four load-to-LDS copies (lane L of the wave fetches 16 bytes from
// gbase + voff[it] and writes them to LDS byte lds_at + 4096 it + 16 L): rows wave * 4 + L / 16 + 16 it
// of the stage, whose chunk order the lane offsets already permute. Inline assembly, so that the
// compiler neither tracks nor counts the copies: the kernel waits for them itself (s_waitcnt vmcnt)
// before the barrier that publishes the stage. gbase and lds_at are wave-uniform.
__device__ __forceinline__ void k_copy_stage(unsigned lds_at, const void *gbase, const unsigned (&voff)[4]) {
#define DAM_CAP_COPY(IT)                                                               \
  asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"    \
               :                                                                         \
               : "s"(lds_at), "n"(4096 * (IT)), "v"(voff[IT]), "s"(gbase)                \
               : "memory", "scc", "m0")
  DAM_CAP_COPY(0);
  DAM_CAP_COPY(1);
  DAM_CAP_COPY(2);
  DAM_CAP_COPY(3);
#undef DAM_CAP_COPY
}

// Bits 0 .. 31 of a 32-key block starting at key0 that are causal for row i (key <= i).
__device__ __forceinline__ unsigned causal_bits(int i, int key0) {
  const int u = i - key0;
  return u >= 31 ? 0xFFFFFFFFu : (u < 0 ? 0u : ((2u << u) - 1u));
}

// Position, among the 32 keys of a block, of accumulator e of a lane of the lower half-wave.
__device__ __forceinline__ constexpr int key_of_acc(int e) { return 8 * (e / 4) + (e % 4); }

// Start value of a block's accumulators: 0 where the key is causal for this lane's row, -inf where
// it is not (the products add to it). `mine` = the causal bits already shifted by 4 hf.
__device__ __forceinline__ f32x16 causal_start(unsigned mine) {
  f32x16 s;
  const int inv = (int)~mine;
#pragma unroll
  for (int e = 0; e < 16; ++e)
    s[e] = __int_as_float(__builtin_amdgcn_sbfe(inv, key_of_acc(e), 1) & (int)0xFF800000u);
  return s;
}

template <int V>
struct IntC {
  static constexpr int value = V;
};

// Which (query head, item) a workgroup takes: workgroup g runs on XCD g % 8. Where the KV heads divide evenly among the
// XCDs, all query heads and items of one KV head stay on one of them, whose L2 then holds that head's K; otherwise (four
// KV heads: half the chip would stay empty) they go round robin. Items of a KV head are handed out in ascending order.
__device__ __forceinline__ void cap_numbering(const CapArgs &a, int items, int &h, int &item) {
  const int G = a.Hq / a.Hkv, per_kv = G * items;
  const bool even = a.Hkv % kXcd == 0;
  const int within = even ? blockIdx.x / kXcd % per_kv : blockIdx.x / a.Hkv;
  const int kv = even ? blockIdx.x / kXcd / per_kv * kXcd + blockIdx.x % kXcd : blockIdx.x % a.Hkv;
  h = kv * G + within % G;
  item = within / G;
}

// The log2-sum-exp of row i of head h from what the first pass left: of a row in one part the number itself, of a row in
// several (reference, sum) of every part, [part][head][L], with reference -inf where a part held no key of the row. (Not a
// log-sum-exp of every part: rounding those as well made the probabilities' error against 64 bits 6 % larger, 7.4e-7 for
// 7.0e-7 in the 2-norm over captures of 384 to 1936 tokens; this way it is
// 6.9e-7.)
__device__ __forceinline__ float row_lse(const CapArgs &a, const float *__restrict__ lse2, int h, int i) {
  const int64_t at = (int64_t)h * a.L + i;
  if (a.parts == 1) return lse2[at];
  const float2 *pair = reinterpret_cast<const float2 *>(lse2) + at;
  float2 v[kMaxParts];
  float M = -INFINITY, sum = 0.0f;
#pragma unroll
  for (int x = 0; x < kMaxParts; ++x) v[x] = x < a.parts ? pair[(int64_t)x * a.Hq * a.L] : make_float2(-INFINITY, 0.0f);
#pragma unroll
  for (int x = 0; x < kMaxParts; ++x) M = fmaxf(M, v[x].x);  // finite: part 0 holds key 0
#pragma unroll
  for (int x = 0; x < kMaxParts; ++x) sum += v[x].y * __builtin_amdgcn_exp2f(v[x].x - M);
  return M + __builtin_amdgcn_logf(sum);
}

// Emission of the summed form: probabilities p = exp2(logit * c2 - lse) of every causal pair, added to
// A (and 1 to C).
// Bound by the read-modify-write of A and C (16 bytes per pair against 256 flop), so the kernel is laid out for bytes in
// flight: a wave owns 32 rows x 64 keys and nothing else, fetches its part of A and C up front (16 KiB) behind the Q and K
// operands, which come from L2 straight in the products' layout (no LDS, no barrier), and stores when its products are
// done. The workgroup's waves lie side by side along the rows, 1 KiB of each (128 bytes per row and wave, spread over
// 128 rows, took twice the time). In the product S = Q K^T a lane holds one key of 16 rows, so a row's 32 keys are one
// 128-byte line across the lanes, whatever the row length. A row tile per workgroup with K staged through LDS had one
// block of A and C in flight and as many workgroups as row tiles (256 at 32 heads x 1000 tokens): 208 -> 81 us there
// with its first pass (3.8 TB/s of A and C without it), 64 heads x 4096 tokens 2150 -> 1740 us (5.3 TB/s).
// BLOCKS: 32-key blocks of a wave, two or one. Waves of 64 keys move more bytes for what they fetch besides, waves of 32 fit the
// chip three to a SIMD instead of two and come out more even where there are few (64 keys / 32, us, whole calls): 16 heads x 400
// tokens 22.7 / 17.7, 16 x 900 47.0 / 44.2, 32 x 1000 83.1 / 81.7, 32 x 1472 153.5 / 152.8, 64 x 2000 491 / 520.
constexpr int kSumNarrow = 6144;  // workgroups of 64 keys per wave up to which they get 32
constexpr int sum_span(int blocks) { return 4 * 32 * blocks; }  // keys of a workgroup's waves side by side: 1 KiB or 512 bytes of every row
// Workgroups of a head: rows come in groups of 32, and the groups of block R of a span's rows need R + 1 of them each.
__host__ __device__ constexpr int sum_items_before(int blocks, int R) { return 2 * blocks * R * (R + 1); }
// STREAM: non-temporal loads and stores. 5 to 10 % faster where a wave's 256 bytes of a row are whole 128-byte lines (A and
// C pass through once), twice as slow where they are not (the neighbour's half of a line then does not meet it in L2).
template <bool STREAM, int BLOCKS>
__global__ __launch_bounds__(256, BLOCKS == 1 ? 3 : 2) void k_capture_sum(CapArgs a, const __hip_bfloat16 *__restrict__ q,
                                                        const __hip_bfloat16 *__restrict__ k,
                                                        const float *__restrict__ lse2, float *__restrict__ attn_sum,
                                                        float *__restrict__ attn_cnt) {
  constexpr int kSpan = 4 * 32 * BLOCKS;
  auto before = [](int R) { return sum_items_before(BLOCKS, R); };
  int h, t;
  cap_numbering(a, before((a.n + kSpan - 1) / kSpan), h, t);
  int R = (int)((sqrtf((float)t * (2.0f / BLOCKS) + 1.0f) - 1.0f) * 0.5f);  // before(R) <= t
  while (before(R) > t) --R;
  while (before(R + 1) <= t) ++R;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hf = lane >> 5;
  const int within = t - before(R);
  const int row0 = R * kSpan + within / (R + 1) * 32, key0 = within % (R + 1) * kSpan + wave * 32 * BLOCKS;
  if (row0 >= a.n || key0 > row0 + 31) return;  // (whole waves) no row, or every key above the diagonal
  const int n_blk = min(BLOCKS, (row0 + 31 - key0) / 32 + 1);  // blocks of 32 keys that reach below the diagonal

  bf16x8 qf[8], kf[BLOCKS][8];
  const __hip_bfloat16 *qp = q + (int64_t)h * a.q_sh + (int64_t)min(row0 + n, a.n - 1) * a.q_ss + 8 * hf;
#pragma unroll
  for (int c = 0; c < 8; ++c) qf[c] = *reinterpret_cast<const bf16x8 *>(qp + 16 * c);
#pragma unroll
  for (int b = 0; b < BLOCKS; ++b) {
    const __hip_bfloat16 *kp =
        k + (int64_t)(h / (a.Hq / a.Hkv)) * a.k_sh + (int64_t)min(key0 + 32 * b + n, a.n - 1) * a.k_ss + 8 * hf;
    if (b < n_blk) {
#pragma unroll
      for (int c = 0; c < 8; ++c) kf[b][c] = *reinterpret_cast<const bf16x8 *>(kp + 16 * c);
    }
  }
  // accumulator e is row 8 (e / 4) + 4 hf + e % 4 of the wave with key n of the block
  auto row_of = [&](int e) { return 8 * (e >> 2) + 4 * hf + (e & 3); };
  float lse[16];
  const float lse_n = row_lse(a, lse2, h, min(row0 + n, a.n - 1));
#pragma unroll
  for (int e = 0; e < 16; ++e) lse[e] = __shfl(lse_n, row_of(e));
  const int64_t at0 = ((int64_t)h * a.L + row0) * a.L + key0;  // of row row0, key key0
  // (one lane offset for every element: the row of an element differs by a wave-uniform step)
  const int lane_at = 4 * hf * a.L + n;
  auto take = [](const float *p) { return STREAM ? __builtin_nontemporal_load(p) : *p; };
  auto put = [](float v, float *p) {
    if (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
  };
  // (inside: every pair of the tile is causal and exists, so nothing is tested)
  auto body = [&](auto inside) {
    float av[BLOCKS][16], cv[BLOCKS][16];
    auto wanted = [&](int b, int e) {
      return decltype(inside)::value || (row0 + row_of(e) < a.n && key0 + 32 * b + n <= row0 + row_of(e));
    };
    auto each = [&](auto f) {
#pragma unroll
      for (int b = 0; b < BLOCKS; ++b)
        if (b < n_blk) {
#pragma unroll
          for (int e = 0; e < 16; ++e) f(b, e, at0 + (int64_t)(8 * (e >> 2) + (e & 3)) * a.L + 32 * b);
        }
    };
    each([&](int b, int e, int64_t at) { av[b][e] = wanted(b, e) ? take(attn_sum + at + lane_at) : 0.0f; });
    if (attn_cnt) each([&](int b, int e, int64_t at) { cv[b][e] = wanted(b, e) ? take(attn_cnt + at + lane_at) : 0.0f; });
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b)
      if (b < n_blk) {
        f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 8; ++c) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[c], kf[b][c], s, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e) av[b][e] += __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], a.c2, -lse[e]));
      }
    each([&](int b, int e, int64_t at) {
      if (wanted(b, e)) put(av[b][e], attn_sum + at + lane_at);
    });
    if (attn_cnt)
      each([&](int b, int e, int64_t at) {
        if (wanted(b, e)) put(cv[b][e] + 1.0f, attn_cnt + at + lane_at);
      });
  };
  if (row0 + 31 < a.n && key0 + 32 * BLOCKS - 1 <= row0) body(std::true_type{});
  else body(std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// Pipelined form of the two passes that emit no probabilities: PASS 0 reduces every row to its
// log-sum-exp, PASS 1 compares every logit with the row's threshold and packs the true-mask bits.
// A wave works on its blocks of 32 keys one after the other (block g: keys 32 g .. 32 g + 31, in
// half g & 1 of LDS buffer (g >> 1) & 1, i.e. at byte (g & 3) * 8 KiB); in step g it issues
//   the eight products of block g + 1 (one dependent chain into the other accumulator set),
//   the vector work on the finished logits of block g, cut into eight slices that sit between
//     the products (the wave issues in order: what stands between two products of a chain runs
//     in the shadow of the first),
//   the operand reads of block g + 2, each into the registers its product has just consumed.
// So the operands run two blocks ahead of the vector work, and a stage of 64 keys must be resident
// one stage before its first product: the rows of stage st + 2 are copied (load-to-LDS) during stage st
// into the buffer of stage st itself, which no wave reads then: the operand reads of a stage all fall
// into the stage before it. One barrier per stage.
template <int PASS>
__global__ __launch_bounds__(256) void k_capture_pipe(CapArgs a, const __hip_bfloat16 *__restrict__ q,
                                                      const __hip_bfloat16 *__restrict__ k, float *__restrict__ lse2,
                                                      uint64_t *__restrict__ true_bits) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kStageBytes];
  const int nQt = (a.n + kRows - 1) / kRows;
  int h, item;
  cap_numbering(a, nQt * a.parts, h, item);
  const int qt = nQt - 1 - item / a.parts, part = item % a.parts, kv = h / (a.Hq / a.Hkv);  // the long rows first
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 31, hf = lane >> 5;
  const int wave_first = qt * kRows + wave * 32;
  const int i = wave_first + n;  // this lane's query row
  const bool live = i < a.n;
  const int kbase = n * 256 + ((hf ^ (n & 15)) << 4);
  const unsigned char *kaddr[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) kaddr[c] = lds + (kbase ^ (c << 5));
  // K rows reach LDS by load-to-LDS copies: thread t brings piece (t & 15) ^ (row & 15) of row
  // t >> 4 (+ 16 per copy) of a stage to position t & 15 of that row. Rows past the sequence end are
  // redirected to the last row (such keys are masked by causality anyway).
  // (everything below counts stages, blocks and keys from this part's first stage, an even one)
  const int key_first = part * a.chunk * kStageKeys, n_keys = a.n - key_first, i_rel = i - key_first;
  const char *kh = reinterpret_cast<const char *>(k + (int64_t)kv * a.k_sh + (int64_t)key_first * a.k_ss);
  const int64_t row_bytes = a.k_ss * 2;
  const int srow = threadIdx.x >> 4;
  const unsigned piece = (((threadIdx.x & 15) ^ (srow & 15)) << 4);
  unsigned voff_full[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) voff_full[it] = (unsigned)((srow + 16 * it) * row_bytes) + piece;
  const unsigned lds_mine =
      __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)lds + wave * 1024);
  auto copy_stage = [&](int st, int buf) {
    const int key0 = st * kStageKeys;
    const char *gbase = kh + (int64_t)key0 * row_bytes;
    if (key0 + kStageKeys <= n_keys) {  // workgroup-uniform
      k_copy_stage(lds_mine + buf * kStageBytes, gbase, voff_full);
    } else {
      unsigned voff[4];
#pragma unroll
      for (int it = 0; it < 4; ++it) voff[it] = (unsigned)(min(srow + 16 * it, n_keys - 1 - key0) * row_bytes) + piece;
      k_copy_stage(lds_mine + buf * kStageBytes, gbase, voff);
    }
  };

  bf16x8 qf[8];
  {
    const __hip_bfloat16 *qp = q + (int64_t)h * a.q_sh + (int64_t)i * a.q_ss + 8 * hf;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4 raw = {0u, 0u, 0u, 0u};
      if (live) raw = *reinterpret_cast<const u32x4 *>(qp + 16 * c);
      qf[c] = __builtin_bit_cast(bf16x8, raw);
    }
  }
  const int last_row = min(qt * kRows + kRows - 1, a.n - 1);
  const int word_first = 2 * part * a.chunk;
  // the words up to the next part's, or to the end of the row
  const int nw32 = part == a.parts - 1 ? a.tbw * 2 - word_first : min(a.tbw * 2 - word_first, 2 * a.chunk);
  // the tile's words of this part from word w_done on (keys above the diagonal): all zero; written by the whole
  // workgroup, 16 bytes per thread along a row
  auto clear_words = [&](int w_done) {
    const int rest = nw32 - w_done;
    if (rest <= 0) return;
    const int rows = min(kRows, a.n - qt * kRows), per_row = (rest + 3) / 4;
    unsigned *tile_out = reinterpret_cast<unsigned *>(true_bits + ((int64_t)h * a.L + qt * kRows) * a.tbw) + word_first;
    for (int x = threadIdx.x; x < rows * per_row; x += 256) {
      const int r = x / per_row, w = w_done + 4 * (x % per_row);
      unsigned *dst = tile_out + (int64_t)r * (2 * a.tbw) + w;
      if (w + 3 < nw32 && (a.tbw & 1) == 0) {
        *reinterpret_cast<uint4 *>(dst) = make_uint4(0u, 0u, 0u, 0u);
      } else {
        for (int y = 0; y < 4 && w + y < nw32; ++y) dst[y] = 0u;
      }
    }
  };
  float2 *my_pair = reinterpret_cast<float2 *>(lse2) + ((int64_t)part * a.Hq + h) * a.L + i;  // (several parts; row_lse)
  if (key_first > last_row) {  // no key of this part lies below the tile's diagonal
    if (PASS == 1) clear_words(0);
    else if (live && hf == 0) *my_pair = make_float2(-INFINITY, 0.0f);
    return;
  }
  // this part's stages, of those that hold a key <= the tile's last live row. (In this form, quotient plus one: with the
  // equal min(stages - first, chunk) the compiler takes 202 registers instead of 142, and a wave per SIMD less fits.)
  const int n_stage = (unsigned)min(last_row - key_first, a.chunk * kStageKeys - 1) / kStageKeys + 1;
  const int diag_g = qt * 4 + wave - 2 * part * a.chunk;  // the wave's last block: the one the diagonal crosses
  // blocks 0 .. n_blocks - 1 hold a key <= a row of the wave (a wave with a live row needs no more than the stages hold)
  const int n_blocks = min(diag_g + 1, 2 * a.chunk);

  // PASS 0 state: reference m_ref (log2 units; moves only when a maximum outgrows it by more than 8,
  // so that the sum rarely has to be rescaled) and the sum of exp2(t - m_ref) over this lane's keys
  float m_ref = -INFINITY, l_run = 0.0f;
  // PASS 1: p >= theta  <=>  raw logit >= (lse + log2 theta) / c2 up to rounding. The threshold arrives as an
  // ordered key: 0 keeps every causal entry, all ones keeps none; so do theta <= 0 and theta = +inf.
  float thr = 0.0f;
  if (PASS == 1) {
    const float my_lse = live ? row_lse(a, lse2, h, i) : 0.0f;
    const unsigned tk = a.theta_key;
    if (a.out_bmin && blockIdx.x == 0 && threadIdx.x == 0) *a.out_bmin = a.bmin;
    const float theta = __uint_as_float((tk & 0x80000000u) ? (tk & 0x7FFFFFFFu) : ~tk);
    if (tk == 0u || theta <= 0.0f) thr = -INFINITY;
    else if (tk == 0xFFFFFFFFu || !(theta < INFINITY)) thr = INFINITY;
    else thr = (my_lse + __builtin_amdgcn_logf(theta)) / a.c2;
  }
  unsigned words[4] = {0u, 0u, 0u, 0u};  // bits of the current 128-key group of this lane's row
  unsigned *out32 = reinterpret_cast<unsigned *>(true_bits + ((int64_t)h * a.L + (live ? i : 0)) * a.tbw) + word_first;
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 S0 = zero, S1 = zero;  // logits of the even / odd blocks
  bf16x8 kf[8];                 // operands of the next chain

  // ---- vector work of one block, in slices -------------------------------------------------------
  float blk_off = 0.0f, add0 = 0.0f, add1 = 0.0f;   // PASS 0, between the slices of a block
  unsigned neg = 0u;                                // PASS 1
  // PASS 0, first part: the block's maximum decides whether the reference moves
  auto ref_update = [&](const f32x16 &s) {
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; e += 2) mx = fmaxf(fmaxf(s[e], s[e + 1]), mx);
    mx *= a.c2;  // c2 > 0
    const bool move = mx - m_ref > 8.0f;  // false while both are -inf (NaN)
    if (__ballot(move)) {
      if (move) {
        l_run *= __builtin_amdgcn_exp2f(m_ref - mx);  // m_ref = -inf: 0
        m_ref = mx;
      }
    }
    blk_off = m_ref == -INFINITY ? 0.0f : m_ref;
    add0 = add1 = 0.0f;
  };
  // elements e0 .. e1 - 1 of a block
  auto slice = [&](const f32x16 &s, auto e0c, auto e1c) {
    constexpr int E0 = decltype(e0c)::value, E1 = decltype(e1c)::value;
    if (PASS == 0) {
#pragma unroll
      for (int e = E0; e < E1; ++e) {
        const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], a.c2, -blk_off));
        if (e & 1) add1 += w;
        else add0 += w;
      }
    } else {
      // logit >= thr <=> the difference is not negative: the sign bits are shifted into a word one
      // by one, the last accumulator first, so that accumulator e ends at bit e
#pragma unroll
      for (int e = E0; e < E1; ++e)
        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(s[15 - e] - thr), 31);
    }
  };
  auto finish = [&](auto g4c, int g) {
    constexpr int G4 = decltype(g4c)::value;
    if (PASS == 0) {
      l_run += add0 + add1;
    } else {
      // the four nibbles go to the key positions of a lower half-wave lane and are inverted
      unsigned v = neg & 0xFFFFu;
      v = (v | (v << 8)) & 0x00FF00FFu;
      v = (v | (v << 4)) & 0x0F0F0F0Fu;
      unsigned mine = (v ^ 0x0F0F0F0Fu) << (4 * hf);
      mine |= (unsigned)__shfl_xor((int)mine, 32);
      if (g == diag_g) mine &= causal_bits(i_rel, g * kBlk);  // wave-uniform
      words[G4] = mine;
    }
  };

  // ---- one step -----------------------------------------------------------------------------------
  // G4 = g & 3. cur = logits of block g, nxt = accumulators of block g + 1.
  auto step = [&](auto g4c, int g) {
    constexpr int G4 = decltype(g4c)::value;
    constexpr int OFF2 = ((G4 + 2) & 3) * kBlkBytes;  // where block g + 2 lies
    f32x16 &cur = (G4 & 1) ? S1 : S0;
    f32x16 &nxt = (G4 & 1) ? S0 : S1;
    if (g >= 0 && g + 2 < n_blocks) {
      // steady state: neither block g nor block g + 1 touches the diagonal
#define DAM_CAP_SEG(C, VALU)                                                                       \
  nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[C], qf[C], (C) == 0 ? zero : nxt, 0, 0, 0);      \
  kf[C] = *reinterpret_cast<const bf16x8 *>(kaddr[C] + OFF2);                                       \
  VALU;                                                                                             \
  __builtin_amdgcn_sched_barrier(0);
      if (PASS == 0) {
        // the maximum first (it needs every logit); its instructions are short and stay in front
        ref_update(cur);
        __builtin_amdgcn_sched_barrier(0);
        DAM_CAP_SEG(0, slice(cur, IntC<0>{}, IntC<2>{}))
        DAM_CAP_SEG(1, slice(cur, IntC<2>{}, IntC<4>{}))
        DAM_CAP_SEG(2, slice(cur, IntC<4>{}, IntC<6>{}))
        DAM_CAP_SEG(3, slice(cur, IntC<6>{}, IntC<8>{}))
        DAM_CAP_SEG(4, slice(cur, IntC<8>{}, IntC<10>{}))
        DAM_CAP_SEG(5, slice(cur, IntC<10>{}, IntC<12>{}))
        DAM_CAP_SEG(6, slice(cur, IntC<12>{}, IntC<14>{}))
        DAM_CAP_SEG(7, slice(cur, IntC<14>{}, IntC<16>{}))
      } else {
        DAM_CAP_SEG(0, slice(cur, IntC<0>{}, IntC<2>{}))
        DAM_CAP_SEG(1, slice(cur, IntC<2>{}, IntC<4>{}))
        DAM_CAP_SEG(2, slice(cur, IntC<4>{}, IntC<6>{}))
        DAM_CAP_SEG(3, slice(cur, IntC<6>{}, IntC<8>{}))
        DAM_CAP_SEG(4, slice(cur, IntC<8>{}, IntC<10>{}))
        DAM_CAP_SEG(5, slice(cur, IntC<10>{}, IntC<12>{}))
        DAM_CAP_SEG(6, slice(cur, IntC<12>{}, IntC<14>{}))
        DAM_CAP_SEG(7, slice(cur, IntC<14>{}, IntC<16>{}))
      }
#undef DAM_CAP_SEG
      finish(g4c, g);
      return;
    }
    // the first step (g = -1: only the chain of block 0) and the last ones of the wave
    const bool do_chain = g + 1 < n_blocks, do_read = g + 2 < n_blocks, do_valu = g >= 0 && g < n_blocks;
    if (do_chain) {
      // entries above the diagonal start from -inf, so that the products leave them there
      f32x16 acc = zero;
      if (PASS == 0 && g + 1 == diag_g) acc = causal_start(causal_bits(i_rel, (g + 1) * kBlk) >> (4 * hf));
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c], qf[c], acc, 0, 0, 0);
        if (do_read) kf[c] = *reinterpret_cast<const bf16x8 *>(kaddr[c] + OFF2);
      }
      nxt = acc;
    }
    if (do_valu) {
      if (PASS == 0) ref_update(cur);
      slice(cur, IntC<0>{}, IntC<16>{});
      finish(g4c, g);
    }
  };

  // One stage of 64 keys (st & 1 = B): the steps of its two blocks; the rows of stage st + 2 travel
  // through registers meanwhile and replace this stage's, which nobody reads any more.
  auto stage = [&](auto bc, int st) {
    constexpr int B = decltype(bc)::value;
    const bool more2 = st + 2 < n_stage;
    if (more2) copy_stage(st + 2, B);
    step(IntC<2 * B>{}, 2 * st);
    step(IntC<2 * B + 1>{}, 2 * st + 1);
    // this wave's copies have landed (and the bit stores of the group before: a whole stage old)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (PASS == 1 && (B == 1 || st + 1 >= n_stage)) {
      // the 128-key group is complete (blocks above this wave's rows contributed zeros)
      if (live && hf == 0) {
        const int w0 = (st >> 1) * 4;
        if (w0 + 3 < nw32 && (a.tbw & 1) == 0) {
          *reinterpret_cast<uint4 *>(out32 + w0) = make_uint4(words[0], words[1], words[2], words[3]);
        } else {
#pragma unroll
          for (int x = 0; x < 4; ++x)
            if (w0 + x < nw32) out32[w0 + x] = words[x];
        }
      }
      words[0] = words[1] = words[2] = words[3] = 0u;
    }
    __syncthreads();
  };

  copy_stage(0, 0);
  if (n_stage > 1) copy_stage(1, 1);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 8; ++c) kf[c] = *reinterpret_cast<const bf16x8 *>(kaddr[c]);
  step(IntC<3>{}, -1);
  __syncthreads();  // buffer 0 is rewritten at the end of stage 0: every wave has read block 0 and 1 by now
  for (int st = 0; st < n_stage; st += 2) {
    stage(IntC<0>{}, st);
    if (st + 1 < n_stage) stage(IntC<1>{}, st + 1);  // workgroup-uniform
  }
  if (PASS == 0) {
    const float m_o = __shfl_xor(m_ref, 32), l_o = __shfl_xor(l_run, 32);
    // M = -inf: no key of the row in this part, and the sums are zero; or no logit above -inf, and a NaN among the logits
    // is in the sums. A part must hand that on; a row in one part has no log-sum-exp then (NaN).
    const float M = fmaxf(m_ref, m_o), ref = M == -INFINITY && a.parts > 1 ? 0.0f : M;
    const float tot = l_run * __builtin_amdgcn_exp2f(m_ref - ref) + l_o * __builtin_amdgcn_exp2f(m_o - ref);
    if (live && hf == 0) {
      if (a.parts == 1) lse2[(int64_t)h * a.L + i] = M + __builtin_amdgcn_logf(tot);
      else *my_pair = make_float2(M, tot);
    }
  } else {
    clear_words(((n_stage + 1) / 2) * 4);
    if (a.vslices) {
      // The tile's 128 rows are one chunk of the pattern counts: counted here, where its words come out of L2 and other
      // workgroups' products run meanwhile. (64 heads x 4096 tokens, whole call: 342 us with the counts in a launch of 56 us,
      // 321 with the launch as it is now, 316 so.)
      __syncthreads();
      const int64_t at = ((int64_t)h * nQt + qt) * kSlices * a.tbw;
      count_chunk(true_bits + ((int64_t)h * a.L + qt * kRows) * a.tbw, min(kRows, a.n - qt * kRows), a.tbw, qt,
                  reinterpret_cast<uint64_t *>(lds), a.vslices + at, a.dslices + at);
    }
  }
}
static_assert(kRows == kChunkRows && kSliceLds <= 2 * kStageBytes, "a row tile is a chunk, counted in the LDS of its stages");

bool mfma_path(const dam_capture_params *p) { return p->dtype == DAM_BF16 && p->head_dim == 128; }

CapArgs make_args(const dam_capture_params *p) {
  CapArgs a;
  a.Hq = p->hq; a.Hkv = p->hkv; a.n = p->len; a.L = p->pcl; a.d = p->head_dim;
  a.tbw = (p->pcl + 63) / 64;
  a.c2 = (p->scale > 0.0f ? p->scale : 1.0f / sqrtf((float)p->head_dim)) * kLog2e;
  a.q_sh = p->q_stride[0]; a.q_ss = p->q_stride[1];
  a.k_sh = p->k_stride[0]; a.k_ss = p->k_stride[1];
  a.theta_key = 0;
  a.bmin = 0.0f;
  a.out_bmin = nullptr;
  a.vslices = a.dslices = nullptr;
  a.parts = 1;
  a.chunk = 0;
  if (mfma_path(p)) {
    // A workgroup walks its row tile's stages one after the other, about a microsecond each: while the row tiles alone
    // leave the chip (three workgroups per CU) with room, up to four workgroups share a tile's stages, an even number
    // each. 32 heads x 1000 tokens, first pass: 18 -> 12 us.
    const int n_stage = (p->len + kStageKeys - 1) / kStageKeys, tiles = p->hq * ((p->len + kRows - 1) / kRows);
    const int parts = std::max(1, std::min(kMaxParts, kPartTiles / tiles));
    a.chunk = ((n_stage + parts - 1) / parts + 1) / 2 * 2;
    a.parts = (n_stage + a.chunk - 1) / a.chunk;
  }
  return a;
}

template <int MODE>
void launch(const dam_capture_params *p, const CapArgs &a, const void *q, const void *k, float *lse2, uint64_t *true_bits,
            float *attn_sum, float *attn_cnt, hipStream_t st) {
  if (mfma_path(p)) {
    const int nQt = (a.n + kRows - 1) / kRows;
    const int grid = a.Hq * nQt * a.parts;
    const __hip_bfloat16 *qb = static_cast<const __hip_bfloat16 *>(q), *kb = static_cast<const __hip_bfloat16 *>(k);
    k_capture_pipe<0><<<grid, 256, 0, st>>>(a, qb, kb, lse2, true_bits);
    if (MODE == kEmitBits) k_capture_pipe<1><<<grid, 256, 0, st>>>(a, qb, kb, lse2, true_bits);
    else {
      const bool whole_lines = ((a.L * 4) | (int)(reinterpret_cast<uintptr_t>(attn_sum) | reinterpret_cast<uintptr_t>(attn_cnt))) % 128 == 0;
      auto groups = [&](int blocks) { return a.Hq * sum_items_before(blocks, (a.n + sum_span(blocks) - 1) / sum_span(blocks)); };
      const int blocks = groups(2) <= kSumNarrow ? 1 : 2;
      auto kern = blocks == 1 ? (whole_lines ? k_capture_sum<true, 1> : k_capture_sum<false, 1>)
                              : (whole_lines ? k_capture_sum<true, 2> : k_capture_sum<false, 2>);
      kern<<<groups(blocks), 256, 0, st>>>(a, qb, kb, lse2, attn_sum, attn_cnt);
    }
    return;
  }
  const dim3 grid(a.n, a.Hq);
  const size_t lds = (size_t)(a.d + a.n) * sizeof(float);
  if (p->dtype == DAM_BF16)
    k_capture_rows<__hip_bfloat16, MODE><<<grid, 256, lds, st>>>(a, static_cast<const __hip_bfloat16 *>(q),
                                                                static_cast<const __hip_bfloat16 *>(k), true_bits,
                                                                attn_sum, attn_cnt);
  else
    k_capture_rows<float, MODE><<<grid, 256, lds, st>>>(a, static_cast<const float *>(q), static_cast<const float *>(k),
                                                       true_bits, attn_sum, attn_cnt);
}

}  // namespace

namespace dam {

int capture_validate(const dam_capture_params *p, const void *q, const void *k) {
  if (!p || !q || !k) return DAM_ERR_INVALID_ARG;
  if (p->hq < 1 || p->hkv < 1 || p->hq % p->hkv || p->len < 1 || p->pcl < p->len) return DAM_ERR_INVALID_ARG;
  if (p->dtype != DAM_F32 && p->dtype != DAM_BF16) return DAM_ERR_UNSUPPORTED;
  if (p->head_dim < 8 || p->head_dim > 256 || p->head_dim % 8) return DAM_ERR_UNSUPPORTED;
  if (p->pcl > 8192) return DAM_ERR_UNSUPPORTED;  // a row's logits stay in LDS in the plain kernel
  if (p->k_stride[1] >= (1 << 24)) return DAM_ERR_UNSUPPORTED;  // byte offsets inside a stage of 64 rows are 32-bit
  if (!(p->scale >= 0.0f)) return DAM_ERR_INVALID_ARG;
  const int align = p->dtype == DAM_BF16 ? 8 : 4;  // elements per 16 bytes
  const int64_t strides[] = {p->q_stride[0], p->q_stride[1], p->k_stride[0], p->k_stride[1]};
  for (int64_t s : strides)
    if (s < 0 || s % align) return DAM_ERR_INVALID_ARG;
  return DAM_OK;
}

// By the size of the statistics alone, whatever the length of the sequence: a caller sizes one workspace for several. A
// sequence is cut into the more parts the fewer row tiles it has, so this is what one row tile per head could take.
size_t capture_lse_bytes(const dam_capture_params *p) {
  const int most_parts = mfma_path(p) ? std::max(1, std::min(kMaxParts, kPartTiles / p->hq)) : 1;
  const size_t row_bytes = most_parts > 1 ? most_parts * sizeof(float2) : sizeof(float);
  return align_up(row_bytes * p->hq * (size_t)p->pcl, 256);
}

bool launch_capture_true_bits(const dam_capture_params *p, const void *q, const void *k, float *lse2,
                              unsigned theta_key, float bmin, float *out_bmin, uint64_t *true_bits, uint64_t *vslices,
                              uint64_t *dslices, hipStream_t st) {
  CapArgs a = make_args(p);
  a.theta_key = theta_key;
  a.bmin = bmin;
  a.out_bmin = out_bmin;
  const bool counts = vslices && mfma_path(p) && a.parts == 1 && p->len == p->pcl;  // (no workgroup has whole rows otherwise)
  if (counts) {
    a.vslices = vslices;
    a.dslices = dslices;
  }
  launch<kEmitBits>(p, a, q, k, lse2, true_bits, nullptr, nullptr, st);
  return counts;
}

}  // namespace dam

extern "C" size_t dam_capture_workspace(const dam_capture_params *p) {
  if (!p || p->hq < 1 || p->pcl < 1) return 0;
  return dam::capture_lse_bytes(p);
}

extern "C" int dam_capture_accumulate(const dam_capture_params *p, const void *q, const void *k, float *attn_sum,
                                      float *attn_cnt, void *ws, size_t ws_bytes, void *stream_v) {
  const int bad = dam::capture_validate(p, q, k);
  if (bad != DAM_OK) return bad;
  if (!attn_sum) return DAM_ERR_INVALID_ARG;
  if (!ws || ws_bytes < dam_capture_workspace(p)) return DAM_ERR_WORKSPACE;
  launch<kEmitSum>(p, make_args(p), q, k, static_cast<float *>(ws), nullptr, attn_sum, attn_cnt,
                   static_cast<hipStream_t>(stream_v));
  return dam::launch_status();
}
