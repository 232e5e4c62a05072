// dam_sparse_attn_prefill: masked causal self-attention evaluated only inside the listed tiles.
//
// Paper (arXiv 2506.11104): Sec. 3 (S = Q K^T / sqrt(d_k), softmax, O = A V) with the per-head mask
// of Sec. 4.3 applied as -inf before the softmax. The tiling, the online softmax and the use of
// the block index are this library's own.
//
// bf16 kernel (head_dim 128, tiles 128 x 128), one workgroup of 4 waves per (head, query tile),
// each wave owning 32 query rows:
//   S^T = K Q^T on v_mfma_f32_32x32x16_bf16 (A = K rows from LDS, B = Q rows held in registers).
//     In the transposed product a lane's 64 accumulators all belong to ONE query, so the row max
//     and row sum of the online softmax are in-lane reductions plus a single exchange between the
//     two half-waves.
//   O^T += V^T P^T on the same instruction: the accumulator layout of S^T is, up to a fixed
//     permutation of each 16-key group, already the B-operand layout, so P never leaves
//     registers; V stays row-major in LDS and its transposed A operand comes from the
//     transposing LDS read (ds_read_b64_tr_b16), addressed with the same permutation.
//   The unit of work is a block of 32 keys (an occupied key quarter of a listed tile). K / V blocks
//     move through two LDS rings of four slots filled by load-to-LDS instructions (no registers in
//     between), three blocks ahead of their use; one barrier per block. Within a wave the products
//     of three consecutive blocks are interleaved with the softmax arithmetic (see the kernel).
//     The blocks of a query tile are listed in LDS first (its tiles expanded 128 at a time by the whole
//     workgroup), so that an iteration reads one descriptor instead of walking tiles in scalar code.
//   Tiles not in the block index are never touched, key quarters of a tile without a kept entry are
//     never loaded, and full tiles skip the element mask.
// fp32 kernel (the 1e-4 variant): v_mfma_f32_16x16x4_f32, 16 query rows per workgroup, blocks of 16 keys.
#include <hip/hip_bf16.h>
#include <math.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "dam_blocks.h"
#include "dam_internal.h"
#include "dam_mfma.h"

namespace {
using namespace dam;

constexpr int kXcd = 8;
// control words at the start of the bf16 kernel's workspace: the eight queue counters
// The words lie 256 bytes apart: atomics on one line are served one after the other, and everything else that memory
// channel holds waits behind them. (With the counters side by side and every finished workgroup trying all of them, the
// workgroups still at work took up to 9 us for an iteration of 0.7: 2000 tokens, 32 heads.)
constexpr int kCtlStep = 64, kCtlWords = kXcd, kCtlBytes = kCtlWords * kCtlStep * 4;

// Longest queue whose items are put into order of their length (order_items): eight items per workgroup, 64 of them on an
// XCD. Longer queues stay in the order of their numbers: by length neighbours in time no longer share windows of K and V, which
// with 16 items per workgroup (32 heads x 32768 tokens) costs 1 % and more than the ends, even already, give back.
constexpr int kOrderMax = 512;

struct AttnArgs {
  int B, Hq, Hkv, S, nQt, nKt, tile_m, tile_n, wpr;
  int gather_rows, gather_stride;  // gathered column tiles (tile index >= nKt), 0 when the index has none
  float scale;
  int64_t q_sb, q_sh, q_ss, k_sb, k_sh, k_ss, v_sb, v_sh, v_ss, o_sb, o_sh, o_ss;
};

// ================================================================================================
// fp32 variant, on v_mfma_f32_16x16x4_f32 (fp32 products and sums: the matrix instruction rounds like a chain of
// fused multiply-adds).
//
// A workgroup takes 16 query rows of a query tile; its four waves share the rows' occupied blocks of 16 keys and are
// merged through LDS at the end. Sixteen rows, not the whole tile, because a row's keys form one dependent chain and
// the fp32 problems are small: 16-row groups times four waves are what fills 256 CUs (2 x 8 heads of 1500 rows are
// 1504 groups), and a 16 x 16 block is the finest square the mask can be skipped at.
// Both products keep a lane on one query (lane % 16): S^T = K Q^T leaves key 4 (lane / 16) + r in accumulator r, and
// that is the B operand of step r of O^T += V^T P^T when the lanes of group g fetch V row 4 g + r, so P stays in
// registers. The dims are dealt out so that every operand is a 16-byte load straight from memory in the product's
// layout: K and Q lane (row, g) holds dims 16 c + 4 g .. + 3 of chunk c, V lane m dims 64 h + 4 m .. + 3. What an iteration
// has used of its block's K and V rows is replaced at once by that part of the wave's next block.
// A wave has three blocks on average in the size below, so the time is as much the list in front of them (4 us, a chain of
// loads) and the first block's loads as the products: the matrix rate (64 flop per cycle and SIMD) is used to about 30 % on the
// blocks that are issued, each of which brings 16 KiB of K and V from L2 however few of its entries are kept. 2 sequences x 8
// heads x 1500 keys, d 128, windows and stripes (46 % of the issued entries kept) 46.2 us; 55.7 with V fetched in front of its
// own block's Q K products and two workgroups on a CU, 51.4 with the fetches as they are (1 x 4 x 300 12.8 -> 11.7). That form
// before it: 391 -> 60 us against a row per d / 4 plain lanes, each visiting its kept keys only. At the same size
// a window of 64 101 -> 34 us; where nothing but isolated diagonals is kept (9 to 14 entries per block) the plain lanes
// were faster, 1 % of the diagonals 50 -> 63 us, 4 % 92 -> 114, 10 % 176 -> 130.
constexpr int kF32Seg = 64;  // listed tiles expanded at a time

// GATHER: the block index may hold gathered column tiles, whose key rows are looked up in gather_idx. (A template
// argument, because the look-up in front of every row's address makes the loads of a block wait for each other.)
//
// ODD: for row groups whose V holds an infinity or a NaN in a block that they visit. It must reach the rows that keep that key and
// no others, and a product would multiply it with the others' zero weights, so such a block's kept entries are added one by one.
// The first form (ODD = false) only notices; the workgroup then takes its rows again through the second, a function of its own:
// with both ways behind a branch of the loop the kernel holds 242 registers instead of 168, two workgroups on a CU instead of three.
struct F32Args {
  AttnArgs a;
  const float *q, *k, *v;
  const int *row_ptr, *blk_col;
  const uint8_t *blk_kind;
  const uint64_t *tile_bits;
  const int *gather_idx;
  float *out, *lse;
};
template <int D>
struct F32Lds {
  // one LDS area, two lives: mask words, columns and block list of a segment of tiles; then the waves' partial results
  struct Lists {
    unsigned words[kF32Seg][64];  // [tile][32-key word g * 16 + row]
    int col[kF32Seg];
    unsigned char occ[kF32Seg];   // bit kb: block kb of the tile holds a kept entry of these rows
    unsigned short blk[kF32Seg * 8];
  };
  struct Parts {
    float o[4][16 * (D + 4)];  // (rows padded: 16 rows, 16 different banks)
    float m[4][16], l[4][16];
    unsigned any[4][16];
    int odd[4];
  };
  static constexpr size_t kBytes = sizeof(Lists) > sizeof(Parts) ? sizeof(Lists) : sizeof(Parts);
};

// Whether the rows have to be taken again (ODD = false).
template <int D, bool GATHER, bool ODD>
__device__ __forceinline__ bool prefill_f32_rows(const AttnArgs &a, const float *__restrict__ q, const float *__restrict__ k,
                                                 const float *__restrict__ v, const int *__restrict__ row_ptr,
                                                 const int *__restrict__ blk_col, const uint8_t *__restrict__ blk_kind,
                                                 const uint64_t *__restrict__ tile_bits, const int *__restrict__ gather_idx,
                                                 float *__restrict__ out, float *__restrict__ lse, unsigned char *lds) {
  constexpr int CK = D / 16, HV = D / 64, kPad = D + 4;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  using Lists = typename F32Lds<D>::Lists;
  using Parts = typename F32Lds<D>::Parts;
  Lists &L = *reinterpret_cast<Lists *>(lds);
  Parts &P = *reinterpret_cast<Parts *>(lds);

  // Numbering: workgroup n runs on XCD n % 8, and the longest rows of the causal triangle go first. Where the
  // (sequence, KV head) pairs divide evenly among the XCDs, the row groups of a pair stay on one of them and share
  // its L2 copy of K and V; otherwise (two heads: 6 of 8 XCDs would stay empty) they go round robin.
  const int G = a.Hq / a.Hkv, n_pairs = a.B * a.Hkv, RG = a.tile_m / 16, per_pair = G * a.nQt * RG;
  const bool even = n_pairs % kXcd == 0;
  const int within = even ? blockIdx.x / kXcd % per_pair : blockIdx.x / n_pairs;
  const int pair = even ? blockIdx.x / kXcd / per_pair * kXcd + blockIdx.x % kXcd : blockIdx.x % n_pairs;
  const int wb = pair / a.Hkv, whkv = pair % a.Hkv, whq = whkv * G + within % G;
  const int wqt = a.nQt - 1 - within / (G * RG), rg = RG - 1 - within / G % RG, row0 = wqt * a.tile_m + rg * 16;
  if (row0 >= a.S) return false;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int i = row0 + r16;
  const bool live = i < a.S;
  const int t0 = row_ptr[(int64_t)whq * (a.nQt + 1) + wqt];
  const int t1 = row_ptr[(int64_t)whq * (a.nQt + 1) + wqt + 1];
  const float *kb = k + wb * a.k_sb + whkv * a.k_sh + 4 * g;
  const float *vb = v + wb * a.v_sb + whkv * a.v_sh;

  float4 qf[CK];
  {
    const float *qp = q + wb * a.q_sb + whq * a.q_sh + (int64_t)min(i, a.S - 1) * a.q_ss + 4 * g;
#pragma unroll
    for (int c = 0; c < CK; ++c) qf[c] = *reinterpret_cast<const float4 *>(qp + 16 * c);
  }
  f32x4 o[HV * 4];
#pragma unroll
  for (int x = 0; x < HV * 4; ++x) o[x] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.0f;  // of the lane's row; l is this lane's part
  unsigned any = 0;               // bits of kept keys
  float odd_any = 0.0f;           // 0, or NaN when a V entry was infinite or NaN

  for (int seg = t0; seg < t1; seg += kF32Seg) {
    const int n_seg = min(kF32Seg, t1 - seg);
    if (seg > t0) __syncthreads();  // every wave is done with the previous segment's lists
    // ---- the rows' mask words of every listed tile, and which blocks of 16 keys they occupy
    const int kinds = lane < n_seg ? blk_kind[seg + lane] : 0;
    // (a column outside its range, from a list that was never filled, is pulled inside it)
    if (wave == 0 && lane < n_seg)
      L.col[lane] = min(max(blk_col[seg + lane], 0), a.nKt + (GATHER ? a.gather_stride / a.tile_n : 0) - 1);
    for (int x0 = wave; x0 < n_seg; x0 += 16) {  // four tiles' words in flight per wave
      unsigned word[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = seg + min(x0 + 4 * u, n_seg - 1);
        word[u] = reinterpret_cast<const unsigned *>(tile_bits)[((int64_t)t * a.tile_m + rg * 16 + r16) * (2 * a.wpr) +
                                                                min(g, 2 * a.wpr - 1)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int x = x0 + 4 * u;
        if (x >= n_seg) break;
        if (__builtin_amdgcn_readlane(kinds, x) & 1)  // every entry kept: the words do not count (they may be unwritten)
          word[u] = ~0u;
        if (!live || g >= 2 * a.wpr) word[u] = 0u;
        L.words[x][lane] = word[u];
        const uint64_t lo = __ballot((word[u] & 0xFFFFu) != 0), hi = __ballot((word[u] >> 16) != 0);
        if (lane == 0) {
          unsigned occ = 0;
          for (int y = 0; y < 4; ++y)
            occ |= ((lo >> (16 * y)) & 0xFFFF ? 1u << (2 * y) : 0u) | ((hi >> (16 * y)) & 0xFFFF ? 2u << (2 * y) : 0u);
          L.occ[x] = (unsigned char)occ;
        }
      }
    }
    __syncthreads();
    // ---- the block list: every wave adds up the same prefix, wave 0 writes
    unsigned occ = lane < n_seg ? L.occ[lane] : 0u;
    int at = wave_prefix(__popc(occ));
    const int n_blk = __builtin_amdgcn_readlane(at, 63);
    if (wave == 0)
      for (at -= __popc(occ); occ; occ &= occ - 1) L.blk[at++] = (unsigned short)(lane * 8 + __builtin_ctz(occ));
    __syncthreads();

    // row of K and V that slot s of tile x stands for
    auto key_row = [&](int x, int s) -> int64_t {
      const int col = __builtin_amdgcn_readfirstlane(L.col[x]);
      int j = col * a.tile_n + s;
      if (GATHER) {  // a gathered tile (index >= nKt): its slots are the head's matched columns
        const int c = gather_idx[(int64_t)whq * a.gather_stride + max(col - a.nKt, 0) * a.tile_n + s];
        if (col >= a.nKt) j = c;
      }
      return min(max(j, 0), a.S - 1);
    };
    // A block's K and V rows sit in registers; where an iteration has used a part of them it fetches that part of the wave's
    // next block, a whole iteration ahead of its use.
    float4 kf[CK], vf[4][HV];  // K row r16, dims 16 c + 4 g; V row 4 g + s, dims 64 h + 4 r16
    const float *kp, *vp[4];
    auto find_rows = [&](int e) {  // the rows of block e; returns its entry
      const int blk = __builtin_amdgcn_readfirstlane(L.blk[e]), x = blk >> 3, s0 = (blk & 7) * 16;
      kp = kb + key_row(x, s0 + r16) * a.k_ss;
#pragma unroll
      for (int s = 0; s < 4; ++s) vp[s] = vb + key_row(x, s0 + 4 * g + s) * a.v_ss + 4 * r16;
      return blk;
    };
    auto take = [](const float *at) { return *reinterpret_cast<const float4 *>(at); };
    // more: there is a next block, whose rows find_rows has found
    auto compute = [&](int blk, auto more) {
      constexpr bool MORE = decltype(more)::value;
      const int x = blk >> 3, b16 = blk & 7;
      const unsigned kept = L.words[x][(b16 >> 1) * 16 + r16] >> (16 * (b16 & 1));  // low 16 bits: the block's keys
      any |= kept & 0xFFFFu;
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;  // two chains: a product's result is ready only after the next has started
#pragma unroll
      for (int c = 0; c < CK; ++c) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].x, qf[c].x, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].y, qf[c].y, s1, 0, 0, 0);
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].z, qf[c].z, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c].w, qf[c].w, s1, 0, 0, 0);
        if (MORE) {
          kf[c] = take(kp + 16 * c);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      float p[4], mx = m, odd = ODD ? 0.0f : odd_any;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[r] = (kept >> (4 * g + r)) & 1 ? (s0[r] + s1[r]) * a.scale : -INFINITY;
        mx = fmaxf(mx, p[r]);
      }
      {  // the maximum of the row's four lanes: the rows of 16 lanes in pairs, then the halves of the wave
        u32x2 sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      }
      if (__ballot(mx > m)) {
        const float corr = mx > m ? expf(m - mx) : 1.0f;  // m = -inf: 0
        l *= corr;
#pragma unroll
        for (int y = 0; y < HV * 4; ++y) o[y] *= corr;
        m = fmaxf(m, mx);
      }
      const float ref = m == -INFINITY ? 0.0f : m;  // (no key of the row so far)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[r] = expf(p[r] - ref);
        l += p[r];
#pragma unroll
        for (int h = 0; h < HV; ++h) {  // 0, or NaN where a V entry is infinite or NaN
          odd = fmaf(vf[r][h].x, 0.0f, fmaf(vf[r][h].y, 0.0f, odd));
          odd = fmaf(vf[r][h].z, 0.0f, fmaf(vf[r][h].w, 0.0f, odd));
        }
      }
      if (!ODD) odd_any = odd;
      if (!ODD || __ballot(odd != 0.0f) == 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int h = 0; h < HV; ++h) {
            o[4 * h + 0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[s][h].x, p[s], o[4 * h + 0], 0, 0, 0);
            o[4 * h + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[s][h].y, p[s], o[4 * h + 1], 0, 0, 0);
            o[4 * h + 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[s][h].z, p[s], o[4 * h + 2], 0, 0, 0);
            o[4 * h + 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[s][h].w, p[s], o[4 * h + 3], 0, 0, 0);
            if (MORE) {
              vf[s][h] = take(vp[s] + 64 * h);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
      } else {
#pragma unroll 1
        for (int key = 0; key < 16; ++key) {
          const float pk = __shfl(key & 2 ? (key & 1 ? p[3] : p[2]) : (key & 1 ? p[1] : p[0]), r16 + 16 * (key >> 2));
          const float *at = vb + key_row(x, b16 * 16 + key) * a.v_ss + 16 * g;
          if (!((kept >> key) & 1)) continue;
#pragma unroll
          for (int h = 0; h < HV; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float4 vv = *reinterpret_cast<const float4 *>(at + 64 * h + 4 * r);
              o[4 * h + 0][r] = fmaf(pk, vv.x, o[4 * h + 0][r]);
              o[4 * h + 1][r] = fmaf(pk, vv.y, o[4 * h + 1][r]);
              o[4 * h + 2][r] = fmaf(pk, vv.z, o[4 * h + 2][r]);
              o[4 * h + 3][r] = fmaf(pk, vv.w, o[4 * h + 3][r]);
            }
        }
        if (MORE) {
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int h = 0; h < HV; ++h) vf[s][h] = take(vp[s] + 64 * h);
        }
      }
    };
    if (wave < n_blk) {
      int e = wave, blk = find_rows(e);
#pragma unroll
      for (int c = 0; c < CK; ++c) kf[c] = take(kp + 16 * c);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int h = 0; h < HV; ++h) vf[s][h] = take(vp[s] + 64 * h);
      for (; e + 4 < n_blk; e += 4) {
        const int next = find_rows(e + 4);
        compute(blk, std::true_type{});
        blk = next;
      }
      compute(blk, std::false_type{});
    }
  }

  // ---- merge the four waves. Accumulator r of o[4 h + x] is dim 64 h + 16 g + 4 r + x of the lane's row.
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  __syncthreads();  // the lists are done with
  if (g == 0) {
    P.m[wave][r16] = m;
    P.l[wave][r16] = l;
    P.any[wave][r16] = any;
  }
  if (!ODD) {
    const bool odd = __ballot(odd_any != 0.0f) != 0;
    if (lane == 0) P.odd[wave] = odd;
  }
#pragma unroll
  for (int h = 0; h < HV; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<float4 *>(&P.o[wave][r16 * kPad + 64 * h + 16 * g + 4 * r]) =
          make_float4(o[4 * h][r], o[4 * h + 1][r], o[4 * h + 2][r], o[4 * h + 3][r]);
  __syncthreads();
  if (!ODD && (P.odd[0] | P.odd[1] | P.odd[2] | P.odd[3])) return true;
  const int row = threadIdx.x >> 4, part = threadIdx.x & 15;
  if (row0 + row >= a.S) return false;
  float M = fmaxf(fmaxf(P.m[0][row], P.m[1][row]), fmaxf(P.m[2][row], P.m[3][row])), sum = 0.0f, wt[4];
#pragma unroll
  for (int y = 0; y < 4; ++y) {
    wt[y] = P.m[y][row] > -INFINITY ? expf(P.m[y][row] - M) : 0.0f;  // (a wave that met no key of the row)
    sum += wt[y] * P.l[y][row];
  }
  // no key: 0; NaN stays NaN, and a softmax over nothing but -inf has no value either
  const bool has_key = (P.any[0][row] | P.any[1][row] | P.any[2][row] | P.any[3][row]) != 0;
  const float inv = sum > 0.0f ? 1.0f / sum : sum == 0.0f && has_key ? NAN : sum * 0.0f;
#pragma unroll
  for (int h = 0; h < HV; ++h) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const float4 x = *reinterpret_cast<const float4 *>(&P.o[y][row * kPad + 64 * h + 4 * part]);
      acc.x = fmaf(wt[y], x.x, acc.x);
      acc.y = fmaf(wt[y], x.y, acc.y);
      acc.z = fmaf(wt[y], x.z, acc.z);
      acc.w = fmaf(wt[y], x.w, acc.w);
    }
    *reinterpret_cast<float4 *>(out + wb * a.o_sb + whq * a.o_sh + (int64_t)(row0 + row) * a.o_ss + 64 * h + 4 * part) =
        make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
  }
  if (lse && part == 0) lse[((int64_t)wb * a.Hq + whq) * a.S + row0 + row] = sum > 0.0f ? M + logf(sum) : -INFINITY;
  return false;
}

template <int D, bool GATHER>
__device__ __attribute__((noinline)) void prefill_f32_odd_rows(uint64_t args_at, __attribute__((address_space(3))) unsigned char *lds) {
  // (an argument in vector registers, the same in every lane)
  const uint64_t at = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(args_at >> 32)) << 32 |
                      (unsigned)__builtin_amdgcn_readfirstlane((int)args_at);
  const F32Args &t = *(const F32Args *)(const __attribute__((address_space(4))) F32Args *)at;
  prefill_f32_rows<D, GATHER, true>(t.a, t.q, t.k, t.v, t.row_ptr, t.blk_col, t.blk_kind, t.tile_bits, t.gather_idx, t.out, t.lse,
                                    (unsigned char *)lds);
}

template <int D, bool GATHER>
__global__ __launch_bounds__(256, D == 128 ? 3 : 4) void k_prefill_f32(F32Args t) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[F32Lds<D>::kBytes];
  if (!prefill_f32_rows<D, GATHER, false>(t.a, t.q, t.k, t.v, t.row_ptr, t.blk_col, t.blk_kind, t.tile_bits, t.gather_idx, t.out, t.lse, lds))
    return;
  __syncthreads();
  prefill_f32_odd_rows<D, GATHER>((uint64_t)__builtin_amdgcn_kernarg_segment_ptr(), (__attribute__((address_space(3))) unsigned char *)lds);
}

// No more workgroups than the chip takes two to a CU: they are all there at once then, and the second form alone is the faster one
// (no private memory to set up: 1 x 4 heads x 300 tokens 11.85 us against 12.0; 11.75 before there were two forms). From there on the first: 2 x 8 x 1500, d 128, 51.4 -> 46.2 us, 4 x 16 x 2000 336 -> 292, d 64 183 -> 166, 3 x 8 x 700
// 23.0 -> 20.5. What that costs is paid where V does hold an infinity or a NaN, by the row groups that meet one, which are taken twice
// and the second time with registers in private memory: 4 x 16 x 2000, d 128, one NaN row in the middle of each sequence 332 -> 637 us,
// one in 50 525 -> 1096, the last quarter of the rows infinite 407 -> 545; d 64 one in 50 259 -> 428. (Leaving the first pass at the
// first odd value saves 1 to 11 % of that, and costs the others 0.2 %.)
constexpr int kF32Few = 512;
template <int D, bool GATHER>
__global__ __launch_bounds__(256, 2) void k_prefill_f32_few(AttnArgs a, const float *__restrict__ q, const float *__restrict__ k,
                                                            const float *__restrict__ v, const int *__restrict__ row_ptr,
                                                            const int *__restrict__ blk_col, const uint8_t *__restrict__ blk_kind,
                                                            const uint64_t *__restrict__ tile_bits, const int *__restrict__ gather_idx,
                                                            float *__restrict__ out, float *__restrict__ lse) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[F32Lds<D>::kBytes];
  prefill_f32_rows<D, GATHER, true>(a, q, k, v, row_ptr, blk_col, blk_kind, tile_bits, gather_idx, out, lse, lds);
}

// ================================================================================================
// bf16 MFMA variant
constexpr int kBM = 128, kBN = 128;

// LDS layout. Rows are 256 B = 16 chunks of 16 B and are not padded, because the global -> LDS
// copies are done by the load-to-LDS instruction, which writes the 64 lanes of a wave to 1 KiB of
// consecutive LDS. Bank conflicts are avoided by permuting the chunks of a row instead:
//   K row r: chunk c lives at position c ^ (r & 15)        (16-byte reads of 16 consecutive rows
//            and one logical chunk then cover all 64 banks once)
//   V row r: chunk c lives at position c ^ ((r & 3) << 2)  (a transposing read touches 4 rows x 64 B
//            per half-wave; the four 64-byte groups land in different bank quarters)
// The permutation is applied on the global side of the copy (which chunk a lane fetches).

// Scheduling hints: instruction classes of __builtin_amdgcn_sched_group_barrier.
#define DAM_SCHED_MFMA 0x008
#define DAM_SCHED_DSREAD 0x100

// ================================================================================================
// Block-pipelined bf16 kernel. The unit of work is a block of 32 keys (one occupied key quarter of
// a listed tile). In iteration b a wave issues, interleaved in one instruction stream,
//     the 8 MFMAs of S_{b+1} = K_{b+1} Q^T   (one dependent chain),
//     the 8 MFMAs of O^T += V_{b-1}^T P_{b-1}^T (four independent accumulators),
//     the softmax arithmetic of block b (VALU) on S_b, which finished one iteration earlier,
// so that the matrix pipe and the vector ALU of a SIMD are busy at the same time from within one
// wave. K and V blocks live in two LDS rings of four 8 KiB slots each, filled by load-to-LDS
// copies issued three iterations ahead (K_{b+4} and V_{b+2} in iteration b); one barrier per
// iteration. The stream is padded with "dummy" blocks (mask bits all zero, so S = -inf and P = 0)
// at both ends, which keeps every iteration identical.
constexpr int kBlkKeys = 32;
constexpr int kBlkBytes = kBlkKeys * 256;
constexpr int kRing = 4;
constexpr int kVRing = kRing * kBlkBytes;  // byte offset of the V ring; K ring at 0
constexpr int kBitsRing = 2 * kRing * kBlkBytes;  // mask words: 4 slots x 4 waves x 64 lanes x 4 B
constexpr int kBlkList = kBitsRing + kRing * 1024;  // the block list of the current segment of tiles
constexpr int kSegTiles = 128;                      // listed tiles expanded into the list at a time
constexpr int kListEntries = kSegTiles * 4 + 1;     // up to four blocks per tile, and the dummy that ends the list
constexpr int kPipeLds = kBlkList + kListEntries * 8;

struct Blk {
  int key0;        // first key of the block (gathered tile: first row of the block in the gathered copy)
  int bits_off;    // byte offset of row 0's mask word for the block from the tile row's first mask word
  int flags;       // bit 0: tile is full (no mask), bit 1: dummy, bit 2: gathered tile (offsets into the gathered copies)
};

// FAST: the softmax without a running maximum. A weight is exp2(logit * scale * log2 e) itself: one multiply and
// one exponential per entry, no row maximum, no subtraction, no rescaling of O. (Folding the factor into the
// bf16 queries would save the multiply, but rounds every logit by up to 2^-9 of its size: 8 % in the weight of a
// logit of 70.) That is exact as long as the weights stay inside the range of fp32 and bf16 (both have 8
// exponent bits); the kernel checks the row sums at the end of a work item and sends the item to the variant
// with a running reference (FAST = false) when a sum left [2^-100, 2^100].
// seen / seen_full: does this lane's row have a kept entry at all (an empty row is not a failed one).
template <int PH, bool FAST>
__device__ __forceinline__ void pipe_iter(const unsigned char *__restrict__ lds, const bf16x8 (&qf)[8],
                                          f32x16 (&oacc)[4], const f32x16 &sA, f32x16 &sB,
                                          const unsigned (&pPrev)[8], unsigned (&pCur)[8], float &m_run,
                                          float &l_run, unsigned &seen, int &seen_full, int flags_next, int bits_addr,
                                          float c2, int kbase, int vbase, int hf) {
  // kbase ^ (c << 5) is this lane's address of chunk pair c of its K row, vbase ^ (db << 6) that of
  // dim block db in its V rows (the chunk permutations are XORs, see the layout note)
  int kaddr[8], vaddr[4];
#pragma unroll
  for (int c = 0; c < 8; ++c) kaddr[c] = kbase ^ (c << 5);
#pragma unroll
  for (int db = 0; db < 4; ++db) vaddr[db] = vbase ^ (db << 6);
  constexpr int KS = PH * kBlkBytes;                          // slot of K_{b+1}
  constexpr int VS = kVRing + ((PH + 2) & 3) * kBlkBytes;     // slot of V_{b-1}
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  // The first product of the S_{b+1} chain. Accumulator e is key 8 (e / 4) + 4 hf + e % 4 of the block
  // and starts at 0 (kept) or -inf (masked); a full tile needs no mask words and starts from a literal
  // zero (wave-uniform branch), and so does a block of a partial tile whose 32 x 32 entries of this wave
  // are all kept (a band edge crosses only some of the sixteen such squares of a tile).
  const bf16x8 kf0 = lds_read_b128(lds, KS + kaddr[0]);
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (flags_next & 1) {
    if (FAST) seen_full = 1;
    sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf0, qf[0], zero, 0, 0, 0);
  } else {
    unsigned bits_next = *reinterpret_cast<const unsigned *>(lds + kBitsRing + PH * 1024 + bits_addr);
    if (flags_next & 2) bits_next = 0u;  // dummy block: nothing kept
    if (FAST) seen |= bits_next;
    if (__builtin_amdgcn_ballot_w64(bits_next != 0xFFFFFFFFu) == 0) {
      sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf0, qf[0], zero, 0, 0, 0);
    } else {
      const int inv = (int)~(bits_next >> (4 * hf));
      // sign-extended one-bit field (0 or all ones), then the bits of -inf; the extract is written as an
      // instruction because the compiler turns the builtin into a three-operation compare and select
      mask_init(sB, inv, std::make_integer_sequence<int, 16>{});
      sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf0, qf[0], sB, 0, 0, 0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // ---- operand fetches, in the order the MFMAs consume them
  bf16x8 kf[8];
  s16x8 vf[2][4];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    if (x > 0) kf[x] = lds_read_b128(lds, KS + kaddr[x]);
    const int a2 = x >> 2, db = x & 3;
    const s16x4 r0 = lds_read_tr(lds, VS + vaddr[db] + (a2 * 16) * 256);
    const s16x4 r1 = lds_read_tr(lds, VS + vaddr[db] + (a2 * 16 + 8) * 256);
    vf[a2][db] = __builtin_shufflevector(r0, r1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
  // ---- matrix work: the rest of the S_{b+1} chain and P_{b-1} V_{b-1}, alternating
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    if (x > 0) sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[x], qf[x], sB, 0, 0, 0);
    const int a2 = x >> 2, db = x & 3;
    const u32x4 praw = {pPrev[4 * a2], pPrev[4 * a2 + 1], pPrev[4 * a2 + 2], pPrev[4 * a2 + 3]};
    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[a2][db]),
                                                       __builtin_bit_cast(bf16x8, praw), oacc[db], 0, 0, 0);
  }
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  if (FAST) {
    // ---- vector work: the weights of block b and their sum, nothing else
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const float p0 = __builtin_amdgcn_exp2f(sA[e] * c2);
      const float p1 = __builtin_amdgcn_exp2f(sA[e + 1] * c2);
      pCur[e / 2] = pack_bf16(p0, p1);
      // the row sum is taken over the rounded weights the P V product uses
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pCur[e / 2]), ones, l_run, false);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) asm volatile("" ::"v"(pCur[e]));
    // ---- interleave: a few operand reads ahead, then per MFMA three VALU ops and the reads it needs
    __builtin_amdgcn_sched_group_barrier(DAM_SCHED_DSREAD, 12, 0);
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      if (x > 0) {
        __builtin_amdgcn_sched_group_barrier(DAM_SCHED_MFMA, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
      }
      __builtin_amdgcn_sched_group_barrier(DAM_SCHED_DSREAD, 2, 0);
      __builtin_amdgcn_sched_group_barrier(DAM_SCHED_MFMA, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
      __builtin_amdgcn_sched_group_barrier(DAM_SCHED_DSREAD, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    return;
  }
  // ---- vector work: online softmax of block b; one query per lane pair (lane, lane ^ 32)
  float mx = fmaxf(fmaxf(sA[0], sA[1]), sA[2]);
#pragma unroll
  for (int e = 3; e < 15; e += 2) mx = fmaxf(fmaxf(sA[e], sA[e + 1]), mx);
  mx = fmaxf(mx, sA[15]);
  {
    // the other half-wave's maximum of the same query row: one swap of the 32-lane halves (operands
    // both mx: the results are the lower half's values in all lanes, and the upper half's)
    typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;
    const u32x2_t sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  }
  // m_run is the reference the weights are taken against, not necessarily the running maximum: it
  // only moves when the maximum has grown past it by more than 8 in log2 units (weights then stay
  // below 2^8, far inside the range of bf16 and of the fp32 sums), so that O rarely has to be rescaled.
  // The quotient O / l at the end does not depend on the reference. (-inf) - (-inf) is NaN: no move.
  const float m_top = fmaxf(m_run, mx);
  const bool move = (m_top - m_run) * c2 > 8.0f;
  const float m_new = move ? m_top : m_run;
  const float m_ref = m_new == -INFINITY ? 0.0f : m_new;
  const float off = m_ref * c2;
  const float m_old = m_run;
  m_run = m_new;
  float psum = 0.0f;
#pragma unroll
  for (int e = 0; e < 16; e += 2) {
    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sA[e], c2, -off));
    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sA[e + 1], c2, -off));
    pCur[e / 2] = pack_bf16(p0, p1);
    // the row sum is taken over the rounded weights the P V product uses
    psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pCur[e / 2]), ones, psum, false);
  }
  // keep the weights of block b inside this block of code (they are only consumed an iteration later
  // and would otherwise be sunk below the matrix work)
#pragma unroll
  for (int e = 0; e < 8; ++e) asm volatile("" ::"v"(pCur[e]));
  // ---- interleave: a few operand reads ahead, then per MFMA pair three reads and eight VALU ops
  __builtin_amdgcn_sched_group_barrier(DAM_SCHED_DSREAD, 12, 0);
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    if (x > 0) {
      __builtin_amdgcn_sched_group_barrier(DAM_SCHED_MFMA, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
    __builtin_amdgcn_sched_group_barrier(DAM_SCHED_DSREAD, 2, 0);
    __builtin_amdgcn_sched_group_barrier(DAM_SCHED_MFMA, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    __builtin_amdgcn_sched_group_barrier(DAM_SCHED_DSREAD, 1, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  // O and the row sum were accumulated against the old reference: when some row's reference moved,
  // rescale them, after P_{b-1} V_{b-1} is in (rare after the first blocks of a row)
  if (__ballot(move)) {
    const float corr = move ? __builtin_amdgcn_exp2f((m_old - m_ref) * c2) : 1.0f;  // old = -inf: 0
    l_run *= corr;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[db][e] *= corr;
  }
  l_run += psum;
}

// The FAST iteration laid out by hand in eight segments, one per pair of products (S chain step x, P V step x).
// The wave issues in order, so what stands between the last product of one iteration and the first of the next
// is time the matrix pipe of this wave idles: the bookkeeping of an iteration (decoding the next descriptor,
// issuing the five copies, fetching the descriptor after that) therefore sits inside the stream of products,
// one piece per segment (bk(x)), behind the operand reads (the copies are volatile statements that LDS reads do
// not move across), and only the flag test, the wait for the copies, the barrier and the first operand reads
// remain between two iterations.
// PART says which of the three streams the iteration holds: kAll in the steady state; the first iteration of a
// pass (block -1, kChainOnly) has no weights to compute and nothing to add to O, the second one (block 0,
// kNoPV) nothing to add to O yet (P_{-1} is zero). (The last iteration, whose block is the trailing dummy, stays
// whole: a second way out of the loop's iterations makes the compiler copy the 64 accumulators of O every time.)
enum { kAll = 0, kChainOnly = 1, kNoPV = 2 };
template <int PH, int PART, class Bk>
__device__ __forceinline__ void pipe_iter_seg(const unsigned char *__restrict__ lds, const bf16x8 (&qf)[8],
                                              f32x16 (&oacc)[4], const f32x16 &sA, f32x16 &sB,
                                              const unsigned (&pPrev)[8], unsigned (&pCur)[8], float &l_run,
                                              unsigned &seen, int &seen_full, int flags_next, int bits_addr, float c2,
                                              int kbase, int vbase, int hf, Bk &&bk) {
  int kaddr[8], vaddr[4];
#pragma unroll
  for (int c = 0; c < 8; ++c) kaddr[c] = kbase ^ (c << 5);
#pragma unroll
  for (int db = 0; db < 4; ++db) vaddr[db] = vbase ^ (db << 6);
  constexpr int KS = PH * kBlkBytes;                          // slot of K_{b+1}
  constexpr int VS = kVRing + ((PH + 2) & 3) * kBlkBytes;     // slot of V_{b-1}
  typedef __attribute__((ext_vector_type(8))) short s16x8;
  bf16x8 kf[8];
  s16x8 vf[2][4];
  constexpr bool kChain = true, kWeights = PART != kChainOnly, kPV = PART == kAll;
  auto fetch = [&](int x) {
    if (kChain) kf[x] = lds_read_b128(lds, KS + kaddr[x]);
    if (kPV) {
      const int a2 = x >> 2, db = x & 3;
      const s16x4 r0 = lds_read_tr(lds, VS + vaddr[db] + (a2 * 16) * 256);
      const s16x4 r1 = lds_read_tr(lds, VS + vaddr[db] + (a2 * 16 + 8) * 256);
      vf[a2][db] = __builtin_shufflevector(r0, r1, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  // ---- the operands of the first four segments, and this row's mask word of the block
  const bool full_tile = (flags_next & 1) != 0;
  unsigned bits_next = 0xFFFFFFFFu;
  if (kChain && !full_tile) bits_next = *reinterpret_cast<const unsigned *>(lds + kBitsRing + PH * 1024 + bits_addr);
#pragma unroll
  for (int x = 0; x < 4; ++x) fetch(x);
  __builtin_amdgcn_sched_barrier(0);
  if (kChain) {
    if (full_tile) {
      seen_full = 1;
    } else {
      if (flags_next & 2) bits_next = 0u;  // dummy block: nothing kept
      seen |= bits_next;
    }
  }
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // no entry of this wave's 32 x 32 square is kept (wave-uniform): every logit is -inf without any product. (The
  // weights of such a square and its products with V stay: branches around them cost more than they save.)
  const bool skip_s = __builtin_amdgcn_ballot_w64(bits_next != 0u) == 0;
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int a2 = x >> 2, db = x & 3;
    // P_{b-1} V_{b-1}, step x (first: it needs no mask)
    if (kPV) {
      const u32x4 praw = {pPrev[4 * a2], pPrev[4 * a2 + 1], pPrev[4 * a2 + 2], pPrev[4 * a2 + 3]};
      oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vf[a2][db]),
                                                         __builtin_bit_cast(bf16x8, praw), oacc[db], 0, 0, 0);
    }
    // S_{b+1} chain, step x. Accumulator e is key 8 (e / 4) + 4 hf + e % 4 of the block and starts at 0 (kept)
    // or -inf (masked); a block whose 32 x 32 entries of this wave are all kept starts from a literal zero
    if (kChain) {
      if (x == 0) {
        if (__builtin_amdgcn_ballot_w64(bits_next != 0xFFFFFFFFu) == 0) {
          sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0], zero, 0, 0, 0);
        } else if (skip_s) {
#pragma unroll
          for (int e = 0; e < 16; ++e) sB[e] = -INFINITY;
        } else {
          const int inv = (int)~(bits_next >> (4 * hf));
          mask_init(sB, inv, std::make_integer_sequence<int, 16>{});
          sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[0], sB, 0, 0, 0);
        }
      } else if (!skip_s) {
        sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[x], qf[x], sB, 0, 0, 0);
      }
    }
    if (x < 4) fetch(x + 4);
    // the weights of two entries of block b and their part of the row sum
    if (kWeights) {
      const float p0 = __builtin_amdgcn_exp2f(sA[2 * x] * c2);
      const float p1 = __builtin_amdgcn_exp2f(sA[2 * x + 1] * c2);
      pCur[x] = pack_bf16(p0, p1);
      l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pCur[x]), ones, l_run, false);
      asm volatile("" ::"v"(pCur[x]));
    }
    if (kChain) bk(std::integral_constant<int, 0>{} , x);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The queues of work items, a (batch, query head, query tile) each. Where the (sequence, KV head) pairs divide evenly among
// the XCDs a queue holds whole pairs, whose K and V then stay in that XCD's L2; otherwise every eighth item of all pairs (with
// four pairs half the chip would have nothing to start with). Numbered with the longest rows of a pair's causal triangle
// first.
struct Queues {
  int G, n_pairs, per_pair, nQt, Hkv;
  bool even;
  __device__ __forceinline__ explicit Queues(const AttnArgs &a)
      : G(a.Hq / a.Hkv), n_pairs(a.B * a.Hkv), per_pair(a.Hq / a.Hkv * a.nQt), nQt(a.nQt), Hkv(a.Hkv), even(a.B * a.Hkv % kXcd == 0) {}
  __device__ __forceinline__ int items(int qu) const {
    return even ? n_pairs / kXcd * per_pair : (n_pairs * per_pair - qu + kXcd - 1) / kXcd;
  }
  __device__ __forceinline__ int pair_of(int item, int qu) const { return even ? item / per_pair * kXcd + qu : (item * kXcd + qu) % n_pairs; }
  __device__ __forceinline__ int within_of(int item, int qu) const { return even ? item % per_pair : (item * kXcd + qu) / n_pairs; }
  // offsets of an item's listed tiles
  __device__ __forceinline__ const int *span(const int *row_ptr, int item, int qu) const {
    const int within = within_of(item, qu), hkv = pair_of(item, qu) % Hkv;
    return row_ptr + (int64_t)(hkv * G + within % G) * (nQt + 1) + (nQt - 1 - within / G);
  }
};

// A queue's items in falling order of their number of blocks: {item, t0, t1, -} each, so that a workgroup that draws one has
// its listed tiles with it. By numbers alone a dense head's long items started among the last ones: 32 heads x 4096 tokens
// (2 items per workgroup) took 57 us where the workgroups worked 42 us on average. A counting sort by one workgroup per queue, in
// the launch that precedes the attention kernel anyway (5.3 us with it, 5.2 without). By number / by length, us, whole prefills:
// captured masks, whose heads differ most, 32 heads x 4096 captured at 1024 57.7 / 51.0, 32 x 12345 at 1024 134 / 122, 16 x 16000
// at 1024 88.6 / 78.7, 32 x 16384 at 256 119 / 117, 64 x 8000 at 2048 278 / 279; patterns of several sequences 8 x 16 x 2000 98 /
// 90, 3 x 16 x 3500 92 / 80, 4 x 32 x 3001 158 / 150 (159 / 157 on another chip); patterns of one long sequence, whose heads are
// alike, 32 x 8000 149 / 146, 32 x 12345 283 / 285, 16 x 30000 524 / 527, 16 x 8000 (16 KV heads) 87 / 92.
// Where a queue holds several pairs they are taken in groups of at least kOrderGroup items, three per workgroup: all at once they
// share the L2 less, in small groups the last one has too few items to end evenly. (21 shapes of 8 to 160 items per pair: groups
// of 96 -2 to +4.5 %, 384 -1 to +3, all -1.5 to +3.)
// (Blocks are counted over an item's first 64 tiles, the others taken for two each.)
constexpr int kOrderBins = 512, kOrderGroup = 192;
template <int THREADS>
__device__ __forceinline__ void order_items(const AttnArgs &a, const int *__restrict__ row_ptr, const uint8_t *__restrict__ blk_kind, int qu,
                                            int4 *__restrict__ order) {
  __shared__ int start[kOrderBins];
  __shared__ int wave_sum[THREADS / 64];
  const Queues qs(a);
  const int n = qs.items(qu), tid = threadIdx.x;
  int4 *out = order + (int64_t)qu * kOrderMax;
  constexpr int kEach = kOrderMax / THREADS;
  int t0[kEach], t1[kEach], bin[kEach];
#pragma unroll
  for (int x = 0; x < kEach; ++x) {
    const int item = x * THREADS + tid;
    t0[x] = t1[x] = 0;
    if (item < n) {
      const int *rp = qs.span(row_ptr, item, qu);
      t0[x] = rp[0];
      t1[x] = rp[1];
    }
  }
  const int group_pairs = (kOrderGroup + qs.per_pair - 1) / qs.per_pair;
  const int groups = qs.even ? max(1, qs.n_pairs / kXcd / group_pairs) : 1, bins_each = kOrderBins / groups;
  for (int x = tid; x < kOrderBins; x += THREADS) start[x] = 0;
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kEach; ++x) {
    const int item = x * THREADS + tid;
    if (item < n) {
      const int n_tiles = t1[x] - t0[x], m = min(n_tiles, 64);
      const int blocks = blocks_of_tiles(blk_kind + t0[x], m) + 2 * (n_tiles - m);
      const int group = groups > 1 ? min(item / (group_pairs * qs.per_pair), groups - 1) : 0;
      bin[x] = (group + 1) * bins_each - 1 - min(blocks, bins_each - 1);
      atomicAdd(&start[bin[x]], 1);
    }
  }
  __syncthreads();
  // exclusive prefix over the bins, kOrderBins / THREADS consecutive ones per thread
  constexpr int kPer = (kOrderBins + THREADS - 1) / THREADS;
  int c[kPer], mine = 0;
#pragma unroll
  for (int y = 0; y < kPer; ++y) {
    c[y] = tid * kPer + y < kOrderBins ? start[tid * kPer + y] : 0;
    mine += c[y];
  }
  int incl = wave_prefix(mine);
  if ((tid & 63) == 63) wave_sum[tid >> 6] = incl;
  __syncthreads();
  int at = incl - mine;
  for (int y = 0; y < (tid >> 6); ++y) at += wave_sum[y];
#pragma unroll
  for (int y = 0; y < kPer; ++y) {
    if (tid * kPer + y < kOrderBins) start[tid * kPer + y] = at;
    at += c[y];
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kEach; ++x) {
    const int item = x * THREADS + tid;
    if (item < n) out[atomicAdd(&start[bin[x]], 1)] = make_int4(item, t0[x], t1[x], 0);
  }
}

// RAGGED: the sequence length is not a multiple of the block size, so the last block of a row of tiles
// may reach past the end of K and V.
// GATHER: the block index may hold gathered column tiles (tile index >= nKt), whose K / V rows come from
// the per-head gathered copies.
// FAST: the softmax without a running maximum (see pipe_iter). An item in which some row's sum of weights left the safe
// range goes onto the workgroup's own list (Shared::redo, threaded through `next`, a word per item), and when the queues
// are empty the FAST = false instantiation takes exactly those items and overwrites their rows. With well-scaled inputs
// the lists stay empty. (Behind the items, not among them: both variants inside one loop over the items spilled registers
// in its pipeline. As a launch of its own the second variant cost 4 to 5 us per call, almost always for nothing.)
struct Shared {
  int4 item[2];  // the next item: its number and queue, its listed tiles [t0, t1); its sequence, KV head, query head, query tile
  int nblk, bad;
  int redo;     // first item of the workgroup's redo list (8 * item + queue), or -1
};
struct Operands {
  const __hip_bfloat16 *q, *k, *v;
  const int *row_ptr, *blk_col;
  const uint8_t *blk_kind;
  const uint64_t *tile_bits;
  __hip_bfloat16 *out;
  float *lse;
  int *ctl, *next;
  const int4 *order;  // the queues' items by length, or nullptr
  const __hip_bfloat16 *kgath, *vgath;
};

// The kernel's arguments, read where they arrive at every item's start and end (opaque to the compiler, so that it does not keep
// them). Held in scalar registers through the items, 54 to 102 of those were spilled to vector lanes and taken back lane by lane,
// how many by the allocator's chance: an argument more had cost every ragged length 1 to 2 %. Now none is. 2 x 32 heads x 1017
// tokens 35.2 -> 34.6 us, 8 x 700 20.3 -> 19.5, 32 x 2048 38.5 -> 37.8, 8 x 16 x 2000 94 -> 91; 16k tokens and more as before.
struct KernelArgs {
  AttnArgs a;
  Operands t;
};
using ArgsAt = const __attribute__((address_space(4))) KernelArgs *;
__device__ __forceinline__ const KernelArgs &reread(ArgsAt at) {
  asm volatile("" : "+s"(at));
  return *(const KernelArgs *)at;
}

// These values stand in scalar registers here: their loads are issued together and waited for once. (Left to the compiler each
// was fetched where it was first used, ten waits one after the other: 64 heads x 128k tokens 1628 -> 1642 us, 1636 so.)
template <typename T>
__device__ __forceinline__ int arrived_one(T &x) {
  asm volatile("" : "+s"(x));
  return 0;
}
template <typename... T>
__device__ __forceinline__ void arrived(T &...x) {
  (void)(arrived_one(x) + ...);
}

// A pointer that came out of the arguments in memory, as one into global memory (unknown to the compiler, whose flat loads and
// stores count as LDS operations too: every wait for one kind then waits for the other).
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *in_global(T *p) {
  return (__attribute__((address_space(1))) T *)p;
}

template <bool RAGGED, bool GATHER, bool FAST>
__device__ __forceinline__ void prefill_items(ArgsAt args_at, unsigned char *lds, Shared &sh, bool from_list) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, hf = lane >> 5;
  const float c2 = reread(args_at).a.scale * 1.4426950408889634f;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)lds;

  // LDS byte offsets of this lane's operand fragments inside a block (layout note above), chunk pair 0
  // and dim block 0; the others differ by an XOR
  const int kbase = n * 256 + ((hf ^ (n & 15)) << 4);
  const int vbase = (4 * hf + ((n & 15) >> 2)) * 256 + (((n & 15) >> 2) << 6) + 32 * (n >> 4) + 8 * (n & 3);
  // load-to-LDS copies of a block: instruction `it` (0, 1) of wave w fills rows 16 it + 4 w .. + 3; a
  // lane's byte offset from the block's first row is constant
  const int sub = lane >> 4, pos = lane & 15;
  const int row0 = wave * 4 + sub;
  const unsigned kss2 = (unsigned)reread(args_at).a.k_ss * 2u, vss2 = (unsigned)reread(args_at).a.v_ss * 2u;  // row strides in bytes
  const unsigned koff = (unsigned)row0 * kss2 + ((pos ^ (row0 & 15)) << 4);
  const unsigned voff = (unsigned)row0 * vss2 + ((pos ^ (sub << 2)) << 4);
  const unsigned boff = (unsigned)((wave * 32 + n) * 16);  // this lane's row in a tile's mask words
  const int bits_addr = wave * 256 + lane * 4;             // where its copy lands inside a bits slot
  const unsigned lds_kv = __builtin_amdgcn_readfirstlane(lds_base + wave * 1024);              // this wave's part of a K/V slot
  const unsigned lds_bits = __builtin_amdgcn_readfirstlane(lds_base + kBitsRing + wave * 256);  // ... of a bits slot

  const int my_xcd = __builtin_amdgcn_s_getreg((3 << 11) | 20) & (kXcd - 1);  // XCC_ID, 4 bits
  uint2 *blk_list = reinterpret_cast<uint2 *>(lds + kBlkList);
  // The listed tiles [seg0, seg0 + n_seg) of an item that starts at t0 -> list of block descriptors in LDS (two words:
  // first key, and mask offset | flags << 28), closed by a dummy entry that every read past the end returns. By wave 0
  // alone, two tiles per lane: between two barriers, whatever the other waves do. In two steps, so that the loads of the
  // item's query rows can be issued behind those of its tiles and travel while the list is written.
  struct Tiles {
    int col[kSegTiles / 64], kind[kSegTiles / 64];
  };
  auto fetch_tiles = [&](const Operands &t, int seg0, int n_seg) {
    Tiles x;
#pragma unroll
    for (int half = 0; half < kSegTiles / 64; ++half) {
      const int at = seg0 + min(half * 64 + lane, n_seg - 1);
      x.col[half] = in_global(t.blk_col)[at];
      x.kind[half] = in_global(t.blk_kind)[at];
    }
    return x;
  };
  auto expand = [&](const AttnArgs &a, const Tiles &tiles, int t0, int seg0, int n_seg) {
    int before = 0;
#pragma unroll
    for (int half = 0; half < kSegTiles / 64; ++half) {
      const int x = half * 64 + lane;
      // a column outside the index's range (a list that was never filled) is pulled inside it: the result is
      // then wrong, but every address formed from it stays within the head's rows
      const int col = min(max(tiles.col[half], 0), a.nKt + (GATHER ? a.gather_rows / kBN : 0) - 1);
      int quarters = x < n_seg ? (tiles.kind[half] >> 1) & 15 : 0;
      const int full = tiles.kind[half] & 1;
      const int cnt = __popc(quarters);
      const int incl = wave_prefix(cnt);
      int at = before + incl - cnt;
      before += __builtin_amdgcn_readlane(incl, 63);
      while (quarters) {
        const int qq = __builtin_ctz(quarters);
        quarters &= quarters - 1;
        const bool gth = GATHER && col >= a.nKt;  // gathered tile: rows of the head's gathered copy (flag 4)
        const int key0 = gth ? min((col - a.nKt) * kBN + kBlkKeys * qq, a.gather_rows - kBlkKeys) : col * kBN + kBlkKeys * qq;
        const unsigned off_bits = (unsigned)((seg0 + x - t0) * (kBM * 16) + 4 * qq);
        blk_list[at++] = make_uint2((unsigned)key0, off_bits | (unsigned)(full | (gth ? 4 : 0)) << 28);
      }
      if (n_seg <= 64) break;
    }
    if (lane == 0) {
      blk_list[before] = make_uint2(0u, 2u << 28);  // dummy: key 0, the item's first mask words, nothing kept
      sh.nblk = before;
    }
  };
  // The queues. A workgroup's first item is its rank among those numbered for the same queue, without an atomic (all 512
  // of them start at once, and atomics on one counter are served one after the other: up to 7 us); the counters hand out
  // what follows.
  // Between two items the matrix pipe of the workgroup idles for a chain of round trips to memory, so each of them travels
  // under something else: wave 0 asks for the next item when the blocks of the one before are done, and the answer is under
  // way while the rows are divided; where the item's tiles lie, while the rows are turned around, and is looked at in front of
  // their stores (a load behind stores waits for them); the tiles in front of the query rows, and both while the list is
  // written; and the pipeline starts on its first block, with the copies of three more in flight. Atomic, look-up, list, query
  // rows and four blocks one after the other, with two more barriers, took 6.1 us an item where this takes 5.0: 4 x 32 heads x
  // 3001 tokens (19 blocks an item) 159.4 -> 153.0 us, 8 x 32 x 700 57.9 -> 55.6, 32 x 32768 1169 -> 1156, 64 x 128k captured
  // at 4096 9603 -> 9464 (whole layers). Asked in the item's last iterations: no gain, the wave's own copies in flight take
  // as long as the answer.
  auto queue_starts = [&](int qu) { return ((int)gridDim.x - qu + kXcd - 1) / kXcd; };
  int hop = 0;  // (wave 0) queue of the next draw
  // asks the first queue from `hop` on that hands out more than first items
  auto ask = [&](const Queues &qs, int *ctl) {
    int got = 0;
    while (hop < kXcd) {
      const int queue = (my_xcd + hop) & (kXcd - 1);
      if (qs.items(queue) > queue_starts(queue)) {
        if (lane == 0)
          got = __hip_atomic_fetch_add(in_global(ctl) + queue * kCtlStep, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      ++hop;
    }
    return got;
  };
  // the answer: an item and its queue, or -1
  auto answer = [&](const Queues &qs, int *ctl, int got, int &queue) {
    while (hop < kXcd) {
      queue = (my_xcd + hop) & (kXcd - 1);
      const int item = __builtin_amdgcn_readfirstlane(got) + queue_starts(queue);
      if (item < qs.items(queue)) return item;
      ++hop;
      got = ask(qs, ctl);
    }
    return -1;
  };
  // Where an item's listed tiles lie, fetched without waiting: lanes 1 and 2 the offsets, from the index or, with lane 0 the
  // item's number, from its entry in the order (`item` is then the place in it).
  auto ordered = [&](const Operands &t) { return (FAST || !from_list) && t.order; };
  auto look_up = [&](const Operands &t, const Queues &qs, int item, int queue) {
    const int *at = ordered(t) ? reinterpret_cast<const int *>(t.order + queue * kOrderMax + item) : qs.span(t.row_ptr, item, queue) - 1;
    return in_global(at)[min(max(lane, ordered(t) ? 0 : 1), 2)];
  };
  auto publish = [&](const Operands &t, const Queues &qs, int item, int e, int queue) {
    if (ordered(t) && item >= 0) item = __builtin_amdgcn_readlane(e, 0);
    const int pair = qs.pair_of(item, queue), within = qs.within_of(item, queue);
    const int wb = pair / qs.Hkv, whkv = pair % qs.Hkv;
    if (lane == 0) {
      sh.item[0] = make_int4(item, queue, __builtin_amdgcn_readlane(e, 1), __builtin_amdgcn_readlane(e, 2));
      sh.item[1] = make_int4(wb, whkv, whkv * qs.G + within % qs.G, qs.nQt - 1 - within / qs.G);
    }
  };
  if (wave == 0) {
    const KernelArgs &args = reread(args_at);
    const Queues qs(args.a);
    int item = -1, queue = blockIdx.x % kXcd;
    if (!FAST && from_list) {
      const int id = __builtin_amdgcn_readfirstlane(sh.redo);  // (not empty)
      item = id / kXcd;
      queue = id % kXcd;
      if (lane == 0) sh.redo = args.t.next[id];
    } else if ((int)blockIdx.x / kXcd < qs.items(queue)) {
      item = blockIdx.x / kXcd;
    } else {
      item = answer(qs, args.t.ctl, ask(qs, args.t.ctl), queue);
    }
    publish(args.t, qs, item, item < 0 ? 0 : look_up(args.t, qs, item, queue), queue);
  }
  int id = -1;  // (item, queue) as the redo list has it
  while (true) {
    // previous item: every wave is done with the LDS rings (its stores stay in flight), the next one is known
    KernelArgs args = reread(args_at);
    arrived(args.a.S, args.a.nKt, args.a.gather_rows, args.a.Hq, args.t.blk_col, args.t.blk_kind);
    arrived(args.t.q, args.t.k, args.t.v, args.t.tile_bits, args.a.q_sb, args.a.q_sh, args.a.q_ss, args.a.k_sb, args.a.k_sh, args.a.v_sb,
            args.a.v_sh);
    if (GATHER) arrived(args.t.kgath, args.t.vgath);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (FAST && wave == 0 && id >= 0 && sh.bad && lane == 0) {  // some row of the previous item needs the running reference
      args.t.next[id] = sh.redo;
      sh.redo = id;
      sh.bad = 0;
    }
    const int4 what = sh.item[0], where = sh.item[1];
    const int item = __builtin_amdgcn_readfirstlane(what.x), queue = __builtin_amdgcn_readfirstlane(what.y);
    if (item < 0) break;
    id = item * kXcd + queue;
    const AttnArgs &a = args.a;
    const int S = a.S;
    const int t0 = __builtin_amdgcn_readfirstlane(what.z), t1 = __builtin_amdgcn_readfirstlane(what.w);
    const int wb = __builtin_amdgcn_readfirstlane(where.x), whkv = __builtin_amdgcn_readfirstlane(where.y);
    const int whq = __builtin_amdgcn_readfirstlane(where.z), wqt = __builtin_amdgcn_readfirstlane(where.w);
    const int qrow_l = wave * 32 + n;  // this lane's query row inside the tile
    const int qrow = wqt * kBM + qrow_l;
    const bool qlive = qrow < S;
    const unsigned char *kg = reinterpret_cast<const unsigned char *>(args.t.k + wb * a.k_sb + whkv * a.k_sh);
    const unsigned char *vg = reinterpret_cast<const unsigned char *>(args.t.v + wb * a.v_sb + whkv * a.v_sh);
    // the head's gathered column rows (tiles with index >= nKt): [gather_rows] rows at the row stride of K
    // (of V), so that a block of them is addressed exactly like a block of the cache
    const int64_t g_rows = ((int64_t)wb * a.Hq + whq) * a.gather_rows;
    const unsigned char *kgg = reinterpret_cast<const unsigned char *>(args.t.kgath) + g_rows * kss2;
    const unsigned char *vgg = reinterpret_cast<const unsigned char *>(args.t.vgath) + g_rows * vss2;

    // ---- the stream of occupied 32-key blocks of this query tile. The listed tiles are expanded, kSegTiles at
    // a time, into a list of block descriptors in LDS. The pipeline then reads one descriptor per
    // iteration (fetched before the previous iteration's barrier, so that nothing waits for it) instead of
    // walking tiles and quarters in scalar code, which cost a sixth of the instructions of an iteration.
    int n_blk = 0;      // entries of the current list before the dummy
    int cursor = 0;     // index of the descriptor held in pre_raw
    uint2 pre_raw = make_uint2(0u, 2u << 28);
    auto list_read = [&](int i) { return blk_list[min(i, n_blk)]; };  // the same address in every lane
    auto decode = [&](const uint2 &raw) {
      const int key0 = __builtin_amdgcn_readfirstlane((int)raw.x);
      const unsigned meta = (unsigned)__builtin_amdgcn_readfirstlane((int)raw.y);
      return Blk{key0, (int)(meta & 0x0FFFFFFFu), (int)(meta >> 28)};
    };
    // K or V block -> ring slot: two 1 KiB copies per wave; every address is the head's base plus a
    // 32-bit byte offset (the host checks that a head's rows span less than 4 GiB). In the ragged case
    // a block that reaches past the sequence end redirects such keys (masked anyway) to the last row,
    // which keeps the slot finite.
    auto copy_blk = [&](auto slot_off, const unsigned char *g, unsigned stride2, unsigned lane_off, int chunk_xor, int key0,
                        unsigned blk_off, bool gathered) {
      constexpr int SO = decltype(slot_off)::value;
      if (!RAGGED || gathered || key0 + kBlkKeys <= S) {
        const unsigned o0 = lane_off + blk_off;
        lds_copy16<SO>(lds_kv, g, o0);
        lds_copy16<SO + 4096>(lds_kv, g, o0 + 16u * stride2);
      } else {
        const unsigned c = (unsigned)((pos ^ chunk_xor) << 4);
        lds_copy16<SO>(lds_kv, g, (unsigned)min(key0 + row0, S - 1) * stride2 + c);
        lds_copy16<SO + 4096>(lds_kv, g, (unsigned)min(key0 + 16 + row0, S - 1) * stride2 + c);
      }
    };
    auto copy_k = [&](const Blk &d, auto slot) {
      const bool gth = GATHER && (d.flags & 4) != 0;  // wave-uniform
      copy_blk(std::integral_constant<int, decltype(slot)::value * kBlkBytes>{}, gth ? kgg : kg, kss2, koff, row0 & 15, d.key0,
               (unsigned)d.key0 * kss2, gth);
    };
    auto copy_v = [&](const Blk &d, auto slot) {
      const bool gth = GATHER && (d.flags & 4) != 0;
      copy_blk(std::integral_constant<int, kVRing + decltype(slot)::value * kBlkBytes>{}, gth ? vgg : vg, vss2, voff, sub << 2, d.key0,
               (unsigned)d.key0 * vss2, gth);
    };
    // the block's mask word of every row of this wave (also issued for full and dummy blocks, so that
    // every iteration has the same number of copies in flight)
    const unsigned char *bits_row = reinterpret_cast<const unsigned char *>(args.t.tile_bits) + (int64_t)t0 * (kBM * 16);
    auto copy_bits = [&](const Blk &d, auto slot) {
      lds_copy4<decltype(slot)::value * 1024>(lds_bits, bits_row, boff + (unsigned)d.bits_off);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;

    // block i of the stream is described by d[i & 3]
    Blk d[4] = {};
    f32x16 oacc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) oacc[db][e] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;  // running max (raw logits) and this lane's part of the row sum
    unsigned seen = 0u;                     // FAST: union of the mask words of this lane's row, and whether a full
    int seen_full = 0;                      // tile was met: together "the row has a kept entry"

    if (t1 > t0) {
      // the first segment's tiles (wave 0), then the Q fragments, B operand of S^T = K Q^T: chunk c covers dims
      // 16c .. 16c+15; this lane holds dims 16c + 8 hf .. + 7 of its query row. (A row past the sequence's end is its last
      // one: nothing is kept for it, and nothing of it stored.)
      const int n_first = min(kSegTiles, t1 - t0);
      Tiles tiles;
      if (wave == 0) tiles = fetch_tiles(args.t, t0, n_first);
      bf16x8 qf[8];
      {
        const auto qp = in_global(args.t.q + wb * a.q_sb + whq * a.q_sh + (int64_t)min(qrow, S - 1) * a.q_ss + 8 * hf);
#pragma unroll
        for (int c = 0; c < 8; ++c)
          qf[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const __attribute__((address_space(1))) u32x4 *>(qp + 16 * c));
      }
      if (wave == 0) expand(a, tiles, t0, t0, n_first);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      // one pass of the pipeline per segment of kSegTiles listed tiles (a query tile of c3 has at most 32;
      // the accumulators, the softmax state and the Q fragments carry over)
      for (int seg0 = t0; seg0 < t1; seg0 += kSegTiles) {
        if (seg0 > t0) {
          __syncthreads();  // every wave is done with the previous list and with the rings
          if (wave == 0) {
            const KernelArgs &again = reread(args_at);
            const int n_seg = min(kSegTiles, t1 - seg0);
            expand(again.a, fetch_tiles(again.t, seg0, n_seg), t0, seg0, n_seg);
          }
          __syncthreads();
        }
        // the Q fragments are waited for here (the compiler waits in front of an empty statement that takes them), before
        // there are copies in flight, which the compiler cannot count: it would wait for all of them at the first use of a
        // fragment in each iteration
#pragma unroll
        for (int c = 0; c < 8; ++c) asm volatile("" : "+v"(qf[c]));
        n_blk = __builtin_amdgcn_readfirstlane(sh.nblk);
        d[0] = decode(list_read(0));
        d[1] = decode(list_read(1));
        d[2] = decode(list_read(2));
        cursor = 3;
        pre_raw = list_read(cursor);
        copy_k(d[0], I0{});
        copy_bits(d[0], I0{});
        copy_k(d[1], I1{});
        copy_bits(d[1], I1{});
        copy_k(d[2], I2{});
        copy_bits(d[2], I2{});
        copy_v(d[0], I0{});
        // the first block's K and mask words; the eight copies behind them count like those of two iterations
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        // The variant with a reference multiplies the zero weights of the leading dummy blocks too, with V slots 2 and 3,
        // which therefore have to be finite: not what an earlier kernel or item left there, whose V may hold an infinity
        // or a NaN. (FAST leaves those products out. Each wave clears what it copies itself: nothing of its is in flight.)
        if constexpr (!FAST) {
#pragma unroll
          for (int x = 0; x < 4; ++x)
            *reinterpret_cast<uint4 *>(lds + kVRing + 2 * kBlkBytes + x * 4096 + wave * 1024 + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();
        // S_b lives in sbuf[PH & 1] and S_{b+1} is written to the other one; P_b goes to pbuf[PH & 1] and
        // P_{b-1} is read from the other one, so nothing is copied between iterations
        f32x16 sbuf[2];
        unsigned pbuf[2][8];
#pragma unroll
        for (int e = 0; e < 16; ++e) sbuf[0][e] = -INFINITY;  // block -1 is a dummy
#pragma unroll
        for (int e = 0; e < 8; ++e) pbuf[1][e] = 0u;
        d[3].flags = 0;  // stands for block -1: the leading dummy must not end the loop
        // iteration b with (b + 1) % 4 == PH; returns true when the stream is finished
        auto step = [&](auto ph, auto partc) {
          constexpr int PH = decltype(ph)::value, PART = decltype(partc)::value;
          const int flag_cur = d[(PH + 3) & 3].flags;  // block b, whose descriptor is replaced now
          if constexpr (FAST) {

            // the bookkeeping of this iteration, dealt out over the segments of the product stream: the copies
            // only behind the last operand reads (segments 0 .. 3 issue those of segments 4 .. 7)
            auto bk = [&](auto, int x) {
              if (x == 2) d[(PH + 3) & 3] = decode(pre_raw);           // block b+4
              if (x == 4) copy_k(d[(PH + 3) & 3], std::integral_constant<int, (PH + 3) & 3>{});  // five copies per wave and iteration, always
              if (x == 5) copy_bits(d[(PH + 3) & 3], std::integral_constant<int, (PH + 3) & 3>{});
              if (x == 6) copy_v(d[(PH + 1) & 3], std::integral_constant<int, (PH + 1) & 3>{});  // block b+2
              if (x == 7) pre_raw = list_read(++cursor);               // block b+5 (a read past the list returns its dummy)
            };
            pipe_iter_seg<PH, PART>(lds, qf, oacc, sbuf[PH & 1], sbuf[(PH + 1) & 1], pbuf[(PH + 1) & 1], pbuf[PH & 1], l_run,
                                    seen, seen_full, d[PH].flags, bits_addr, c2, kbase, vbase, hf, bk);
            if (flag_cur & 2) return true;      // block b was the trailing dummy: P_{b-1} V_{b-1} is in
          } else {
            d[(PH + 3) & 3] = decode(pre_raw);           // block b+4
            copy_k(d[(PH + 3) & 3], std::integral_constant<int, (PH + 3) & 3>{});  // five copies per wave and iteration, always
            copy_bits(d[(PH + 3) & 3], std::integral_constant<int, (PH + 3) & 3>{});
            copy_v(d[(PH + 1) & 3], std::integral_constant<int, (PH + 1) & 3>{});  // block b+2
            pipe_iter<PH, FAST>(lds, qf, oacc, sbuf[PH & 1], sbuf[(PH + 1) & 1], pbuf[(PH + 1) & 1], pbuf[PH & 1], m_run,
                                l_run, seen, seen_full, d[PH].flags, bits_addr, c2, kbase, vbase, hf);
            if (flag_cur & 2) return true;      // block b was the trailing dummy: P_{b-1} V_{b-1} is in
            pre_raw = list_read(++cursor);      // block b+5, decoded at the start of the next iteration
          }
          // K_{b+2}, its mask words and V_b (issued two iterations ago) must have landed; the ten
          // youngest copies (this iteration's and the previous one's) may stay in flight
          // (wait and barrier as one statement: the library barrier would add a fence that waits for
          // everything in flight; the LDS rings are only written by the copies counted here)
          asm volatile("s_waitcnt vmcnt(10)\n\ts_barrier" ::: "memory");
          return false;
        };
        using PAll = std::integral_constant<int, kAll>;
        // block -1 (nothing to weigh, nothing to add) and block 0 (nothing to add yet) in front of the loop,
        // which therefore starts at phase 2
        if (!step(I0{}, std::integral_constant<int, FAST ? kChainOnly : kAll>{}) &&
            !step(I1{}, std::integral_constant<int, FAST ? kNoPV : kAll>{})) {
          // (from a line of the instruction cache on, wherever the code in front of it ends: up to 0.5 %)
          asm volatile(".p2align 6" ::: "memory");
          while (true) {
            if (step(I2{}, PAll{})) break;
            if (step(I3{}, PAll{})) break;
            if (step(I0{}, PAll{})) break;
            if (step(I1{}, PAll{})) break;
          }
        }
      }
    } else {
      asm volatile("s_barrier" ::: "memory");  // (the next item is not written before every wave has this one)
    }

    // finish: total sum over both half-waves, normalise, store. Accumulator e of block db is dim
    // 32 db + 8 (e / 4) + 4 hf + e % 4 of this lane's query.
    KernelArgs end = reread(args_at);
    arrived(end.t.out, end.t.lse, end.a.o_sb, end.a.o_sh, end.a.o_ss, end.a.Hq, end.a.B, end.a.Hkv, end.a.nQt, end.t.ctl, end.t.order,
            end.t.row_ptr);
    const Queues qs(end.a);
    int got = 0;
    if (wave == 0 && !(!FAST && from_list)) got = ask(qs, end.t.ctl);
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    if (FAST) {
      // a row with a kept entry whose sum of weights is zero, tiny, huge, infinite or NaN: its logits lie outside
      // what exp2 without a reference can carry (|logit * log2 e| of the order of 100)
      const bool bad = qlive && (seen != 0u || seen_full) && !(l_tot >= 0x1p-100f && l_tot <= 0x1p100f);
      if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) sh.bad = 1;  // read by wave 0 after the loop's barrier
    }
    uint2 pr[16];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        pr[4 * db + g].x = pack_bf16(oacc[db][4 * g] * inv, oacc[db][4 * g + 1] * inv);
        pr[4 * db + g].y = pack_bf16(oacc[db][4 * g + 2] * inv, oacc[db][4 * g + 3] * inv);
        asm volatile("" : "+v"(pr[4 * db + g].x), "+v"(pr[4 * db + g].y));  // (while the answer is on its way)
      }
    int next = -1, next_queue = 0, next_at = 0;
    if (wave == 0) {
      if (!FAST && from_list) {
        const int next_id = __builtin_amdgcn_readfirstlane(sh.redo);
        if (next_id >= 0) {
          next = next_id / kXcd;
          next_queue = next_id % kXcd;
          if (lane == 0) sh.redo = end.t.next[next_id];
        }
      } else {
        next = answer(qs, end.t.ctl, got, next_queue);
      }
    }
    // The rows go out as whole 256-byte lines: a lane holds eight bytes here and there of its query's row, so the wave
    // turns its 32 rows around in LDS (16-byte chunk c of row r at c ^ (r & 15)) and every store instruction then covers
    // four rows. (Eight bytes per lane and store straight from the accumulators: 2.6 us per item until the stores had
    // drained, up to 20 us with every workgroup storing at once.) The place is the 8 KiB of the K ring that this wave's own
    // copies fill (four rows at 1024 wave of every 4 KiB), so nobody else is waited for: its own copies have landed, and
    // what the other waves still read of K in their last iteration belongs to no block.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); the builtin, so that the compiler knows and waits for nothing below
    asm volatile("" ::: "memory");
    if (wave == 0 && next >= 0) next_at = look_up(end.t, qs, next, next_queue);
    {
      int l = lane;  // (opaque, or the addresses below are computed once for all items and kept through the pipeline)
      asm volatile("" : "+v"(l));
      unsigned char *turn = lds + wave * 1024;
      unsigned char *row_at = turn + ((l & 31) >> 2) * 4096 + (l & 3) * 256 + 8 * (l >> 5);
#pragma unroll
      for (int x = 0; x < 16; ++x) *reinterpret_cast<uint2 *>(row_at + ((x ^ (l & 15)) << 4)) = pr[x];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      u32x4 line[8];
#pragma unroll
      for (int it = 0; it < 8; ++it)
        line[it] = *reinterpret_cast<const u32x4 *>(turn + it * 4096 + (l >> 4) * 256 + (((l & 15) ^ ((4 * it + (l >> 4)) & 15)) << 4));
      if (wave == 0) {
        asm volatile("" : "+v"(next_at));  // (looked at here, not where it was fetched)
        publish(end.t, qs, next, next_at, next_queue);
      }
      const int row_first = wqt * kBM + wave * 32;
      auto op = in_global(end.t.out + wb * end.a.o_sb + whq * end.a.o_sh + (int64_t)(row_first + (l >> 4)) * end.a.o_ss + 8 * (l & 15));
      const int64_t four_rows = 4 * end.a.o_ss;
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        if (row_first + 4 * it + (l >> 4) < S) *reinterpret_cast<__attribute__((address_space(1))) u32x4 *>(op) = line[it];
        op += four_rows;
      }
    }
    if (qlive && end.t.lse && hf == 0)
      in_global(end.t.lse)[((int64_t)wb * end.a.Hq + whq) * S + qrow] =
          l_tot > 0.0f ? ((FAST ? 0.0f : m_run * c2) + log2f(l_tot)) * 0.6931471805599453f : -INFINITY;
  }  // next work item
}

// The second variant behind the first is a function of its own, called when there is something on the list: inlined, it
// spilled registers of the first.
template <bool RAGGED, bool GATHER>
__device__ __attribute__((noinline)) void prefill_with_reference(uint64_t args_at, __attribute__((address_space(3))) unsigned char *lds,
                                                                 __attribute__((address_space(3))) Shared *sh) {
  // (an argument in vector registers, the same in every lane)
  const uint64_t at = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(args_at >> 32)) << 32 |
                      (unsigned)__builtin_amdgcn_readfirstlane((int)args_at);
  prefill_items<RAGGED, GATHER, false>((ArgsAt)at, (unsigned char *)lds, *(Shared *)sh, true);
}

// FAST = false: every item with the running reference (DAM_ATTN_RUNNING_REFERENCE).
template <bool RAGGED, bool GATHER, bool FAST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_prefill_bf16_pipe(KernelArgs) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  __shared__ Shared sh;
  const int tid = threadIdx.x;
  if (tid == 0) {
    sh.bad = 0;
    sh.redo = -1;
  }
  const ArgsAt args_at = (ArgsAt)__builtin_amdgcn_kernarg_segment_ptr();
  prefill_items<RAGGED, GATHER, FAST>(args_at, lds, sh, false);
  if constexpr (FAST) {
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(sh.redo) < 0) return;
    __syncthreads();  // (wave 0 takes the first entry off the list at once: every wave has seen that there is one)
    prefill_with_reference<RAGGED, GATHER>((uint64_t)args_at, (__attribute__((address_space(3))) unsigned char *)lds,
                                           (__attribute__((address_space(3))) Shared *)&sh);
  }
}

// Copies of the K and V rows of every head's matched columns (gather_idx, -1 = empty slot -> zeros) as
// [batch][hq][gather_rows] rows at the row stride of K (of V), so that a gathered tile is loaded like any other.
__global__ __launch_bounds__(256) void k_gather_kv(AttnArgs a, const __hip_bfloat16 *__restrict__ k,
                                                   const __hip_bfloat16 *__restrict__ v, const int *__restrict__ gather_idx,
                                                   __hip_bfloat16 *__restrict__ kgath, __hip_bfloat16 *__restrict__ vgath,
                                                   int *__restrict__ queue_next, const int *__restrict__ row_ptr,
                                                   const uint8_t *__restrict__ blk_kind, int4 *__restrict__ order) {
  // (also prepares the work queues of the attention kernel that follows: one launch less per call. The workgroups that
  // order them come first.)
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kCtlWords) queue_next[threadIdx.x * kCtlStep] = 0;
  const int lead = order ? kXcd : 0;  // rows of the grid in front
  if ((int)blockIdx.y < lead) {
    if (blockIdx.x == 0) order_items<256>(a, row_ptr, blk_kind, blockIdx.y, order);
    return;
  }
  const int bh = blockIdx.y - lead, b = bh / a.Hq, hq = bh % a.Hq, hkv = hq / (a.Hq / a.Hkv);
  const int s = blockIdx.x * 16 + (threadIdx.x >> 4), chunk = threadIdx.x & 15;
  if (s >= a.gather_rows) return;
  const int c = s < a.gather_stride ? gather_idx[(int64_t)hq * a.gather_stride + s] : -1;
  uint4 kv = make_uint4(0u, 0u, 0u, 0u), vv = kv;
  if (c >= 0 && c < a.S) {
    kv = *reinterpret_cast<const uint4 *>(k + b * a.k_sb + hkv * a.k_sh + (int64_t)c * a.k_ss + chunk * 8);
    vv = *reinterpret_cast<const uint4 *>(v + b * a.v_sb + hkv * a.v_sh + (int64_t)c * a.v_ss + chunk * 8);
  }
  const int64_t row = (int64_t)bh * a.gather_rows + s;
  *reinterpret_cast<uint4 *>(kgath + row * a.k_ss + chunk * 8) = kv;
  *reinterpret_cast<uint4 *>(vgath + row * a.v_ss + chunk * 8) = vv;
}

__global__ __launch_bounds__(kOrderMax) void k_order_items(AttnArgs a, int *__restrict__ queue_next, const int *__restrict__ row_ptr,
                                                      const uint8_t *__restrict__ blk_kind, int4 *__restrict__ order) {
  if (threadIdx.x == 0) queue_next[blockIdx.x * kCtlStep] = 0;
  if (order) order_items<kOrderMax>(a, row_ptr, blk_kind, blockIdx.x, order);
}

int validate(const dam_attn_params *p, const void *q, const void *k, const void *v, const dam_mask_view *mk,
             const void *out) {
  if (!p || !q || !k || !v || !mk || !out) return DAM_ERR_INVALID_ARG;
  if (!mk->blk_row_ptr || !mk->blk_col || !mk->blk_kind || !mk->tile_bits) return DAM_ERR_INVALID_ARG;
  if (p->batch < 1 || p->hq < 1 || p->hkv < 1 || p->hq % p->hkv || p->seq < 1) return DAM_ERR_INVALID_ARG;
  if (p->tile_m < 64 || p->tile_n < 64 || p->tile_m % 64 || p->tile_n % 64) return DAM_ERR_INVALID_ARG;
  if (mk->gather_idx) {  // gathered column tiles (checked after the tile sizes: the test divides by tile_n)
    if (!mk->gather_cnt || mk->gather_stride < 1 || p->gather_rows < 0 || p->gather_rows % p->tile_n ||
        p->gather_rows > mk->gather_stride)
      return DAM_ERR_INVALID_ARG;
  } else if (p->gather_rows != 0) {
    return DAM_ERR_INVALID_ARG;
  }
  if (!(p->scale >= 0.0f)) return DAM_ERR_INVALID_ARG;
  if (p->flags & ~DAM_ATTN_RUNNING_REFERENCE) return DAM_ERR_INVALID_ARG;
  const int align = p->dtype == DAM_BF16 ? 8 : 4;
  const int64_t *sets[4] = {p->q_stride, p->k_stride, p->v_stride, p->o_stride};
  for (auto s : sets)
    for (int x = 0; x < 3; ++x)
      if (s[x] < 0 || s[x] % align) return DAM_ERR_INVALID_ARG;
  if (p->dtype == DAM_BF16) {
    if (p->head_dim != 128 || p->tile_m != 128 || p->tile_n != 128) return DAM_ERR_UNSUPPORTED;
    // the bf16 kernel addresses the rows of one K or V head with 32-bit byte offsets
    if ((int64_t)p->seq * p->k_stride[2] * 2 >= (int64_t(1) << 32) || (int64_t)p->seq * p->v_stride[2] * 2 >= (int64_t(1) << 32))
      return DAM_ERR_UNSUPPORTED;
  } else if (p->dtype == DAM_F32) {
    if (p->head_dim != 64 && p->head_dim != 128) return DAM_ERR_UNSUPPORTED;
    if (p->tile_m > 128 || p->tile_n > 128) return DAM_ERR_UNSUPPORTED;
  } else {
    return DAM_ERR_UNSUPPORTED;
  }
  return DAM_OK;
}

AttnArgs make_args(const dam_attn_params *p) {
  AttnArgs a;
  a.B = p->batch; a.Hq = p->hq; a.Hkv = p->hkv; a.S = p->seq;
  a.tile_m = p->tile_m; a.tile_n = p->tile_n;
  a.nQt = (p->seq + p->tile_m - 1) / p->tile_m;
  a.nKt = (p->seq + p->tile_n - 1) / p->tile_n;
  a.gather_rows = 0;
  a.gather_stride = 0;
  a.wpr = p->tile_n / 64;
  a.scale = p->scale > 0.0f ? p->scale : 1.0f / sqrtf((float)p->head_dim);
  a.q_sb = p->q_stride[0]; a.q_sh = p->q_stride[1]; a.q_ss = p->q_stride[2];
  a.k_sb = p->k_stride[0]; a.k_sh = p->k_stride[1]; a.k_ss = p->k_stride[2];
  a.v_sb = p->v_stride[0]; a.v_sh = p->v_stride[1]; a.v_ss = p->v_stride[2];
  a.o_sb = p->o_stride[0]; a.o_sh = p->o_stride[1]; a.o_ss = p->o_stride[2];
  return a;
}

}  // namespace

// bytes of the redo lists' links: a word per (batch, query head, query tile) and one per queue, rounded up to 256
static size_t redo_bytes(const dam_attn_params *p) {
  const size_t items = (size_t)p->batch * p->hq * (size_t)((p->seq + p->tile_m - 1) / p->tile_m);
  return ((items + kXcd) * sizeof(int) + 255) / 256 * 256;
}

// Items from which they are taken by length: with fewer most are some workgroup's first one and the look-up costs more than the
// order brings (512 workgroups on this chip; 576 items 39.8 us by number, 41.7 by length, 960 items 53.5 / 52).
constexpr int64_t kOrderMin = 768;

// bytes of the queues' order, in the workspace of every call that a smaller one of kOrderMin items or more may share
static size_t order_bytes(int64_t items) { return items >= kOrderMin ? (size_t)kXcd * kOrderMax * sizeof(int4) : 0; }

// the control words of the bf16 kernel (queue counters), the links of the redo lists, then the gathered K and V copies
// (rows at the caches' strides); what the kernel cannot do without
static size_t least_bytes(const dam_attn_params *p) {
  return kCtlBytes + redo_bytes(p) +
         (size_t)p->batch * p->hq * p->gather_rows * (size_t)(p->k_stride[2] + p->v_stride[2]) * sizeof(__hip_bfloat16);
}

extern "C" size_t dam_sparse_attn_prefill_workspace(const dam_attn_params *p) {
  if (!p || p->batch < 1 || p->hkv < 1 || p->hq < 1 || p->seq < 1 || p->gather_rows < 0) return 0;
  if (p->dtype != DAM_BF16) return 0;
  if (p->hq % p->hkv || p->tile_m < 64) return 0;
  return least_bytes(p) + order_bytes((int64_t)p->batch * p->hq * ((p->seq + p->tile_m - 1) / p->tile_m));
}

extern "C" int dam_sparse_attn_prefill(const dam_attn_params *p, const void *q, const void *k, const void *v,
                                       const dam_mask_view *mk, void *out, float *lse, void *ws, size_t ws_bytes,
                                       void *stream_v) {
  const int bad = validate(p, q, k, v, mk, out);
  if (bad != DAM_OK) return bad;
  // (a workspace without room for the order does without it)
  if (p->dtype == DAM_BF16 && (!ws || ws_bytes < least_bytes(p))) return DAM_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream_v);
  AttnArgs a = make_args(p);
  if (mk->gather_idx) {
    a.gather_rows = p->gather_rows;
    a.gather_stride = mk->gather_stride;
  }
  if (p->dtype == DAM_F32) {
    // (a list shorter than a tile's slots holds no gathered tile, and the kernel that looks slots up would read past it)
    const bool looks_up = mk->gather_idx && mk->gather_stride >= p->tile_n;
    const int groups = p->batch * p->hq * a.nQt * (p->tile_m / 16);
    const F32Args t{a, (const float *)q, (const float *)k, (const float *)v, mk->blk_row_ptr, mk->blk_col, mk->blk_kind, mk->tile_bits,
                    mk->gather_idx, (float *)out, lse};
    if (groups <= kF32Few) {
      auto kern = looks_up ? (p->head_dim == 64 ? k_prefill_f32_few<64, true> : k_prefill_f32_few<128, true>)
                           : (p->head_dim == 64 ? k_prefill_f32_few<64, false> : k_prefill_f32_few<128, false>);
      kern<<<groups, 256, 0, st>>>(a, t.q, t.k, t.v, t.row_ptr, t.blk_col, t.blk_kind, t.tile_bits, t.gather_idx, t.out, t.lse);
    } else {
      auto kern = looks_up ? (p->head_dim == 64 ? k_prefill_f32<64, true> : k_prefill_f32<128, true>)
                           : (p->head_dim == 64 ? k_prefill_f32<64, false> : k_prefill_f32<128, false>);
      kern<<<groups, 256, 0, st>>>(t);
    }
    return launch_status();
  }
  const int blocks = p->batch * p->hq * a.nQt;  // work items
  // (queried per call: the library keeps no state, and the device may differ from call to call)
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    return DAM_ERR_DEVICE;
  int *ctl = static_cast<int *>(ws);
  int *next = reinterpret_cast<int *>(static_cast<char *>(ws) + kCtlBytes);
  __hip_bfloat16 *kgath = reinterpret_cast<__hip_bfloat16 *>(static_cast<char *>(ws) + kCtlBytes + redo_bytes(p));
  __hip_bfloat16 *vgath = kgath + (size_t)p->batch * p->hq * a.gather_rows * (size_t)a.k_ss;
  int4 *order = nullptr;
  const bool even = p->batch * p->hkv % kXcd == 0;
  const int longest_queue = even ? blocks / kXcd : (blocks + kXcd - 1) / kXcd;
  if (blocks > 2 * n_cu && blocks >= kOrderMin && longest_queue <= kOrderMax && ws_bytes >= least_bytes(p) + order_bytes(blocks))
    order = reinterpret_cast<int4 *>(static_cast<char *>(ws) + least_bytes(p));
  if (a.gather_rows > 0)
    k_gather_kv<<<dim3((a.gather_rows + 15) / 16, p->batch * p->hq + (order ? kXcd : 0)), 256, 0, st>>>(
        a, (const __hip_bfloat16 *)k, (const __hip_bfloat16 *)v, mk->gather_idx,
        kgath, vgath, ctl, mk->blk_row_ptr, mk->blk_kind, order);
  else if (blocks > 2 * n_cu)  // (fewer items are all first items: no counter is asked)
    k_order_items<<<kXcd, kOrderMax, 0, st>>>(a, ctl, mk->blk_row_ptr, mk->blk_kind, order);
  const int persistent = std::min(blocks, 2 * n_cu);  // two workgroups fit a CU (registers and LDS)
  const bool ragged = p->seq % kBlkKeys != 0, gather = a.gather_rows > 0;
  using Kernel = void (*)(KernelArgs);
  static const Kernel kernels[2][4] = {
      {k_prefill_bf16_pipe<false, false, false>, k_prefill_bf16_pipe<true, false, false>,
       k_prefill_bf16_pipe<false, true, false>, k_prefill_bf16_pipe<true, true, false>},
      {k_prefill_bf16_pipe<false, false, true>, k_prefill_bf16_pipe<true, false, true>,
       k_prefill_bf16_pipe<false, true, true>, k_prefill_bf16_pipe<true, true, true>}};
  const Kernel kern = kernels[(p->flags & DAM_ATTN_RUNNING_REFERENCE) ? 0 : 1][(ragged ? 1 : 0) + (gather ? 2 : 0)];
  // (idempotent; set on every call rather than remembered in a static)
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kPipeLds) != hipSuccess)
    return DAM_ERR_DEVICE;
  const KernelArgs t{a, {(const __hip_bfloat16 *)q, (const __hip_bfloat16 *)k, (const __hip_bfloat16 *)v, mk->blk_row_ptr, mk->blk_col,
                   mk->blk_kind, mk->tile_bits, (__hip_bfloat16 *)out, lse, ctl, next, order, kgath, vgath}};
  kern<<<persistent, 256, kPipeLds, st>>>(t);
  return launch_status();
}

extern "C" int dam_version(void) { return 1; }
