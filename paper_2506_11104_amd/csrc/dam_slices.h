// Sec. 4.2.4 numerators, shared by the mask builder and the capture: kept entries per column and per diagonal of 128 rows of
// the true mask, counted with carry-save adders on whole 64-bit words. A thread owns one word (64 columns) of some of the
// rows and adds the row words into a bit-sliced counter (slice k holds bit k of the 64 column counts). For the diagonals the
// row word is first re-aligned: word l of row i then holds m[i][i - r] for r = 64 l .. 64 l + 63, highest r first (a funnel
// shift of two adjacent words), after which diagonals are columns. The slices of every chunk of rows go to the workspace;
// k_pattern_finish sums them per pattern and applies the ratio test. No atomics.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dam {

constexpr int kChunkRows = 128;
constexpr int kSlices = 8;        // counts 0 .. 128
constexpr int kThreadSlices = 7;  // of one thread: at most 64 rows
constexpr size_t kSliceLds = (size_t)2 * 256 * kThreadSlices * sizeof(uint64_t);

// A full adder on 64 counters at once: sum and majority of three words, an instruction per 32-bit half each.
__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  const unsigned lo = __builtin_amdgcn_bitop3_b32((unsigned)a, (unsigned)b, (unsigned)c, 0x96);
  const unsigned hi = __builtin_amdgcn_bitop3_b32((unsigned)(a >> 32), (unsigned)(b >> 32), (unsigned)(c >> 32), 0x96);
  return (uint64_t)hi << 32 | lo;
}
__device__ __forceinline__ uint64_t majority(uint64_t a, uint64_t b, uint64_t c) {
  const unsigned lo = __builtin_amdgcn_bitop3_b32((unsigned)a, (unsigned)b, (unsigned)c, 0xE8);
  const unsigned hi = __builtin_amdgcn_bitop3_b32((unsigned)(a >> 32), (unsigned)(b >> 32), (unsigned)(c >> 32), 0xE8);
  return (uint64_t)hi << 32 | lo;
}
__device__ __forceinline__ void csa(uint64_t &carry, uint64_t &sum, uint64_t a, uint64_t b, uint64_t c) {
  const uint64_t m = majority(a, b, c);
  sum = xor3(a, b, c);
  carry = m;
}

// Eight words into a bit-sliced counter of N slices.
template <int N>
__device__ __forceinline__ void add_eight(uint64_t (&s)[N], const uint64_t (&w)[8]) {
  uint64_t t0, t1, f0, f1, e;
  csa(t0, s[0], s[0], w[0], w[1]);
  csa(t1, s[0], s[0], w[2], w[3]);
  csa(f0, s[1], s[1], t0, t1);
  csa(t0, s[0], s[0], w[4], w[5]);
  csa(t1, s[0], s[0], w[6], w[7]);
  csa(f1, s[1], s[1], t0, t1);
  csa(e, s[2], s[2], f0, f1);
#pragma unroll
  for (int k = 3; k < N; ++k) {  // the eights ripple up
    const uint64_t c = s[k] & e;
    s[k] ^= e;
    e = c;
  }
}

// One chunk of 128 rows by a workgroup of 256 threads, both pattern kinds from one reading of the rows' words up to the
// diagonal. tb: the chunk's first row; rows of them exist; tbw <= 128 words per row. sm: kSliceLds bytes of LDS.
// vout, dout: [tbw][kSlices] of this chunk.
// W = the number of words up to the diagonal rounded up to a power of two; thread t owns word t % W of the rows t / W,
// t / W + 256 / W, ...: for the columns that is the word it has loaded, for the diagonals two words of the same row, which
// its neighbours have loaded and pass on through LDS. Up to 64 words a row lies within one wave, so the only barriers are
// those around the last addition, and a wave has its next eight words in flight while it counts the ones before.
// Bound by the vector ALU: some 40 instructions per word and lane, of which the two counters are 11 and the window 9. 64 maps of
// 4096 x 4096: 48.5 -> 25.5 us (five operations per full adder, 64-bit shifts, index tests, barriers around a copy of 64 whole
// rows), and half as many chunk counts for k_pattern_finish.
__device__ __forceinline__ void count_chunk(const uint64_t *__restrict__ tb, int rows, int tbw, int chunk, uint64_t *sm,
                                            uint64_t *__restrict__ vout, uint64_t *__restrict__ dout) {
  const int tid = threadIdx.x;
  const int wmax = min(tbw, 2 * chunk + 2);  // words that can hold a kept entry of these rows
  int W = 16;
  while (W < wmax) W *= 2;
  const int wl = tid & (W - 1), sub = tid / W, nsub = 256 / W, n_batch = W / 16;
  auto sync = [&] {
    if (W > 64) {  // workgroup-uniform
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  };
  uint64_t next[8];
  const int last = wl < wmax ? rows : 0;  // rows this thread has a word of
  const uint64_t *mine = tb + min(wl, wmax - 1);
  auto load = [&](int b) {
#pragma unroll
    for (int u = 0; u < 8; ++u) next[u] = mine[min(sub + nsub * (8 * b + u), rows - 1) * tbw];
  };
  // The staged rows: two zero words in front of each, so that a word left of the row's first reads as nothing without a
  // test (one right of its last meets the zeros of the row behind; two more stand behind the last row).
  const int stride = W + 2;
  uint64_t *const stage = sm + sub * stride + 2;  // row (u, sub) lies u * nsub rows further
  for (int x = tid; x < 2 * (8 * nsub + 1); x += 256) sm[(x >> 1) * stride + (x & 1)] = 0;
  __syncthreads();
  uint64_t sc[kThreadSlices], sd[kThreadSlices];
#pragma unroll
  for (int k = 0; k < kThreadSlices; ++k) sc[k] = sd[k] = 0;
  load(0);
  for (int b = 0; b < n_batch; ++b) {
    uint64_t c[8], d[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      c[u] = sub + nsub * (8 * b + u) < last ? next[u] : 0;
      stage[u * nsub * stride + wl] = c[u];
    }
    sync();
    if (b + 1 < n_batch) load(b + 1);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = sub + nsub * (8 * b + u);
      const uint64_t *at = stage + u * nsub * stride + max(2 * chunk + (r >> 6) - wl, -1);  // word of column i - 64 wl
      // the window: bits up to r % 64 of hi, the rest from the top of lo; as 32-bit funnel shifts, first by one
      const uint64_t hi = at[0], lo = at[-1];
      const unsigned d0 = (unsigned)lo, d1 = (unsigned)(lo >> 32), d2 = (unsigned)hi, d3 = (unsigned)(hi >> 32);
      const unsigned e0 = __builtin_amdgcn_alignbit(d1, d0, 1), e1 = __builtin_amdgcn_alignbit(d2, d1, 1);
      const unsigned e2 = __builtin_amdgcn_alignbit(d3, d2, 1), e3 = d3 >> 1;
      const bool far = (r & 32) != 0;
      const unsigned f0 = far ? e1 : e0, f1 = far ? e2 : e1, f2 = far ? e3 : e2;
      d[u] = (uint64_t)__builtin_amdgcn_alignbit(f2, f1, r & 31) << 32 | __builtin_amdgcn_alignbit(f1, f0, r & 31);
    }
    sync();
    add_eight(sc, c);
    add_eight(sd, d);
  }
  __syncthreads();  // the row words are no longer needed: their place takes the partial counters
#pragma unroll
  for (int k = 0; k < kThreadSlices; ++k) {
    sm[((0 * nsub + sub) * kThreadSlices + k) * W + wl] = sc[k];
    sm[((1 * nsub + sub) * kThreadSlices + k) * W + wl] = sd[k];
  }
  __syncthreads();
  if (tid < 2 * W) {
    const int kind = tid / W;  // 0 columns, 1 diagonals
    uint64_t acc[kSlices];
#pragma unroll
    for (int k = 0; k < kSlices; ++k) acc[k] = 0;
    for (int x = 0; x < nsub; ++x) {
      uint64_t carry = 0;
#pragma unroll
      for (int k = 0; k < kSlices; ++k)
        csa(carry, acc[k], acc[k], k < kThreadSlices ? sm[((kind * nsub + x) * kThreadSlices + k) * W + wl] : 0, carry);
    }
    if (wl < tbw) {
#pragma unroll
      for (int k = 0; k < kSlices; ++k) (kind ? dout : vout)[wl * kSlices + k] = kind ? __brevll(acc[k]) : acc[k];
    }
  }
  // words past the chunk's diagonal: nothing counted
  const int rest = tbw - W;
  for (int x = tid; x < kSlices * rest; x += 256) vout[W * kSlices + x] = dout[W * kSlices + x] = 0;
}

}  // namespace dam
