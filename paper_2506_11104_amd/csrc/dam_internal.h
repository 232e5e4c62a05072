// Internal helpers shared by the HIP translation units of libdam.so (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "dam.h"

namespace dam {

constexpr int kWave = 64;  // CDNA wavefront width

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Converts the status of the launches enqueued so far into a dam_status.
inline int launch_status() { return hipGetLastError() == hipSuccess ? DAM_OK : DAM_ERR_DEVICE; }

// Carves consecutive 256-byte aligned regions out of one workspace allocation.
struct Carver {
  char *base;
  size_t off = 0;
  explicit Carver(void *p) : base(static_cast<char *>(p)) {}
  template <typename T>
  T *take(size_t n) {
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off = align_up(off + n * sizeof(T), 256);
    return p;
  }
};

// ------------------------------------------------------------------------------------------------
// The last of several workgroups that share an item, without a launch of its own and without anything that has to
// start at zero: every workgroup writes its partial result with stores that go through to memory (store_through),
// then its flag, a 64-bit number drawn anew by the host for every call; the one that then finds the flags of all is
// the last (two that finish together may both be: they then do the same work on the same values), does what is left,
// and clears the flags, so that a replay of the same launch from a HIP graph does not find them set. A memory that was
// never written, or by another call, holds the number with a probability of 2^-64 per flag.
// (An atomic counter would need clearing by a launch, and a release fence writes back the XCD's whole L2: a merge
// kernel of its own costs about 5 us behind a dependent launch, this about 2.)
uint64_t fresh_flag();  // dam_decode.hip; never 0

#ifdef __HIPCC__
// Inclusive prefix sum over the wave, in the vector registers alone (row shifts, then the row totals handed on).
__device__ __forceinline__ int wave_prefix(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // last lane of rows 0 and 2 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // lane 31 to rows 2 and 3
  return v;
}

__device__ __forceinline__ int wave_total(int v) { return __builtin_amdgcn_readlane(wave_prefix(v), 63); }

// 16 bytes to memory past this XCD's L2, for readers on other XCDs; not complete before stores_done()
__device__ __forceinline__ void store_through(void *p, float x, float y, float z, float w) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  const f32x4_t v = {x, y, z, w};
  asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through(float *p, float x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// What store_through stored on another XCD, once its workgroup's flag has been seen.
__device__ __forceinline__ float2 load_through(const float2 *p) {
  return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// To be called by one whole wave after the stores of its workgroup are done; n <= 64 flags, this workgroup's is `self`.
// True in the last workgroup, which may then read what the others stored, with load_through. (An acquire fence and ordinary
// loads instead drop what this XCD's L2 holds, also the K and V rows that other lists' workgroups are about to share: a list
// per head, 32 fp32 heads of 8 KV heads, 3000 keys, 4 sequences 27.0 us instead of 25.1.)
__device__ __forceinline__ bool arrive_last(uint64_t *flags, int n, int self, uint64_t flag) {
  const int lane = threadIdx.x & 63;
  if (lane == 0) __hip_atomic_store(&flags[self], flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  stores_done();
  const uint64_t seen = lane < n ? __hip_atomic_load(&flags[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : flag;
  if (__ballot(seen != flag) != 0) return false;
  if (lane < n) __hip_atomic_store(&flags[lane], (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}
#endif

// dam_capture.hip: argument check of a capture, bytes of its row log-sum-exp buffer, and the fused
// form that writes the true mask of one captured sequence (bit = probability >= threshold, the
// threshold given as the ordered fp32 key the mask builder uses). vslices != nullptr: the patterns' chunk counts are wanted
// too (dam_slices.h); says whether they were written.
int capture_validate(const dam_capture_params *p, const void *q, const void *k);
size_t capture_lse_bytes(const dam_capture_params *p);
bool launch_capture_true_bits(const dam_capture_params *p, const void *q, const void *k, float *lse2,
                              unsigned theta_key, float bmin, float *out_bmin, uint64_t *true_bits, uint64_t *vslices,
                              uint64_t *dslices, hipStream_t stream);

// dam_decode_mfma.hip: the partial pass of the grouped-query decode on the matrix cores. `fits` says
// whether a call can take it (bf16, head_dim 128, at most 8 query heads per KV head, a head's cache rows
// within 4 GiB). A list is shared by `waves` waves of each of `groups` workgroups; with more than one group the partial
// results go through part_o [pair][group][128 G], part_ml [pair][group][G][2] and flags [pair][group].
// plan_table != nullptr: the lists are a position-independent plan (DAM_MASK_PATTERN_PLAN) decoded at position pos;
// n_flags is the table's row length.
struct GroupSplit {
  int waves, groups;
};
bool decode_group_mfma_fits(const dam_decode_params *p);
int launch_decode_group_mfma(const dam_decode_params *p, GroupSplit split, float scale, const void *q, const void *kc,
                             const void *vc, const int32_t *kept_ptr, const int32_t *kept_idx,
                             const uint8_t *kept_member, float *part_o, float *part_ml, uint64_t *flags, void *out,
                             float *lse, hipStream_t st, const uint8_t *plan_table = nullptr, int n_flags = 0, int pos = 0);

}  // namespace dam
