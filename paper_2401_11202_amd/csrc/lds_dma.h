// Device helpers shared by the kernels that stream tiles into LDS with
// direct-to-LDS buffer loads (GEMMs, attention forward and backward).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace partir {

typedef short lds_i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) lds_i16x4_t lds_i16x4;
typedef __attribute__((address_space(3))) void lds_void;

// Buffer descriptor of a workgroup-uniform base pointer (kept in SGPRs); an
// offset at or beyond `bytes` reads as zero (and writes LDS zeros when the
// load targets LDS).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  void* u = (void*)(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(u, (short)0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// ds_read_b64_tr_b16 through a restrict pointer: the alias scope this gives
// the read keeps the compiler's wait insertion from making it wait for every
// LDS DMA in flight (the callers order their LDS stages by explicit vmcnt
// waits and barriers).
__device__ __forceinline__ lds_i16x4_t lds_read_tr16(const char* __restrict__ p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
}

// An LDS read through a restrict pointer, for the same reason.
template <typename T>
__device__ __forceinline__ T lds_read(const char* __restrict__ p) { return *(const T*)p; }

// LDS tiles of the bf16 GEMMs.
//
// K-contiguous tile: [row][64 k] = 128-byte rows of eight 16-byte chunks;
// chunk c of row r sits at position c ^ gemm_swz(r), gemm_swz(r) = bit1(r) |
// bit3(r) << 1 | bit2(r) << 2.  A fragment read takes 16 rows (lane % 16) at
// 4 chunks (lane / 16); the LDS serves it 8 lanes of each half-wave at a
// time, i.e. 8 rows at two chunks 2 apart, and the swizzle gives the 4 rows of
// each parity distinct bits 0 and 2, so the 16 reads hit 16 different bank
// groups (as do any 16 consecutive lanes: the 8 rows of each parity get all 8
// values).
__device__ __forceinline__ int gemm_swz(int r) {
  return ((r >> 1) & 1) | (((r >> 3) & 1) << 1) | (((r >> 2) & 1) << 2);
}

// MN-major tile of W columns: [k][W] = rows of 2 W bytes; 16-byte chunk c of k
// row r sits at position c ^ gemm_mn_swz<W>(r).  A transposed fragment read
// covers 4 k rows x 16 columns per 16-lane group, groups 0 and 1 (one pass) on
// rows 8 apart, which must fall on different banks: by the row's bits 0, 1 and
// 3, except that with 128-byte rows (W = 64) bit 0 already selects the other
// half of the banks.
template <int W>
__device__ __forceinline__ int gemm_mn_swz(int r) {
  return W > 64 ? ((4 * (r & 3)) ^ (2 * ((r >> 3) & 1))) : ((2 * (r & 2)) ^ (2 * ((r >> 3) & 1)));
}

}  // namespace partir

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding)
#define WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt((((n) & 15) | (((n) >> 4) << 14)) | (0x7 << 4) | (0xF << 8))

// s_waitcnt with only the LDS / scalar-memory counter constrained (gfx9 encoding)
#define WAIT_LGKMCNT(n) __builtin_amdgcn_s_waitcnt((((n) & 15) << 8) | 0xF | (0x3 << 14) | (0x7 << 4))
