// The slab layout of split (hi/lo) 16-bit operands and the waits of the
// kernels that stream it through LDS, shared by gemm_bf16x3.hip and
// gemm_f16x3.hip.
//
// Slab layout.  Every split operand (rows x K) is stored as K/16 slabs; slab
// q holds k = 16q..16q+15 of all rows, 32 bytes per row, row after row, and
// the two 16-byte halves of row r are swapped when bit 3 of r is set.  The
// 16-wide K slice of a tile is then one contiguous block per array, copied
// verbatim into LDS by buffer loads with LDS destination (1 KB per wave
// instruction, whole cache lines), and the swap spreads the 128-bit fragment
// reads of 16 lanes (rows c..c+15, one k half) over all 64 LDS banks.  The
// last slab of an operand whose K is not a multiple of 16 is zero beyond K.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "buffer_rsrc.h"

namespace rot {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSlabK = 16;  // k per slab

inline __host__ __device__ int64_t n_slabs(int64_t K) { return (K + kSlabK - 1) / kSlabK; }

// Element (r, k) of a slab-layout operand with `rows` rows.
inline __host__ __device__ int64_t slab_off(int64_t r, int64_t k, int64_t rows) {
    return (k >> 4) * rows * kSlabK + r * kSlabK + ((((k >> 3) & 1) ^ ((r >> 3) & 1)) << 3) + (k & 7);
}

// Buffer descriptor over one slab-layout operand (raw addressing; loads past
// its last slab return zero).
__device__ inline __amdgpu_buffer_rsrc_t operand_rsrc(const uint16_t* p, int rows, int K) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p), (short)0,
                                             (int)(n_slabs(K) * rows * kSlabK * 2), kBufferFlags);
}

// s_waitcnt immediate that waits until at most n vector-memory operations
// of this wave are outstanding (other counters unconstrained).
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x70 | 0xF00; }
// s_waitcnt immediate that waits for every LDS access of this wave.
constexpr int kLgkmcnt0 = 0xF | (3 << 14) | 0x70;

// Ordering point for the compiler only: memory accesses are not moved across
// it (s_barrier alone does not order them for the optimiser).
__device__ inline void compiler_fence() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

inline size_t al256(size_t n) { return (n + 255) / 256 * 256; }

}  // namespace
}  // namespace rot
