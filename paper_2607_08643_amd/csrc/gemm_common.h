// Shared by the two GEMM paths (gemm.hip, gemm_dense.hip): vector types, the
// workspace header, the protected payload and the LDS pipeline primitives.
#pragma once

#include "bsq_internal.h"

namespace bsq {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 128;    // inputs per K step

// The workspace starts with a 256-byte header that the product leaves
// untouched (no block of it waits for another, so there is no poison word
// or flagged slot to keep); the scratch of a call follows: T = X A^T, X~, the
// gathered protected activations and the split-K partials.
constexpr int64_t GEMM_HDR = 256;

// Eight stored protected bytes (two words, byte e of the pair at bits
// 8 (e % 4) of word e / 4) times their scales, in format FMT; the run-time
// format is dispatched once per eight bytes (a uniform branch).
template <int FMT>
__device__ __forceinline__ void payload8_t(uint2 qv, const float *sc, float (&v)[8])
{
    v[0] = payload_byte<FMT, 0>(qv.x) * sc[0];
    v[1] = payload_byte<FMT, 1>(qv.x) * sc[1];
    v[2] = payload_byte<FMT, 2>(qv.x) * sc[2];
    v[3] = payload_byte<FMT, 3>(qv.x) * sc[3];
    v[4] = payload_byte<FMT, 0>(qv.y) * sc[4];
    v[5] = payload_byte<FMT, 1>(qv.y) * sc[5];
    v[6] = payload_byte<FMT, 2>(qv.y) * sc[6];
    v[7] = payload_byte<FMT, 3>(qv.y) * sc[7];
}

__device__ __forceinline__ void payload8(uint2 qv, const float *sc, float (&v)[8], int fmt)
{
    if (fmt == BSQ_PROT_E4M3) payload8_t<BSQ_PROT_E4M3>(qv, sc, v);
    else if (fmt == BSQ_PROT_E5M2) payload8_t<BSQ_PROT_E5M2>(qv, sc, v);
    else payload8_t<BSQ_PROT_INT8>(qv, sc, v);
}

// Workgroup barrier for LDS traffic only: waits for this wave's LDS (and
// scalar) operations, not for its global loads, which stay in flight across
// the barrier (__syncthreads would drain them with its release fence).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0), vmcnt and expcnt unconstrained
    asm volatile("s_barrier" ::: "memory");
}

// Wait until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void wait_vm()
{
    static_assert(N >= 0 && N <= 63, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// LDS of one workgroup (gfx950: 160 KiB per compute unit).
constexpr int GEMM_LDS_BYTES = 160 * 1024;

}  // namespace
}  // namespace bsq
