// device_common.h -- device helpers shared by the GEMM kernels of the conv2d library.
#pragma once

#include "conv2d_internal.h"

namespace cv {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define OOB_OFF 0x80000000u
#define RSRC_WORD3 0x00020000

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, RSRC_WORD3);
}

__device__ __forceinline__ float ld_f32(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ uint16_t ld_u16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}
__device__ __forceinline__ void st_f32(__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
}
__device__ __forceinline__ void st_u16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint16_t v) {
    __builtin_amdgcn_raw_buffer_store_b16(v, r, off, 0, 0);
}

// fp32 -> bf16 bits, round to nearest even (inputs are finite).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <typename TOut>
__device__ __forceinline__ void store_out(__amdgpu_buffer_rsrc_t r, uint32_t elem_off_valid, bool ok,
                                          float v);
template <>
__device__ __forceinline__ void store_out<float>(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float v) {
    st_f32(r, ok ? e * 4u : OOB_OFF, v);
}
template <>
__device__ __forceinline__ void store_out<uint16_t>(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok,
                                                    float v) {
    st_u16(r, ok ? e * 2u : OOB_OFF, f32_to_bf16_rne(v));
}

// Four consecutive output elements starting at element e (e a multiple of 4): one 16-byte
// (fp32) or 8-byte (bf16, round to nearest even) store.
template <typename TOut>
__device__ __forceinline__ void store_out4(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float a, float b, float c,
                                           float d);
template <>
__device__ __forceinline__ void store_out4<float>(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float a, float b,
                                                  float c, float d) {
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                 __builtin_bit_cast(uint32_t, c), __builtin_bit_cast(uint32_t, d)},
                                           r, ok ? e * 4u : OOB_OFF, 0, 0);
}
template <>
__device__ __forceinline__ void store_out4<uint16_t>(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float a, float b,
                                                     float c, float d) {
    __builtin_amdgcn_raw_buffer_store_b64(
        u32x2{(uint32_t)f32_to_bf16_rne(a) | ((uint32_t)f32_to_bf16_rne(b) << 16),
              (uint32_t)f32_to_bf16_rne(c) | ((uint32_t)f32_to_bf16_rne(d) << 16)},
        r, ok ? e * 2u : OOB_OFF, 0, 0);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two consecutive output elements starting at element e (e even): one 8-byte (fp32) or
// 4-byte (bf16: the hardware's packed conversion, round to nearest even) store.
template <typename TOut>
__device__ __forceinline__ void store_out2(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float lo, float hi);
template <>
__device__ __forceinline__ void store_out2<float>(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float lo, float hi) {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)}, r,
                                          ok ? e * 4u : OOB_OFF, 0, 0);
}
template <>
__device__ __forceinline__ void store_out2<uint16_t>(__amdgpu_buffer_rsrc_t r, uint32_t e, bool ok, float lo,
                                                     float hi) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2)),
                                          r, ok ? e * 2u : OOB_OFF, 0, 0);
}

// The value of lane l ^ 1 (a DPP quad permutation, no LDS).
__device__ __forceinline__ float swap_adjacent_lanes(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));
}

// n / d for 0 <= n < 2^31 with the divisor's multiplier and shift (FastDiv).
__device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv f) { return (__umulhi(n, f.m) + n) >> f.s; }

// Linear block id -> tile id such that consecutive tile ids land on the same
// XCD (workgroups are handed to the 8 XCDs round-robin), so the M tiles of one
// pixel tile and neighbouring pixel tiles share an L2.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    const int per = nb >> 3, rem = nb & 7;
    const int xcd = bid & 7, slot = bid >> 3;
    return xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
}

// Tail split: store this piece's partial tile, count its arrival, and in the piece that
// arrives last replace acc by the sum of all pieces of the tile in piece order (the same
// result whatever the arrival order).  Returns false in the other pieces, which are done.
// The pieces of a tile may run on different XCDs, whose L2 caches are not coherent with
// each other.  The partials are therefore stored and loaded with the device-scope cache
// policy (sc1: written through to, and read from, the point where all XCDs agree), and each
// piece waits for its stores to complete before it counts itself; no fence is used, since
// a device-scope fence writes back and invalidates the whole L2 of the XCD and costs every
// other block on it its cached input.  The counter is an atomic, coherent device-wide.
// Partial layout: 16-byte unit ((i*TN + j)*4 + q)*NT + t (NT threads) of the piece's BM x BN tile, through
// buffer operations with a wave-uniform base (no per-lane address kept alive).
template <int TM, int TN, int NT>
__device__ __forceinline__ bool tail_reduce(float* tail_part, uint32_t* tail_count, int tail_tiles, int tail_pieces,
                                            f32x16 (&acc)[TM][TN], int tail_tile, int piece, int t) {
    constexpr uint32_t PIECE = TM * TN * 4 * NT * 16;  // bytes of one partial tile
    constexpr int SC1 = 1 << 4;                         // buffer cache policy bit: device scope
    __shared__ int s_last;
    const __amdgpu_buffer_rsrc_t rp =
        make_rsrc(tail_part, (uint32_t)tail_tiles * (uint32_t)tail_pieces * PIECE);
    const uint32_t tile_base = (uint32_t)tail_tile * (uint32_t)tail_pieces * PIECE;
    const uint32_t lane_off = (uint32_t)t * 16u;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(
                    __builtin_bit_cast(u32x4, v), rp, lane_off,
                    (int)(tile_base + (uint32_t)piece * PIECE + (uint32_t)((i * TN + j) * 4 + q) * (NT * 16u)), SC1);
            }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partial is complete device-wide
    __syncthreads();
    if (t == 0)
        s_last = __hip_atomic_fetch_add(tail_count + tail_tile, 1u, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(tail_pieces - 1);
    __syncthreads();
    if (!s_last) return false;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
#pragma unroll 1
    for (int pc = 0; pc < tail_pieces; ++pc) {
        const uint32_t base = tile_base + (uint32_t)pc * PIECE;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = __builtin_bit_cast(
                        f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                   rp, lane_off, (int)(base + (uint32_t)((i * TN + j) * 4 + q) * (NT * 16u)), SC1));
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
                }
    }
    // ready for the next launch
    if (t == 0) __hip_atomic_store(tail_count + tail_tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Per-column state of the implicit gather: window origin and base offset.
struct ColState {
    int64_t base;  // element offset of x[n, gi*Cg, hi0, wi0] (may be "negative" in padding)
    int32_t hi0, wi0;
};

__device__ __forceinline__ ColState col_state(const GemmArgs& A, int p, int gi) {
    ColState s;
    if (p < A.P) {
        const int n = p / A.HoWo;
        const int hw = p - n * A.HoWo;
        const int ho = hw / A.Wo;
        const int wo = hw - ho * A.Wo;
        s.hi0 = ho * A.sh - A.ph;
        s.wi0 = wo * A.sw - A.pw;
        s.base = (int64_t)n * A.x_nstride + (int64_t)gi * A.b_gstride + (int64_t)s.hi0 * A.W + s.wi0;
    } else {
        s.hi0 = KTAB_DEAD;
        s.wi0 = 0;
        s.base = 0;
    }
    return s;
}

// Byte offset of B[kr][col] for the implicit gather (or OOB_OFF for a zero tap).
template <int ESIZE>
__device__ __forceinline__ uint32_t implicit_off(const GemmArgs& A, const ColState& cs, const KTabEntry& e) {
    const int hi = cs.hi0 + e.roff;
    const int wi = cs.wi0 + e.soff;
    const bool ok = ((unsigned)hi < (unsigned)A.H) & ((unsigned)wi < (unsigned)A.W);
    return ok ? (uint32_t)((cs.base + e.coff) * ESIZE) : OOB_OFF;
}

// Scalar (wave-uniform) read of one table entry.
__device__ __forceinline__ KTabEntry ktab_at(const KTabEntry* t, int kr) {
    kr = __builtin_amdgcn_readfirstlane(kr);
    return t[kr];
}

}  // namespace cv
