// What the kernels on the matrix cores share: the event types as the matrix instructions take them, and
// small pieces of wave-level work.
#pragma once

#include <hip/hip_runtime.h>

#include "idf.h"

namespace idf {

// every lambda of these kernels works on the accumulators or the arguments: called instead of inlined, those would live in memory
#define IDF_INLINE __attribute__((always_inline))

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;

// An activation or none in one instruction: the median of a sum and two bounds -- zero and infinity, or NaN both, which stand aside; a
// NaN sum stays NaN without an activation and is zero with one.  By fmaxf and a choice it is three instructions, one of them for
// signalling NaNs (us per image, vgg-style net 2563 -> 2527, float32 net under eager emission 1131 -> 1108; not in the gathering
// kernel, whose tiles end in few of them: 64 audio streams 5556 -> 5636).  An instruction that the compiler knows, and not inline
// assembly, which took the same time (2420 : 2423, 1027 : 1022): it reads what matrix instructions have written, and the compiler keeps
// the distance that such a read needs for its own instructions only.  The upper bound is in a vector register, since an instruction
// takes one scalar, and hidden, since of bounds that it knows the compiler makes the three instructions again.
struct FloatBounds {
    float lo, hi;
    __device__ __forceinline__ explicit FloatBounds(bool none) : lo(none ? __builtin_nanf("") : 0.f), hi(none ? __builtin_nanf("") : __builtin_inff()) { asm("" : "+v"(hi)); }
    __device__ __forceinline__ float operator()(float c) const { return __builtin_amdgcn_fmed3f(c, lo, hi); }
};
// v between two bounds that are in order: the form of the median that the compiler knows as one instruction.
__device__ __forceinline__ int32_t between(int32_t v, int32_t lo, int32_t hi) { return max(min(v, lo), min(max(v, lo), hi)); }
// Per event type: VL elements per 16-byte cell, EB bytes per element, kInst matrix instructions of
// 16 x 16 per K-step of four cells, pack4: four activated sums as EB words of events.
struct TraitsBf16 {
    static constexpr bool kEvents = false;
    static constexpr int VL = 8, EB = 2, kInst = 1;
    using acc_t = f32x4; using st_t = float; using ev_t = uint16_t;
    static __device__ __forceinline__ acc_t mfma(const i32x4 &w, const i32x4 &x, const acc_t &c, int)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
    }
    static __device__ __forceinline__ int or_of(const i32x4 &v) { return (v.x | v.y | v.z | v.w) & 0x7fff7fff; }      // zero is +0 or -0
    static __device__ __forceinline__ int nonzero(uint32_t w)
    {   // adding 0x7fff to the 15 magnitude bits of a half carries into its top bit unless they are all zero
        return __builtin_popcount(((w & 0x7fff7fffu) + 0x7fff7fffu) & 0x80008000u);
    }
    static __device__ __forceinline__ st_t activate(st_t c, int act, int, int) { return act == IDF_ACT_NONE ? c : fmaxf(c, 0.f); }
    static __device__ __forceinline__ void pack4(const st_t *v, uint32_t *out)
    {   // round to nearest, ties to even (the conversion instruction)
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            bf16x2 p;
            p.x = (__bf16)v[2 * i]; p.y = (__bf16)v[2 * i + 1];
            out[i] = __builtin_bit_cast(uint32_t, p);
        }
    }
    static __device__ __forceinline__ bool ev_nonzero(ev_t v) { return (v & 0x7fffu) != 0; }
};

struct TraitsI8 {
    static constexpr bool kEvents = true;    // sparse stretches can take the event-list path on the vector units
    static constexpr int VL = 16, EB = 1, kInst = 1;
    using acc_t = i32x4; using st_t = int32_t; using ev_t = int8_t;
    static __device__ __forceinline__ acc_t mfma(const i32x4 &w, const i32x4 &x, const acc_t &c, int)
    {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(w, x, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int or_of(const i32x4 &v) { return v.x | v.y | v.z | v.w; }
    static __device__ __forceinline__ int nonzero(uint32_t u)
    {   // per byte: the low seven bits carry into the top bit, or the top bit is set already
        return __builtin_popcount((((u & 0x7f7f7f7fu) + 0x7f7f7f7fu) | u) & 0x80808080u);
    }
    static __device__ __forceinline__ st_t activate(st_t c, int act, int shr, int hi)
    {
        if (act == IDF_ACT_NONE) return c;
        st_t r = c > 0 ? c : 0;
        if (act == IDF_ACT_RELU_SHR_CLAMP) { r >>= shr; r = r > hi ? hi : r; }
        return r;
    }
    static __device__ __forceinline__ void pack4(const st_t *v, uint32_t *out)
    {
        out[0] = __builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x0c0c0400u) | __builtin_amdgcn_perm((uint32_t)v[3], (uint32_t)v[2], 0x04000c0cu);
    }
    static __device__ __forceinline__ bool ev_nonzero(ev_t v) { return v != 0; }
};

// float32: a cell holds four k, served by four 16x16x4 instructions (instruction i takes element i of
// every lane's cell; which four k share an instruction does not matter to the sum).
struct TraitsF32 {
    static constexpr bool kEvents = false;
    static constexpr int VL = 4, EB = 4, kInst = 4;
    using acc_t = f32x4; using st_t = float; using ev_t = float;
    static __device__ __forceinline__ acc_t mfma(const i32x4 &w, const i32x4 &x, const acc_t &c, int i)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(w[i]), __int_as_float(x[i]), c, 0, 0, 0);
    }
    static __device__ __forceinline__ int or_of(const i32x4 &v) { return (v.x | v.y | v.z | v.w) & 0x7fffffff; }      // zero is +0 or -0
    static __device__ __forceinline__ int nonzero(uint32_t w) { return (w & 0x7fffffffu) != 0; }
    static __device__ __forceinline__ st_t activate(st_t c, int act, int, int) { return act == IDF_ACT_NONE ? c : fmaxf(c, 0.f); }
    static __device__ __forceinline__ void pack4(const st_t *v, uint32_t *out)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = __float_as_uint(v[i]);
    }
    static __device__ __forceinline__ bool ev_nonzero(ev_t v) { return v != 0.f; }
};

// A value at a byte offset from a base every lane shares: "scalar base + lane offset", no 64-bit
// arithmetic per lane.
template <class P> __device__ __forceinline__ P *at4(P *base, uint32_t byte_off)
{
    return (P *)((const char *)base + byte_off);
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Sum over the wave's lanes, in every lane: shifts and broadcasts inside the vector units, no LDS.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);       // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);       // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);       // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);       // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);      // lane 15 of a row to the next row
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);      // lane 31 to the upper half
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The value of the neighbouring lane (lane ^ 1).
template <class V> __device__ __forceinline__ V neighbour(V v)
{
    return __builtin_bit_cast(V, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));
}

// Arguments of a launch on their way to the scalar cache, a few of their 64-byte lines by each wave of the workgroup: met one
// after the other, each line would be a trip to memory of its own.  also: a further place whose line is wanted.  (One statement: the
// compiler puts a wait behind each load whose value it believes to be used.)
template <int BYTES, int WAVES> __device__ __forceinline__ void request_arguments(const void __attribute__((address_space(4))) *args, const void __attribute__((address_space(4))) *also)
{
    typedef const __attribute__((address_space(4))) char Byte;
    constexpr int N = (BYTES / 64 + WAVES - 1) / WAVES, PITCH = WAVES * 64;
    static_assert(N >= 1 && N <= 12, "as many loads as stand below");
    const int first = uni(threadIdx.x >> 6) * 64, last = first + (N - 1) * PITCH;
    int sink;
    asm volatile("s_load_dword %0, %1, 0x0\n\t"
                 "s_load_dword %0, %2, 0x0\n\t"
                 "s_load_dword %0, %3, 0x0\n\t"
                 ".if %c4 > 2\n\ts_load_dword %0, %3, 1*%c5\n\t.endif\n\t"
                 ".if %c4 > 3\n\ts_load_dword %0, %3, 2*%c5\n\t.endif\n\t"
                 ".if %c4 > 4\n\ts_load_dword %0, %3, 3*%c5\n\t.endif\n\t"
                 ".if %c4 > 5\n\ts_load_dword %0, %3, 4*%c5\n\t.endif\n\t"
                 ".if %c4 > 6\n\ts_load_dword %0, %3, 5*%c5\n\t.endif\n\t"
                 ".if %c4 > 7\n\ts_load_dword %0, %3, 6*%c5\n\t.endif\n\t"
                 ".if %c4 > 8\n\ts_load_dword %0, %3, 7*%c5\n\t.endif\n\t"
                 ".if %c4 > 9\n\ts_load_dword %0, %3, 8*%c5\n\t.endif\n\t"
                 ".if %c4 > 10\n\ts_load_dword %0, %3, 9*%c5\n\t.endif\n\t"
                 ".if %c4 > 11\n\ts_load_dword %0, %3, 10*%c5\n\t.endif\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(sink)
                 : "s"(also), "s"((Byte *)args + (last < BYTES ? last : 0)), "s"((Byte *)args + (first < BYTES ? first : 0)), "n"(N), "n"(PITCH));
}

__device__ __forceinline__ int taps_of(int v, int n) { return 3 - (v == 0) - (v == n - 1); }      // of a 3-tap axis with one position of padding

// 16-byte cells from one position to the next in LDS.  The lanes of a fragment read 16 positions x 4 consecutive
// cells; one cycle serves eight positions of one cell and the other eight of the next, so that an even distance that
// is no multiple of four keeps all sixteen on banks of their own (measured: 222 bytes per clock and CU at 10 cells,
// 123 at 9, 63 at 8).
__host__ __device__ inline int cell_stride(int cells) { return cells == 1 ? 1 : (cells + 1) / 4 * 4 + 2; }

// Cells of a window of 3 * c_in values, for layers of a few channels.  A K-step takes four cells: behind the window the weights are
// zero, but zero times infinity is not, so that float nets keep zeros there.
__host__ __device__ constexpr int window_cells(int c_in, int vl, bool is_float) { return is_float ? 4 : (3 * c_in + vl - 1) / vl; }

}  // namespace

}  // namespace idf
