// fa_common.h -- device-side helpers shared by the gfx950 attention kernels.
//
// Lane layouts of the matrix instructions used here (checked on gfx950):
//   v_mfma_f32_32x32x16_{f16,bf16}: A lane l holds A[l%32][8*(l/32)+e],
//     B lane l holds B[8*(l/32)+e][l%32] (e = 0..7), C lane l register r holds
//     C[8*(r/4) + 4*(l/32) + r%4][l%32] (r = 0..15).
//   v_mfma_f32_16x16x32_{f16,bf16}: A lane l holds A[l%16][8*(l/16)+e],
//     B lane l holds B[8*(l/16)+e][l%16], C lane l register r holds
//     C[4*(l/16)+r][l%16] (r = 0..3).
//   ds_read_b64_tr_b16: within each group of 16 lanes, result element e of
//     lane j is element j%4 of the 8 bytes addressed by lane 4*e + j/4.  So if
//     lane i of the group addresses row (r0 + i/4), columns c0 + 4*(i%4)..+3 of
//     a row-major 16-bit matrix, lane j receives column c0 + j of rows r0..r0+3.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fa {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uint4_t __attribute__((ext_vector_type(4)));

// Storage types as seen by the kernels.
struct f16_t {
    typedef _Float16 scalar;
    typedef half8_t vec8;
};
struct bf16_t {
    typedef __bf16 scalar;
    typedef bf16x8_t vec8;
};

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// fp32 -> output element, round to nearest even.
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ _Float16 from_f32<_Float16>(float x) { return (_Float16)x; }
template <> __device__ __forceinline__ __bf16 from_f32<__bf16>(float x) { return (__bf16)x; }

// Matrix instruction wrappers, one per input element type.
__device__ __forceinline__ float16_t mfma32(half8_t a, half8_t b, float16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float16_t mfma32(bf16x8_t a, bf16x8_t b, float16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float4_t mfma16(half8_t a, half8_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float4_t mfma16(bf16x8_t a, bf16x8_t b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Eight 16-bit values as one 16-byte word.
template <typename V> __device__ __forceinline__ V as_vec8(uint4_t u) {
    return __builtin_bit_cast(V, u);
}

// bf16 x8 (as raw 16-byte word) -> f16 x8 (raw), round to nearest even.
__device__ __forceinline__ uint4_t bf16x8_to_f16x8(uint4_t u) {
    half8_t h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[2 * i] = (_Float16)__uint_as_float(u[i] << 16);
        h[2 * i + 1] = (_Float16)__uint_as_float(u[i] & 0xffff0000u);
    }
    return __builtin_bit_cast(uint4_t, h);
}

// Pack 8 fp32 values to f16 x8, round to nearest even.
__device__ __forceinline__ half8_t pack_f16x8(float a0, float a1, float a2, float a3, float a4,
                                              float a5, float a6, float a7) {
    half8_t h;
    h[0] = (_Float16)a0; h[1] = (_Float16)a1; h[2] = (_Float16)a2; h[3] = (_Float16)a3;
    h[4] = (_Float16)a4; h[5] = (_Float16)a5; h[6] = (_Float16)a6; h[7] = (_Float16)a7;
    return h;
}

// Reductions over the lane pair (l, l^32).  v_permlane32_swap exchanges the
// upper half of its first operand with the lower half of its second; with the
// same value in both, the two results of every lane are the pair's two values
// (one from each half), whichever result holds which.
__device__ __forceinline__ float pair_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                              false);
    return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                              false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same over the lane pair (l, l ^ 16).
__device__ __forceinline__ float half_max(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float max3(float a, float b, float c) {
    return __builtin_fmaxf(a, __builtin_fmaxf(b, c));
}

// LDS transpose read (see the layout note at the top of this file).
__device__ __forceinline__ short4_t lds_read_tr16(const _Float16 *p) {
    typedef __attribute__((address_space(3))) short4_t lds_s4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(p));
}

__device__ __forceinline__ half8_t cat_half8(short4_t lo, short4_t hi) {
    typedef short short8_t __attribute__((ext_vector_type(8)));
    short8_t s = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(half8_t, s);
}

// Address of an LDS object.
__device__ __forceinline__ unsigned lds_address(void *p) {
    typedef __attribute__((address_space(3))) char lds_char;
    return (unsigned)(unsigned long long)(lds_char *)p;
}

// 16 bytes per lane from a buffer view (its base address and size in bytes)
// straight into LDS: lane l's bytes land at LDS address dst + 16 l (dst the same
// for the wave); lanes past the end of the view write zeros (checked on gfx950).  In
// assembly, with no result register, because the compiler makes every later
// LDS read wait for such loads; nothing waits for them but lds_loads_done(),
// which goes before the barrier that publishes the data.  base, bytes and dst
// are wave-uniform; dst is an operand in m0, so that the compiler knows what m0
// holds; the s_nop covers a scalar register that a vector instruction wrote
// just before (five wait states to its use in an address).
__device__ __forceinline__ void load_lds16(const void *base, int bytes, unsigned dst, int off) {
    const unsigned long long p = (unsigned long long)base;   // below 2^48: the descriptor's stride bits stay 0
    const uint4_t rsrc = {(unsigned)p, (unsigned)(p >> 32), (unsigned)bytes, 0x00020000u};
    asm volatile("s_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(dst), "v"(off), "s"(rsrc) : "memory");
}
template <int N> __device__ __forceinline__ void lds_loads_done() {   // all but the last N loads of the wave
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Workgroup barrier for LDS alone: the wave's own LDS accesses are done, its
// loads from memory stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Global 16-byte load / store helpers.
__device__ __forceinline__ uint4_t ld16(const void *p) {
    return *reinterpret_cast<const uint4_t *>(p);
}
__device__ __forceinline__ void st16(void *p, uint4_t v) { *reinterpret_cast<uint4_t *>(p) = v; }

// Division of n < 2^31 by a launch constant d >= 1 in three scalar
// instructions (an integer division takes some twenty vector ones, which
// delay a kernel's first loads): with 2^(s-1) < d <= 2^s and m =
// ceil(2^(31+s) / d), floor(n / d) = floor(n m / 2^(31+s)), since n (m d -
// 2^(31+s)) < 2^31 d <= 2^(31+s).
struct Divisor {
    unsigned d, m, shift;
    explicit Divisor(unsigned div = 1) : d(div) {
        unsigned s = 0;
        while ((1ull << s) < d) ++s;
        shift = 31 + s;
        m = (unsigned)(((1ull << shift) + d - 1) / d);
    }
    __device__ __forceinline__ unsigned div(unsigned n) const { return (unsigned)(((unsigned long long)n * m) >> shift); }
};

// Sequences by length, at most kMaxRanked of them, one per lane.  uneven: some
// sequence is shorter than 7/8 of the longest.  nth_longest: the batch element
// with the r-th largest length (0: the longest; equal ones in order); each lane
// ranks one element against the others.
constexpr int kMaxRanked = 64;
struct Lengths {
    int len, B, lane;
    __device__ __forceinline__ Lengths(const int *seqlens, int b, int l) : B(b), lane(l) {
        len = seqlens[min(l, b - 1)];
    }
    __device__ __forceinline__ bool uneven() const {
        const int n = max(len, 0);
        int mx = n;   // over the wave: lanes ^ 1, ^ 2, the other half of 8, of 16, lanes ^ 16, ^ 32
        mx = max(mx, __builtin_amdgcn_mov_dpp(mx, 0xb1, 0xf, 0xf, true));
        mx = max(mx, __builtin_amdgcn_mov_dpp(mx, 0x4e, 0xf, 0xf, true));
        mx = max(mx, __builtin_amdgcn_mov_dpp(mx, 0x141, 0xf, 0xf, true));
        mx = max(mx, __builtin_amdgcn_mov_dpp(mx, 0x140, 0xf, 0xf, true));
        auto r = __builtin_amdgcn_permlane16_swap(mx, mx, false, false);
        mx = max((int)r[0], (int)r[1]);
        auto q = __builtin_amdgcn_permlane32_swap(mx, mx, false, false);
        mx = max((int)q[0], (int)q[1]);
        return __builtin_amdgcn_ballot_w64(n < mx - (mx >> 3)) != 0;
    }
    __device__ __forceinline__ int nth_longest(int r) const {
        const unsigned key = (unsigned)min(max(len, 0), 0x3ffffff) << 6 | (63 - lane);   // all different
        int rank = 0;
#pragma unroll 4
        for (int i = 0; i < B; ++i) rank += (unsigned)__builtin_amdgcn_readlane(key, i) > key;
        return __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < B && rank == r));
    }
    __device__ __forceinline__ int of(int b) const { return __builtin_amdgcn_readlane(len, b); }
};

}  // namespace fa
