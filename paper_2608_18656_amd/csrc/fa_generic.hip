// fa_generic.hip -- attention forward with fp32 weights, for the cases the
// half-precision matrix kernels do not take: fp32 inputs, fp16 / bf16 with
// a head dimension other than 64 or 128 (any D with D % 8 == 0 and D <= 256),
// and key rows too long for those kernels' offsets (tile_fits), prefill and decode.
//
// Scores are fp32 sums; weights, their sums and the accumulators are fp32.
// Both products run on the matrix cores:
//   S^T = K Q^T   fp32 inputs: 16x16x4 fp32 MFMA (the rows of K taken in the
//                 order 4 (i % 4) + i / 4); fp16 / bf16: 16x16x32 MFMA of the
//                 inputs as they are (exact products, fp32 sums)
//   O^T += V^T P^T, P straight from the score registers.  fp32 inputs: 16x16x4
//                 fp32 MFMA.  fp16 / bf16: the inputs' 16x16x32 MFMA with each
//                 fp32 weight as the sum of three 16-bit terms, which holds all
//                 its 24 bits; products are exact, sums fp32.  Three of those
//                 take 48 cycles for 32 keys, eight fp32 ones 256.  (fp16 terms
//                 hold a weight in full down to 2^-23 of the largest: 32 keys
//                 with a smaller one are multiplied in fp32.)  V^T operands
//                 by the transposing LDS read.
//
// Work split.  The Nq * G query rows of the G heads that read one key/value
// head are numbered together, v = row * G + head, and 16 consecutive ones are
// the columns of a wave's matrix products, so a group's heads share every
// staged key and a decode call (Nq = 1) fills columns with heads.  A workgroup
// is NSLOT slots of 16 columns times KSP key parts: a tile of KSP * 16 NB keys
// is staged in LDS for all of them, memory to LDS directly (two stages, the
// next tile's loads are in flight during a step), and part j takes its keys
// 16 NB j ...  The parts' states are merged through LDS at the end.
//
// What bounds it.  fp32: the fp32 MFMA (64 flop per cycle and SIMD; a wave's
// 16 x 16 block takes D / 4 score and D / 4 value steps of 32 cycles) with the
// softmax's vector instructions on top, about 25 to 40 for four scores a lane;
// with four waves a SIMD, 2900 cycles a step at D = 64 of which 2048 are MFMA.
// 16 bits: instruction issue, about 150 vector instructions and 4 DP / 16 MFMA
// of 16 cycles a wave's step of 32 keys, and the staging, some 50 bytes per
// clock and CU; a step of one workgroup alone on its CU takes 1800 cycles at
// D = 96 (the loads' issue 600, scores 350, softmax 500, values 490).  The base
// of the weights moves rarely (see GROWTH): a rescale in nearly every step, as
// 16 columns' maxima grow in turn, cost 50 more instructions.
// Timed in turn, before (all fp32 MFMA, copies through registers with the
// 16-bit values widened, a rescale whenever a maximum grows) and now, in us:
// causal bf16 16/2 heads, 1111 rows, D = 96 39 -> 21; D = 256 205 -> 40;
// causal bf16 4 x 32/8, 2048 rows, D = 96 639 -> 222; decode bf16 16 x 32/8 x
// 2048, D = 96 50 -> 25; causal fp32 16 heads, 777 rows, D = 64 27.5 -> 24.2,
// D = 256 227 -> 78; fp32 2 heads, 128 rows, D = 64 7.7 -> 6.1.
#include <type_traits>

#include "fa_common.h"
#include "fa_internal.h"

namespace fa {
namespace {

constexpr int QB = 16;    // query columns per wave
constexpr int CUS = 256;  // compute units of the card

struct GenericArgs {
    const void *q, *k, *v;
    void *o;
    float *lse;
    int B, Hq, Hkv, Nq, Nk, D;
    int causal;
    float c;          // |scale| * log2(e), > 0
    unsigned qsign;   // sign bits of an element word, to negate q (scale < 0), else 0
    int nvb;   // blocks of 16 NSLOT columns per key/value head
    Divisor per_vb, nkv, group;   // B * Hkv, Hkv, Hq / Hkv
    const int *seqlens;   // valid keys per batch element (NULL: Nk for all)
    const int *block_table;   // paged K/V: page of each key block (see Problem)
    Divisor page_size;
    int max_pages, num_pages;
};

__device__ __forceinline__ float4_t mfma4(float a, float b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Maxima that keep NaN, which the compiler forms without quieting its operands
// first (with fmaxf, an instruction more for every score).  Not in assembly:
// the compiler adds no wait states for what an assembly block reads, and these
// read results of matrix instructions.
__device__ __forceinline__ float max_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float max3_nan(float a, float b, float c) { return max_nan(max_nan(a, b), c); }
__device__ __forceinline__ float min_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }
// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float quad_max(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = max_nan(__uint_as_float(r[0]), __uint_as_float(r[1]));
    auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return max_nan(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
// Element types as the kernel uses them: the storage scalar, and for fp16 /
// bf16 the operand type of the matrix products.
template <typename T> struct Elem;
template <> struct Elem<float> { typedef float scalar; };
template <> struct Elem<f16_t> { typedef _Float16 scalar; };
template <> struct Elem<bf16_t> { typedef __bf16 scalar; };

// Two fp32 weights as three 16-bit terms each (t[0] + t[1] + t[2]).
// bf16: the leading 8 bits are cut off three times: 24 bits, exact (the
// remainder after a cut by a two-element dot product, p - 1 h_0 - 0 h_1 or
// p - 0 h_0 - 1 h_1, which needs no shift; exact, checked on gfx950).
__device__ __forceinline__ void split3(float p0, float p1, unsigned t[3], bf16_t) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    unsigned lo = 0x0000bf80u, hi = 0xbf800000u;   // (-1, 0) and (0, -1)
    asm("" : "+s"(lo), "+s"(hi));   // in registers: as an inline operand -1.0 is not this pair
    auto top = [](float a, float b) { return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u); };
    auto rest = [](unsigned h, unsigned one, float x) {
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, h), __builtin_bit_cast(bf16x2_t, one), x, false);
    };
    t[0] = top(p0, p1);
    const float m0 = rest(t[0], lo, p0), m1 = rest(t[0], hi, p1);
    t[1] = top(m0, m1);
    t[2] = top(rest(t[1], lo, m0), rest(t[1], hi, m1));
}
// fp16 (weights up to 2^15): 11 bits at a time; t[1] and t[2] are kLowScale times
// their terms, so that the last place is 2^-35 and a weight of kLeast or more
// keeps all its bits.
constexpr float kLowScale = 2048.f, kLeast = 0x1p-12f;
__device__ __forceinline__ void split3(float p0, float p1, unsigned t[3], f16_t) {
    auto cut = [](float a, float b) { return __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(a, b)); };
    const half2_t h = cut(p0, p1);
    const float m0 = __builtin_fmaf((float)h[0], -kLowScale, kLowScale * p0);   // exact
    const float m1 = __builtin_fmaf((float)h[1], -kLowScale, kLowScale * p1);
    const half2_t g = cut(m0, m1);
    t[0] = __builtin_bit_cast(unsigned, h);
    t[1] = __builtin_bit_cast(unsigned, g);
    t[2] = __builtin_bit_cast(unsigned, cut(m0 - (float)g[0], m1 - (float)g[1]));
}

constexpr int low_bit(int n, int cap) { return (n & -n) < cap ? (n & -n) : cap; }
constexpr int log2i(int n) { return n > 1 ? 1 + log2i(n / 2) : 0; }

// DP: D rounded up to a multiple of 32 (columns past D are zeros); NSLOT
// blocks of 16 columns, KSP key parts, NB blocks of 16 keys per wave and tile.
template <typename TIN, int DP, int NSLOT, int KSP, int NB> struct GCfg {
    static constexpr bool F32 = sizeof(typename Elem<TIN>::scalar) == 4;
    static constexpr int ES = F32 ? 4 : 2;       // bytes per element
    static constexpr int E = 16 / ES;            // elements per 16-byte chunk
    static constexpr int CPR = DP / E;           // chunks per row
    static constexpr int KB = 16 * NB, BC = KB * KSP;
    static constexpr int NW = NSLOT * KSP;
    static constexpr int KBYTES = BC * DP * ES;  // a K tile (V the same)
    static constexpr int STAGE = 2 * KBYTES;
    static constexpr int PIECES = KBYTES / 1024; // loads of 64 chunks per tile, K and V each
    static constexpr int NP = (PIECES + NW - 1) / NW;
    static constexpr int NV = DP / 4 + 2;        // merge: accumulator, maximum and sum of a lane
    static constexpr int MERGE = (KSP - 1) * NSLOT * NV * 64 * 4;
    static constexpr int BYTES = 2 * STAGE > MERGE ? 2 * STAGE : MERGE;   // two stages
    // Swizzles: chunk c of row r is stored at chunk c ^ swz(r) of its row, so
    // that the 16 rows of a 16-byte operand read, the eight rows (fp32: four)
    // of a value read fall into different banks.
    static constexpr int ZK = low_bit(CPR, 16), ZV = F32 ? low_bit(CPR / 4, 4) : low_bit(CPR / 2, 8);
    static __device__ __forceinline__ int kswz(int r) { return (r >> (4 - log2i(ZK))) & (ZK - 1); }
    static __device__ __forceinline__ int vswz(int r) {
        return F32 ? ((r >> (2 - log2i(ZV))) & (ZV - 1)) << 2 : ((r >> (3 - log2i(ZV))) & (ZV - 1)) << 1;
    }
    // waves per SIMD to keep registers for: one workgroup's, and two
    // workgroups' where 128 registers are just enough for that (fp16 takes 133
    // there otherwise)
    static constexpr int WPE = !F32 && DP == 96 && NSLOT == 4 ? 4 : NW >= 4 ? NW / 4 : 1;
    static_assert(KBYTES % 1024 == 0 && (F32 || NB == 2), "tile shape");
};

template <typename TIN, typename TOUT, int DP, int NSLOT, int KSP, int NB>
__global__ __launch_bounds__(64 * NSLOT * KSP) __attribute__((amdgpu_waves_per_eu((GCfg<TIN, DP, NSLOT, KSP, NB>::WPE)))) void generic_kernel(GenericArgs a) {
    using SM = GCfg<TIN, DP, NSLOT, KSP, NB>;
    typedef typename Elem<TIN>::scalar S;
    constexpr bool F32 = SM::F32, F16 = __is_same(TIN, f16_t);
    constexpr int ES = SM::ES, E = SM::E, CPR = SM::CPR, KB = SM::KB, BC = SM::BC, NW = SM::NW, NP = SM::NP;
    constexpr int DT = DP / 16;                  // 16-column tiles of O
    constexpr bool PAGES = !F32 && (DP == 64 || DP == 128);   // K/V may come in pages
    constexpr bool VPRE = DP <= 128;             // value operands are read ahead of the softmax
    // fp32 products are issued at raised wave priority up to 64 columns: the
    // SIMD's other waves then fill the gaps with vector work (causal 16 heads,
    // 777 rows, D = 64 24.8 -> 23.4 us; 2 x 16, 600 rows, D = 32 16.4 -> 15.4;
    // wider rows and the shorter 16-bit products +-1 %)
    constexpr bool PRIO = F32 && DP <= 64;
    // partial sums of a score: fp32 takes D products in steps of four, one sum
    // of 64 steps would round more than the scores of sharp softmaxes allow
    constexpr int NSUM = !F32 ? 1 : DP <= 64 ? 2 : 4;
    // The base of a column's weights moves (and its sums are rescaled) only
    // when a score exceeds the largest one of that time by more than GROWTH.
    // That one then weighs 2^HEADROOM; weights reach 2^(HEADROOM + GROWTH), in
    // fp16 2^15, for the range of their terms.  Otherwise the value products take
    // SHARE of them (exact), so that a weight times any value stays in range; a
    // base higher by GROWTH would do that as well, but exponents further from 0
    // are rounded more coarsely (error against fp64, 16 heads, 777 rows, D = 64,
    // fp32 1.87e-7 -> 1.98e-7, 16/2, 1111 rows, D = 96, bf16 1.33e-7 -> 1.50e-7;
    // the multiplications take -1 to +1 %, bf16 at D = 256 1 to 4).
    constexpr float GROWTH = 4.f, HEADROOM = F16 ? 15.f - GROWTH : 0.f, SHARE = F16 ? 1.f : 0x1p-4f;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[SM::BYTES];

    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = l & 15, lg = l >> 4;
    const int slot = w % NSLOT, kp = w / NSLOT;
    // latest columns (most keys) first
    const int vb_r = (int)a.per_vb.div(blockIdx.x);
    const int rest = (int)(blockIdx.x - vb_r * a.per_vb.d);
    const int vb = a.nvb - 1 - vb_r;
    const int b = (int)a.nkv.div(rest), g = rest - b * (int)a.nkv.d;
    const int G = (int)a.group.d, D = a.D, Nq = a.Nq;
    // valid keys of this batch element (a.Nk rows per element in K and V)
    const int Nk = a.seqlens ? __builtin_amdgcn_readfirstlane(min(max(a.seqlens[b], 0), a.Nk)) : a.Nk;
    const int off = Nk - Nq;
    // Column t of the workgroup is column v0 + t of the key/value head: row
    // row0 + (rem0 + t) / G, head (rem0 + t) % G of the group.
    const long long v0 = (long long)vb * (QB * NSLOT);
    const int row0 = v0 < 0x7fffffffLL ? (int)a.group.div((unsigned)v0) : (int)(v0 / G);
    const unsigned rem0 = (unsigned)(v0 - (long long)row0 * G);
    const int cols = (int)__builtin_elementwise_min((long long)Nq * G - v0, (long long)(QB * NSLOT));
    auto row_of = [&](int t) { return row0 + (int)a.group.div(rem0 + t); };
    const int t0 = QB * slot;
    const bool valid = t0 + lc < cols;
    const int row = row_of(t0 + lc), h = g * G + (int)(rem0 + t0 + lc - (unsigned)(row - row0) * (unsigned)G);

    // Key extents: workgroup, wave, keys that every column of the wave sees,
    // and this lane's column (bottom-right causal alignment).
    auto extent = [&](int i) { return a.causal ? min(Nk, i + off + 1) : Nk; };
    const int kend_wg = extent(row_of(cols - 1));
    const int kend_w = t0 < cols ? extent(row_of(min(t0 + QB, cols) - 1)) : 0;
    const int kfree_w = t0 < cols ? extent(row_of(t0)) : 0;
    const int myend = extent(row);

    // Q operand: fp32, chunk i holds columns 16 i + 4 lg .. + 3; 16-bit, k-step
    // i holds columns 32 i + 8 lg .. + 7
    constexpr int NQF = F32 ? DP / 16 : DP / 32;
    uint4_t qf[NQF];
    {
        const S *qp = reinterpret_cast<const S *>(a.q) + ((size_t)((size_t)b * Nq + (valid ? row : 0)) * a.Hq + (valid ? h : 0)) * D;
#pragma unroll
        for (int i = 0; i < NQF; ++i) {
            const int d = 4 * E * i + E * lg;
            qf[i] = uint4_t{0u, 0u, 0u, 0u};
            if (valid && d < D) qf[i] = ld16(qp + d) ^ a.qsign;
        }
    }

    // Tile staging, memory to LDS directly: piece j of a tile is its chunks
    // 64 j .. 64 j + 63, lane l's the l-th; chunks past D and keys past the
    // end (past the view's) become zeros.
    const long long pitch = (long long)a.Hkv * D * ES;   // bytes between consecutive keys
    // a tile's offsets exceed a buffer view's 31 bits; so they do where K/V
    // come in pages (other paged calls take the prefill and decode kernels)
    const bool far = pitch * BC > 0x7fffffffLL;
    int koff[NP], voff[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int e = 64 * (w + NW * j) + l, r = e / CPR, c = e % CPR;
        const int ck = c ^ SM::kswz(r), cv = c ^ SM::vswz(r);
        koff[j] = E * ck < D ? r * (int)pitch + 16 * ck : (int)0x80000000;
        voff[j] = E * cv < D ? r * (int)pitch + 16 * cv : (int)0x80000000;
    }
    const unsigned lds0 = lds_address(smem);
    const size_t head0 = ((PAGES && a.block_table ? 0 : (size_t)b * a.Nk * a.Hkv) + g) * (size_t)D * ES;
    const char *ktile = reinterpret_cast<const char *>(a.k) + head0;
    const char *vtile = reinterpret_cast<const char *>(a.v) + head0;
    long long left = (long long)(Nk - 1) * pitch + D * ES;   // bytes from the next tile's first key to the last one's end
    auto load_tile = [&](int k0, int st) {   // tiles are loaded in order
        if (!far) {
            const int nrec = (int)__builtin_elementwise_min(left, 0x7fffffffLL);
            const unsigned dst = lds0 + st * SM::STAGE + 1024 * w;
#pragma unroll
            for (int j = 0; j < NP; ++j)
                if (SM::PIECES % NW == 0 || w + NW * j < SM::PIECES) load_lds16(ktile, nrec, dst + 1024 * NW * j, koff[j]);
#pragma unroll
            for (int j = 0; j < NP; ++j)
                if (SM::PIECES % NW == 0 || w + NW * j < SM::PIECES)
                    load_lds16(vtile, nrec, dst + SM::KBYTES + 1024 * NW * j, voff[j]);
        } else {   // the same through registers, with 64-bit offsets, a page number for each row of paged K/V
            for (int e = tid; e < BC * CPR; e += 64 * NW) {
                const int r = e / CPR, c = e % CPR;
                uint4_t kc = uint4_t{0u, 0u, 0u, 0u}, vc = kc;
                if (k0 + r < Nk && E * c < D) {
                    long long row = r;   // from the tile's first key, or from the pool's first row
                    if (PAGES && a.block_table) {
                        const int pi = (int)a.page_size.div(k0 + r);
                        const int page = min(max(a.block_table[(size_t)b * a.max_pages + pi], 0), a.num_pages - 1);
                        row = (long long)page * a.page_size.d + (k0 + r - pi * (int)a.page_size.d);
                    }
                    kc = ld16(ktile + row * pitch + 16 * c);
                    vc = ld16(vtile + row * pitch + 16 * c);
                }
                unsigned char *row_at = smem + st * SM::STAGE + r * (DP * ES);
                st16(row_at + 16 * (c ^ SM::kswz(r)), kc);
                st16(row_at + SM::KBYTES + 16 * (c ^ SM::vswz(r)), vc);
            }
        }
        if (!PAGES || !a.block_table) {
            ktile += BC * pitch;
            vtile += BC * pitch;
        }
        left -= BC * pitch;
    };

    // Accumulators.  16-bit inputs: the weights' first terms in oacc, the
    // others in olow (apart, so that an infinite value, times a zero term,
    // does not turn into NaN; in fp16 kLowScale times their sum).
    float4_t oacc[DT], olow[F32 ? 1 : DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        oacc[dt] = float4_t{};
        if constexpr (!F32) olow[dt] = float4_t{};
    }
    // Base of the column's weights (log2 domain; the same in its four lanes)
    // and the largest score it is kept for; no score seen yet: 0 and -inf.
    float base = 0.f, lim = -INFINITY;
    float lsum = 0.f;      // this lane's part of the sum

    // Lane constants of the operand reads.  Key of a lane's score 4 j + r:
    // 16 j + 4 lg + r, in fp32 (rows of K read in the order 4 (i % 4) + i / 4)
    // 16 j + 4 r + lg, so that the four rows of a value read are consecutive.
    const int krow = KB * kp + (F32 ? 4 * (lc & 3) + (lc >> 2) : lc);
    const int vrow = KB * kp + (F32 ? lg : 4 * lg + (lc >> 2));
    auto block = [&](int kb, const unsigned char *ks) {   // the wave's KB keys of a tile
        const unsigned char *vs = ks + SM::KBYTES;

        // ---- scores
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
        float x[4 * NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            float4_t sc[NSUM];
#pragma unroll
            for (int n = 0; n < NSUM; ++n) sc[n] = float4_t{};
            const unsigned char *kl = ks + (krow + 16 * j) * (DP * ES);
#pragma unroll
            for (int i = 0; i < NQF; ++i) {
                const uint4_t ku = *reinterpret_cast<const uint4_t *>(kl + 16 * ((4 * i + lg) ^ SM::kswz(krow)));
                if constexpr (F32) {
                    const float4_t kf = __builtin_bit_cast(float4_t, ku), q4 = __builtin_bit_cast(float4_t, qf[i]);
#pragma unroll
                    for (int n = 0; n < 4; ++n) sc[n % NSUM] = mfma4(kf[n], q4[n], sc[n % NSUM]);
                } else {
                    typedef typename TIN::vec8 V8;
                    sc[0] = mfma16(as_vec8<V8>(ku), as_vec8<V8>(qf[i]), sc[0]);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) x[4 * j + r] = NSUM == 4 ? (sc[0][r] + sc[NSUM > 1 ? 1 : 0][r]) + (sc[NSUM - 2][r] + sc[NSUM - 1][r]) : NSUM == 2 ? sc[0][r] + sc[NSUM > 1 ? 1 : 0][r] : sc[0][r];
        }
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
        if (kb + KB > kfree_w) {   // wave-uniform: some column does not see all of them
#pragma unroll
            for (int i = 0; i < 4 * NB; ++i)
                x[i] = kb + 16 * (i / 4) + (F32 ? 4 * (i % 4) + lg : 4 * lg + i % 4) < myend ? x[i] : -INFINITY;
        }

        // value operands, ahead of the softmax
        typedef typename std::conditional<F32, float, uint4_t>::type vop_t;
        constexpr int NVO = F32 ? 4 * NB : 1;    // operands per column tile
        auto vread = [&](int i, int dt) {
            if constexpr (F32) {
                return *reinterpret_cast<const float *>(vs + (vrow + 16 * (i / 4) + 4 * (i % 4)) * (DP * ES) +
                                                        64 * (dt ^ (SM::vswz(vrow + 4 * (i % 4)) >> 2)) + 4 * lc);
            } else {
                const _Float16 *p = reinterpret_cast<const _Float16 *>(vs + vrow * (DP * ES) + 32 * (dt ^ (SM::vswz(vrow) >> 1)) + 8 * (lc & 3));
                return __builtin_bit_cast(uint4_t, cat_half8(lds_read_tr16(p), lds_read_tr16(p + 16 * DP)));
            }
        };
        vop_t va[NVO][DT];
        if constexpr (VPRE) {
#pragma unroll
            for (int i = 0; i < NVO; ++i)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) va[i][dt] = vread(i, dt);
        }

        // ---- streaming softmax
        float mx = max3_nan(x[0], x[1], x[2]);
#pragma unroll
        for (int i = 3; i + 1 < 4 * NB; i += 2) mx = max3_nan(mx, x[i], x[i + 1]);
        mx = quad_max(max_nan(mx, x[4 * NB - 1])) * a.c;
        if (__builtin_amdgcn_ballot_w64(mx > lim)) {
            const bool over = mx > lim;
            const float b_new = over ? mx - HEADROOM : base;
            const float alpha = lim == -INFINITY ? 0.f : exp2_fast(base - b_new);
            base = b_new;
            if (over) lim = mx + GROWTH;
            lsum *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                oacc[dt] *= alpha;
                if constexpr (!F32) olow[dt] *= alpha;
            }
        }
        float p[4 * NB];
#pragma unroll
        for (int i = 0; i < 4 * NB; ++i) p[i] = exp2_fast(__builtin_fmaf(x[i], a.c, -base));
#pragma unroll
        for (int j = 0; j < NB; ++j) lsum += (p[4 * j] + p[4 * j + 1]) + (p[4 * j + 2] + p[4 * j + 3]);

        // ---- values
        if constexpr (!F16) {
#pragma unroll
            for (int i = 0; i < 4 * NB; ++i) p[i] *= SHARE;
        }
        if constexpr (F32) {
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < 4 * NB; ++i)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) oacc[dt] = mfma4(VPRE ? va[i][dt] : vread(i, dt), p[i], oacc[dt]);
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
        } else {
            typedef typename TIN::vec8 V8;
            // fp16: does some weight lie below what three terms hold in full?
            unsigned long long small = 0;
            if constexpr (F16) {
                float least = p[0];
#pragma unroll
                for (int i = 1; i < 8; ++i) least = min_nan(least, p[i]);
                if (__builtin_amdgcn_ballot_w64(least < kLeast) != 0) {
                    bool some = false;
#pragma unroll
                    for (int i = 0; i < 8; ++i) some |= p[i] > 0.f && p[i] < kLeast;
                    small = __builtin_amdgcn_ballot_w64(some);
                }
                if (small) {   // the products in fp32: element i of a lane's operand is the value of its weight i
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        const V8 vv = as_vec8<V8>(VPRE ? va[0][dt] : vread(0, dt));
#pragma unroll
                        for (int i = 0; i < 8; ++i) oacc[dt] = mfma4((float)vv[i], p[i], oacc[dt]);
                        __builtin_amdgcn_sched_barrier(0);   // one tile's operands at a time, in few registers
                    }
                }
                asm volatile("" : "+s"(small));   // two conditions: as the sides of one, each has its own registers
            }
            if (!small) {
                uint4_t pt[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    unsigned t[3];
                    split3(p[2 * i], p[2 * i + 1], t, TIN());
#pragma unroll
                    for (int n = 0; n < 3; ++n) pt[n][i] = t[n];
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const V8 vv = as_vec8<V8>(VPRE ? va[0][dt] : vread(0, dt));
                    oacc[dt] = mfma16(vv, as_vec8<V8>(pt[0]), oacc[dt]);
                    olow[dt] = mfma16(vv, as_vec8<V8>(pt[1]), olow[dt]);
                    olow[dt] = mfma16(vv, as_vec8<V8>(pt[2]), olow[dt]);
                }
            }
        }
    };

    if (kend_wg > 0) load_tile(0, 0);
    // Q has arrived here, so that no wait for it stands in the loop
#pragma unroll
    for (int i = 0; i < NQF; ++i) asm volatile("" : "+v"(qf[i]));
    for (int k0 = 0, st = 0; k0 < kend_wg; k0 += BC, st ^= 1) {
        lds_loads_done<0>();
        lds_barrier();
        if (k0 + BC < kend_wg) load_tile(k0 + BC, st ^ 1);
        const int kb = k0 + KB * kp;
        if (kb < kend_w) block(kb, smem + st * SM::STAGE);   // else no column sees these keys (wave-uniform)
    }
    float m = lim == -INFINITY ? -INFINITY : base;
    if constexpr (!F32) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r)   // (the first terms' sum alone where it is not finite)
                oacc[dt][r] = oacc[dt][r] - oacc[dt][r] == 0.f
                                  ? __builtin_fmaf(olow[dt][r], F16 ? 1.f / kLowScale : 1.f, oacc[dt][r]) : oacc[dt][r];
    }

    // ---- merge the key parts of each slot through LDS
    if constexpr (KSP > 1) {
        lds_barrier();
        constexpr int NV = SM::NV;
        float *mf = reinterpret_cast<float *>(smem) + l;
        if (kp > 0) {
            float *mine = mf + ((kp - 1) * NSLOT + slot) * NV * 64;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 4; ++r) mine[(4 * dt + r) * 64] = oacc[dt][r];
            mine[(NV - 2) * 64] = m;
            mine[(NV - 1) * 64] = lsum;
        }
        __syncthreads();
        if (kp > 0) return;
        float M = m;
#pragma unroll
        for (int j = 0; j < KSP - 1; ++j) M = __builtin_fmaxf(M, mf[((j * NSLOT + slot) * NV + NV - 2) * 64]);
        const float a0 = (m == -INFINITY) ? 0.f : exp2_fast(m - M);
        lsum *= a0;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) oacc[dt] *= a0;
#pragma unroll
        for (int j = 0; j < KSP - 1; ++j) {
            const float *other = mf + (j * NSLOT + slot) * NV * 64;
            const float mj = other[(NV - 2) * 64];
            const float aj = (mj == -INFINITY) ? 0.f : exp2_fast(mj - M);
            lsum = __builtin_fmaf(aj, other[(NV - 1) * 64], lsum);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int r = 0; r < 4; ++r) oacc[dt][r] = __builtin_fmaf(aj, other[(4 * dt + r) * 64], oacc[dt][r]);
        }
        m = M;
    }
    lsum = pair_sum(half_sum(lsum));
    if (!valid) return;
    const float inv = lsum > 0.f ? (1.f / SHARE) / lsum : 0.f;   // no visible key: 0
    TOUT *op = reinterpret_cast<TOUT *>(a.o) + ((size_t)((size_t)b * Nq + row) * a.Hq + h) * D;
    if constexpr (sizeof(TOUT) == 4) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const int d = 16 * dt + 4 * lg;
            if (d < D) *reinterpret_cast<float4_t *>(op + d) = oacc[dt] * inv;
        }
    } else {
        // lanes l and l ^ 16 have halves of an 8-column chunk in each of two
        // column tiles and exchange them, so that each stores 16 bytes (16 heads,
        // 300 rows, D = 256, bf16 16.9 -> 16.4 us; 4 x 32/8, 2048 rows, D = 96
        // -3 %; small calls +-1 %)
        typedef TOUT t4 __attribute__((ext_vector_type(4)));
        typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int dt = 0; dt < DT; dt += 2) {
            uint2_t u[2];
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                t4 x;
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] = from_f32<TOUT>(oacc[dt + n][r] * inv);
                u[n] = __builtin_bit_cast(uint2_t, x);
            }
            auto lo = __builtin_amdgcn_permlane16_swap(u[0][0], u[1][0], false, false);
            auto hi = __builtin_amdgcn_permlane16_swap(u[0][1], u[1][1], false, false);
            const int d = 16 * (dt + (lg & 1)) + 8 * (lg >> 1);
            if (d < D) st16(op + d, uint4_t{lo[0], hi[0], lo[1], hi[1]});
        }
    }
    if (a.lse && lg == 0)
        a.lse[((size_t)b * a.Hq + h) * Nq + row] = lsum > 0.f ? (m + log2f(lsum)) * kLn2 : -INFINITY;
}

template <typename TIN, typename TOUT, int DP, int NSLOT, int KSP, int NB>
hipError_t launch_t(const Problem &p, hipStream_t stream) {
    GenericArgs a;
    a.q = p.q; a.k = p.k; a.v = p.v; a.o = p.o; a.lse = p.lse;
    a.B = p.B; a.Hq = p.Hq; a.Hkv = p.Hkv; a.Nq = p.Nq; a.Nk = p.Nk; a.D = p.D;
    a.causal = p.causal;
    a.seqlens = p.seqlens;
    a.block_table = p.block_table;
    a.page_size = Divisor(p.block_table ? p.page_size : 1);
    a.max_pages = p.max_pages;
    a.num_pages = p.num_pages;
    // A zero scale keeps a positive factor, for masked scores of -inf: the least
    // there is, which moves no weight by more than 2^-21.
    a.c = __builtin_fmaxf(__builtin_fabsf(p.scale) * kLog2e, 0x1p-149f);
    a.qsign = p.scale < 0.f ? (sizeof(typename Elem<TIN>::scalar) == 4 ? 0x80000000u : 0x80008000u) : 0u;
    constexpr int COLS = QB * NSLOT;
    const long long nvb = ((long long)p.Nq * (p.Hq / p.Hkv) + COLS - 1) / COLS;
    const long long nblocks = nvb * p.B * p.Hkv;
    if (nblocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.nvb = (int)nvb;
    a.per_vb = Divisor((unsigned)p.B * p.Hkv);   // <= nblocks
    a.nkv = Divisor(p.Hkv);
    a.group = Divisor(p.Hq / p.Hkv);
    hipLaunchKernelGGL((generic_kernel<TIN, TOUT, DP, NSLOT, KSP, NB>), dim3((unsigned)nblocks), dim3(64 * NSLOT * KSP), 0, stream, a);
    return hipGetLastError();
}

// Layouts (column blocks, key parts).  A tile staged for more columns costs
// less per column; more key parts, and more workgroups of fewer columns,
// shorten the longest chain of steps.  So: small workgroups while they all
// start at once (a causal call of about square shape: twice as many, the
// second half being short), large ones for grids that fill the card anyway.
// In us, on both sides of each line:
//   fp32, up to 128 columns: (1, 4) against (2, 4): 16 heads, 777 rows causal,
//     D = 64 24.2 / 26.1; decode 16 x 32/8 x 2048, D = 64 36.5 / 47.5; past
//     the line, 8/2 heads x 1000, D = 96 54.8 / 38.6, 4 x 32/8 x 1024 causal,
//     D = 64 227 / 171
//   16 bits, up to 128: (2, 4) against (4, 2): 16 x 512, D = 80 9.4 / 12.6;
//     16/2 x 100 against 4000, D = 96 35 / 63; 32/8 x 2048 causal, D = 96
//     100 / 65.  Between them, causal calls of about square shape, (2, 2) at 65
//     to 96 columns, where three of its workgroups fit a CU and one of (2, 4):
//     over 96 grids between the lines, D = 72 to 96, -11 to +4 % against (4, 2),
//     slower only from 700 workgroups of many heads on (bf16, D = 80: 16/2 x 1026
//     rows 18.7 / 19.8, x 1526 26.0 / 29.1, 32/8 x 666 14.7 / 15.8, x 758 18.3 /
//     17.5; not causal, 2 x 16/2 x 600, D = 88 25.0 / 19.6).  Up to 64 columns the
//     line of (2, 4) lies at twice as many workgroups, and past it (2, 2) is the
//     slower one (16/2 x 2221, D = 56 36.5 / 31.4; 32/8 x 1108 23.1 / 19.0; D = 32,
//     1531 rows 22.4 / 23.0, 2560 49.3 / 45.0); at 97 to 128 no grid lies between
//   fp32, above 128: (2, 2) against (4, 2): 16 x 777 causal, D = 192 62 / 85;
//     16 x 1024, D = 192 154 / 115; up to 160 columns, where two workgroups of (2,
//     2) fit a CU, no grid is slower with it by more than 2 % (32/8, D = 160:
//     causal, 1024 rows 119 / 116, 1371 199 / 214, 2080 410 / 428; not causal, 1718
//     573 / 653)
//   above 128, (4, 2) against (8, 1): bf16 16/2 x 1111 causal, D = 256
//     40 / 62; from a workgroup of (8, 1) for every CU, 32/8 x 1024, D = 256
//     77 / 66, fp32 32 x 1024, D = 192 224 / 212.  (8, 1) gains 5 to 14 % in bf16, 3
//     to 6 in fp32, where its rounds are full, as they are from some two rounds
//     on; it loses where they are not (not causal, 300 to 390 workgroups, +13 to
//     +26 %) and where a causal call's longest row block then decides (bf16, D =
//     256, 32/8 x 1024 45.6 / 59.5, x 1371 80.6 / 77.3, x 1718 110 / 94)
// The lines are those of a whole card, so that a call's layout, and with it the
// order of its sums, does not go by the device's mode.
template <typename TIN, typename TOUT, int DP>
hipError_t launch_k(const Problem &p, hipStream_t s) {
    constexpr bool F32 = sizeof(typename Elem<TIN>::scalar) == 4, WIDE = DP > 128;
    constexpr int NB = F32 ? 1 : 2;
    const long long cols = (long long)p.Nq * (p.Hq / p.Hkv), kvheads = (long long)p.B * p.Hkv;
    auto groups = [&](int ns) { return (cols + QB * ns - 1) / (QB * ns) * kvheads; };   // workgroups of ns blocks
    constexpr bool PAIR = F32 && WIDE && 2 * GCfg<TIN, DP, 2, 2, NB>::BYTES <= 163840;   // two workgroups of (2, 2) fit a CU
    if constexpr (PAIR) {
        return launch_t<TIN, TOUT, DP, 2, 2, NB>(p, s);
    } else if constexpr (F32 || !WIDE) {
        constexpr int NS = F32 && !WIDE ? 1 : 2, KSP = WIDE ? 2 : 4;
        constexpr int FIT = 163840 / GCfg<TIN, DP, NS, KSP, NB>::BYTES;   // workgroups per CU by LDS
        const int rounds = p.causal && p.Nk < 2LL * p.Nq ? 2 : 1;
        if (groups(NS) <= CUS * (FIT < 2 ? FIT : 2) * rounds) return launch_t<TIN, TOUT, DP, NS, KSP, NB>(p, s);
        if constexpr (!F32 && DP == 96) {
            constexpr int FIT2 = 163840 / GCfg<TIN, DP, 2, 2, NB>::BYTES;
            if (rounds == 2 && groups(2) <= CUS * FIT2) return launch_t<TIN, TOUT, DP, 2, 2, NB>(p, s);
        }
    }
    if constexpr (WIDE && !PAIR) {
        if (groups(8) >= CUS) return launch_t<TIN, TOUT, DP, 8, 1, NB>(p, s);
    }
    if constexpr (F32 && !WIDE) return launch_t<TIN, TOUT, DP, 2, 4, NB>(p, s);
    else if constexpr (!PAIR) return launch_t<TIN, TOUT, DP, 4, 2, NB>(p, s);
}

template <typename TIN, typename TOUT>
hipError_t launch_d(const Problem &p, hipStream_t s) {
    switch ((p.D + 31) / 32) {
    case 1: return launch_k<TIN, TOUT, 32>(p, s);
    case 2: return launch_k<TIN, TOUT, 64>(p, s);
    case 3: return launch_k<TIN, TOUT, 96>(p, s);
    case 4: return launch_k<TIN, TOUT, 128>(p, s);
    case 5: return launch_k<TIN, TOUT, 160>(p, s);
    case 6: return launch_k<TIN, TOUT, 192>(p, s);
    case 7: return launch_k<TIN, TOUT, 224>(p, s);
    default: return launch_k<TIN, TOUT, 256>(p, s);
    }
}

}  // namespace

hipError_t launch_generic(const Problem &p, hipStream_t stream) {
    switch (p.in) {
    case FA_F32:
        return launch_d<float, float>(p, stream);
    case FA_F16:
        return p.out == FA_F32 ? launch_d<f16_t, float>(p, stream)
                               : launch_d<f16_t, _Float16>(p, stream);
    default:
        return p.out == FA_F32 ? launch_d<bf16_t, float>(p, stream)
                               : launch_d<bf16_t, __bf16>(p, stream);
    }
}

}  // namespace fa
