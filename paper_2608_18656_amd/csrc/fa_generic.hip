// fa_generic.hip -- attention forward with fp32 weights, for the cases the
// half-precision matrix kernels do not take: fp32 inputs, and fp16 / bf16 with
// a head dimension other than 64 or 128 (any D with D % 8 == 0 and D <= 256),
// prefill and decode.
//
// Everything after the loads is fp32: scores are fp32 sums, the weights stay
// fp32 and multiply fp32 values.  Both products run on the matrix cores:
//   S^T = K Q^T   fp32 inputs: 16x16x4 fp32 MFMA; fp16 / bf16: 16x16x32 MFMA
//                 of the inputs as they are (exact products, fp32 sums)
//   O^T += V^T P^T   16x16x4 fp32 MFMA; P straight from the score registers
//                 (step r takes key 4 (l / 16) + r of every lane group), V from
//                 LDS in fp32 (fp16 / bf16 values are widened while staged)
//
// Work split.  The Nq * G query rows of the G heads that read one key/value
// head are numbered together, v = row * G + head, and 16 consecutive ones are
// the columns of a wave's matrix products, so a group's heads share every
// staged key and a decode call (Nq = 1) fills columns with heads.  A workgroup
// of eight waves is NSLOT slots of 16 columns times KSP key parts: a tile of
// 16 KSP keys is staged in LDS for all of them (the next tile's loads are in
// flight meanwhile) and part j takes its keys 16 j .. 16 j + 15.  The parts'
// states are merged through LDS at the end.
//
// What bounds it: the fp32 MFMA (64 flop per cycle and SIMD).  One wave's
// 16 x 16 block takes D / 4 score and D / 4 value steps of 32 cycles, against
// D / 4 16-byte and D / 4 4-byte LDS reads, a quarter of what LDS delivers.
#include "fa_common.h"
#include "fa_internal.h"

namespace fa {
namespace {

constexpr int KB = 16;    // keys per wave and tile
constexpr int QB = 16;    // query columns per wave
constexpr int NWAVE = 8;  // waves per workgroup
constexpr int NTH = 64 * NWAVE;

struct GenericArgs {
    const void *q, *k, *v;
    void *o;
    float *lse;
    int B, Hq, Hkv, Nq, Nk, D;
    int causal;
    float c;   // scale * log2(e), signed
    int nvb;   // blocks of 16 NSLOT columns per key/value head
    const int *seqlens;   // valid keys per batch element (NULL: Nk for all)
};

__device__ __forceinline__ float4_t mfma4(float a, float b, float4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Element types as the kernel uses them: the storage scalar, and for fp16 /
// bf16 the operand type of the score product.
template <typename T> struct Elem;
template <> struct Elem<float> { typedef float scalar; };
template <> struct Elem<f16_t> { typedef _Float16 scalar; };
template <> struct Elem<bf16_t> { typedef __bf16 scalar; };

// DP: D rounded up to a multiple of 32 (columns past D are zeros).
template <typename TIN, int DP, int KSP> struct GSmem {
    static constexpr bool F32 = sizeof(typename Elem<TIN>::scalar) == 4;
    static constexpr int NSLOT = NWAVE / KSP;
    static constexpr int BC = KB * KSP;
    // row strides: fp32 rows of DP + 4 words put the 16 rows of a 16-byte
    // operand read, and the rows 4 apart of a value read, in different banks;
    // 16-bit rows of DP + 8 do the same for the score operands
    static constexpr int KS = F32 ? DP + 4 : DP + 8;
    static constexpr int VS = DP + 4;
    static constexpr int KBYTES = BC * KS * (F32 ? 4 : 2);
    static constexpr int STAGE = KBYTES + BC * VS * 4;
    static constexpr int NV = DP / 4 + 2;   // merge: accumulator, maximum and sum of a lane
    static constexpr int MERGE = (KSP - 1) * NSLOT * NV * 64 * 4;
    static constexpr int BYTES = 2 * STAGE > MERGE ? 2 * STAGE : MERGE;   // two stages
};

template <typename TIN, typename TOUT, int DP, int KSP>
__global__ __launch_bounds__(NTH) void generic_kernel(GenericArgs a) {
    using SM = GSmem<TIN, DP, KSP>;
    typedef typename Elem<TIN>::scalar S;
    constexpr bool F32 = SM::F32;
    constexpr int NSLOT = SM::NSLOT, BC = SM::BC, KS = SM::KS, VS = SM::VS;
    constexpr int DT = DP / 16;                  // 16-column tiles of O
    constexpr bool VPRE = DP <= 128;             // value operands are read ahead of the softmax
    constexpr int E = 16 / sizeof(S);            // elements per 16-byte chunk
    constexpr int CPR = DP / E;                  // chunks per row
    constexpr int NCH = (BC * CPR + NTH - 1) / NTH;   // chunks per thread, K and V each
    __shared__ __attribute__((aligned(16))) unsigned char smem[SM::BYTES];
    auto ks_at = [&](int r) { return reinterpret_cast<S *>(smem + r * SM::STAGE); };
    auto vs_at = [&](int r) { return reinterpret_cast<float *>(smem + r * SM::STAGE + SM::KBYTES); };

    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = l & 15, lg = l >> 4;
    const int slot = w % NSLOT, kp = w / NSLOT;
    // latest columns (most keys) first
    const int per_vb = a.B * a.Hkv;
    const int vb = a.nvb - 1 - (int)blockIdx.x / per_vb;
    const int rest = (int)blockIdx.x % per_vb;
    const int g = rest % a.Hkv, b = rest / a.Hkv;
    const int G = a.Hq / a.Hkv, D = a.D, Nq = a.Nq;
    const long long VR = (long long)Nq * G;      // columns of this key/value head
    // valid keys of this batch element (a.Nk rows per element in K and V)
    const int Nk = a.seqlens ? min(max(a.seqlens[b], 0), a.Nk) : a.Nk;
    const int off = Nk - Nq;
    const long long v_wg = (long long)vb * (QB * NSLOT), v_w = v_wg + slot * QB;
    // row of a wave-uniform column (in 32 bits where the columns fit)
    auto row_of = [&](long long v) { return VR <= 0x7fffffffLL ? (int)((unsigned)v / (unsigned)G) : (int)(v / G); };
    const bool valid = v_w + lc < VR;
    const int row_w = row_of(v_w);
    const unsigned vrem = (unsigned)(v_w - (long long)row_w * G) + lc;   // < G + 16
    const int row = row_w + (int)(vrem / (unsigned)G), h = g * G + (int)(vrem % (unsigned)G);

    // Key extents: workgroup, wave, keys that every column of the wave sees,
    // and this lane's column (bottom-right causal alignment).
    auto extent = [&](int i) { return a.causal ? min(Nk, i + off + 1) : Nk; };
    const int kend_wg = extent(row_of(__builtin_elementwise_min(v_wg + QB * NSLOT, VR) - 1));
    const int kend_w = v_w < VR ? extent(row_of(__builtin_elementwise_min(v_w + QB, VR) - 1)) : 0;
    const int kfree_w = v_w < VR ? extent(row_w) : 0;
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
            if (valid && d < D) qf[i] = ld16(qp + d);
        }
    }

    // Tile staging: chunk e = tid + NTH c is key e / CPR, 16-byte chunk e % CPR;
    // columns past D and keys past the end read as zero.
    uint4_t kr[NCH], vr[NCH];
    const size_t kv0 = ((size_t)b * a.Nk * a.Hkv + g) * D;
    auto load_tile = [&](int k0) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int e = tid + NTH * c, key = k0 + e / CPR, d = E * (e % CPR);
            kr[c] = uint4_t{0u, 0u, 0u, 0u};
            vr[c] = uint4_t{0u, 0u, 0u, 0u};
            if (e < BC * CPR && key < Nk && d < D) {
                const size_t o = kv0 + (size_t)key * a.Hkv * D + d;
                kr[c] = ld16(reinterpret_cast<const S *>(a.k) + o);
                vr[c] = ld16(reinterpret_cast<const S *>(a.v) + o);
            }
        }
    };
    auto store_tile = [&](int r) {
        S *ks = ks_at(r);
        float *vs = vs_at(r);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int e = tid + NTH * c, key = e / CPR, d = E * (e % CPR);
            if (BC * CPR % NTH == 0 || e < BC * CPR) {
                st16(ks + key * KS + d, kr[c]);
                if constexpr (F32) {
                    st16(vs + key * VS + d, vr[c]);
                } else {
                    typedef S s8 __attribute__((ext_vector_type(8)));
                    const s8 x = __builtin_bit_cast(s8, vr[c]);
                    *reinterpret_cast<float4_t *>(vs + key * VS + d) =
                        float4_t{to_f32(x[0]), to_f32(x[1]), to_f32(x[2]), to_f32(x[3])};
                    *reinterpret_cast<float4_t *>(vs + key * VS + d + 4) =
                        float4_t{to_f32(x[4]), to_f32(x[5]), to_f32(x[6]), to_f32(x[7])};
                }
            }
        }
    };

    float4_t oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt] = float4_t{};
    float m = -INFINITY;   // running maximum of the column (log2 domain), the same in its four lanes
    float lsum = 0.f;      // this lane's part of the sum

    auto block = [&](int kb, const S *ks, const float *vs) {   // the wave's 16 keys of a tile

        // ---- scores: lane holds keys kb + 4 lg + r of column lc
        float4_t s0 = float4_t{}, s1 = float4_t{};
        const S *kl = ks + (KB * kp + lc) * KS + E * lg;
#pragma unroll
        for (int i = 0; i < NQF; ++i) {
            const uint4_t ku = *reinterpret_cast<const uint4_t *>(kl + 4 * E * i);
            if constexpr (F32) {
                const float4_t kf = __builtin_bit_cast(float4_t, ku), q4 = __builtin_bit_cast(float4_t, qf[i]);
                s0 = mfma4(kf[0], q4[0], s0);
                s1 = mfma4(kf[1], q4[1], s1);
                s0 = mfma4(kf[2], q4[2], s0);
                s1 = mfma4(kf[3], q4[3], s1);
            } else {
                typedef typename TIN::vec8 V8;
                s0 = mfma16(as_vec8<V8>(ku), as_vec8<V8>(qf[i]), s0);
            }
        }
        float x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = (F32 ? s0[r] + s1[r] : s0[r]) * a.c;
        if (kb + KB > kfree_w) {   // wave-uniform: some column does not see all of them
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] = kb + 4 * lg + r < myend ? x[r] : -INFINITY;
        }

        // value operands, ahead of the softmax
        const float *vl = vs + (KB * kp + 4 * lg) * VS + lc;
        float va[4][DT];
        if constexpr (VPRE) {   // (up to 32 registers)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) va[r][dt] = vl[r * VS + 16 * dt];
        }

        // ---- streaming softmax
        float mx = __builtin_fmaxf(__builtin_fmaxf(x[0], x[1]), __builtin_fmaxf(x[2], x[3]));
        mx = __builtin_fmaxf(mx, __shfl_xor(mx, 16));
        mx = pair_max(mx);
        const float m_new = __builtin_fmaxf(m, mx);
        if (__builtin_amdgcn_ballot_w64(m_new > m)) {
            const float alpha = (m == -INFINITY) ? 0.f : exp2_fast(m - m_new);
            m = m_new;
            lsum *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[dt] *= alpha;
        }
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = (x[r] == -INFINITY) ? 0.f : exp2_fast(x[r] - m);
        lsum += (p[0] + p[1]) + (p[2] + p[3]);

        // ---- values: step r multiplies keys kb + 4 lg + r of all lane groups
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[dt] = mfma4(VPRE ? va[r][dt] : vl[r * VS + 16 * dt], p[r], oacc[dt]);
        }
    };

    if (kend_wg > 0) {
        load_tile(0);
        store_tile(0);
    }
    // Q has arrived here, so that no wait for it stands in the loop (where it
    // would also cover the loads of the next tile)
#pragma unroll
    for (int i = 0; i < NQF; ++i) asm volatile("" : "+v"(qf[i]));
    __syncthreads();
    for (int k0 = 0, st = 0; k0 < kend_wg; k0 += BC, st ^= 1) {
        const bool more = k0 + BC < kend_wg;
        if (more) load_tile(k0 + BC);
        const int kb = k0 + KB * kp;
        if (kb < kend_w) block(kb, ks_at(st), vs_at(st));   // else no column sees these keys (wave-uniform)
        if (more) store_tile(st ^ 1);
        __syncthreads();
    }

    // ---- merge the key parts of each slot through LDS
    if constexpr (KSP > 1) {
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
    lsum += __shfl_xor(lsum, 16);
    lsum = pair_sum(lsum);
    if (!valid) return;
    const float inv = lsum > 0.f ? 1.f / lsum : 0.f;   // no visible key: 0
    TOUT *op = reinterpret_cast<TOUT *>(a.o) + ((size_t)((size_t)b * Nq + row) * a.Hq + h) * D;
    typedef TOUT t4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        const int d = 16 * dt + 4 * lg;
        if (d < D) {
            t4 u;
#pragma unroll
            for (int r = 0; r < 4; ++r) u[r] = from_f32<TOUT>(oacc[dt][r] * inv);
            *reinterpret_cast<t4 *>(op + d) = u;
        }
    }
    if (a.lse && lg == 0)
        a.lse[((size_t)b * a.Hq + h) * Nq + row] = lsum > 0.f ? (m + log2f(lsum)) * kLn2 : -INFINITY;
}

template <typename TIN, typename TOUT, int DP, int KSP>
hipError_t launch_t(const Problem &p, hipStream_t stream) {
    GenericArgs a;
    a.q = p.q; a.k = p.k; a.v = p.v; a.o = p.o; a.lse = p.lse;
    a.B = p.B; a.Hq = p.Hq; a.Hkv = p.Hkv; a.Nq = p.Nq; a.Nk = p.Nk; a.D = p.D;
    a.causal = p.causal;
    a.seqlens = p.seqlens;
    a.c = p.scale * kLog2e;
    constexpr int COLS = QB * NWAVE / KSP;
    const long long nvb = ((long long)p.Nq * (p.Hq / p.Hkv) + COLS - 1) / COLS;
    const long long nblocks = nvb * p.B * p.Hkv;
    if (nblocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.nvb = (int)nvb;
    hipLaunchKernelGGL((generic_kernel<TIN, TOUT, DP, KSP>), dim3((unsigned)nblocks), dim3(NTH), 0, stream, a);
    return hipGetLastError();
}

// Key parts: four where two stages of 64 keys leave room for a second
// workgroup on the CU (or nearly: D = 128 in fp32 takes 135 KB), fewer for
// wider rows.  Fewer parts mean longer waves: with two at D = 64 the 16-head,
// 777-row causal fp32 call took 38 us against 27, at D = 96 the 16/2-head,
// 1111-row bf16 call 51 against 37; with eight the 777-row call took 34 (each
// staged tile then serves half the columns).
template <typename TIN, typename TOUT, int DP>
hipError_t launch_k(const Problem &p, hipStream_t s) {
    return launch_t<TIN, TOUT, DP, DP <= 128 ? 4 : DP <= 160 ? 2 : 1>(p, s);
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
