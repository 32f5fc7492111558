// fa_decode.hip -- decode attention (one query row per head against a long
// key/value cache) on gfx950: split-KV partial kernel plus log-sum-exp merge.
//
// Decode has one query row per head (Sec. 4.1: the operands shrink to 1 x D),
// so the only parallelism inside one (batch, key/value head) is across the
// query heads of its group and along the key sequence.  The G query heads
// that share a key/value head are processed together as the 16 columns of a
// 16x16x32 MFMA (the GPU form of packing several heads into one vector
// register, Sec. 4.1.1, with the K/V row loaded once for the whole group,
// Sec. 4.1.2 (iv)); the key range is cut into splits, one workgroup per
// (batch, key/value head, 16-head query group, split), so that enough
// workgroups stream K/V from HBM to keep every CU busy.
//
// Inside a workgroup each of the 8 waves streams its own 32-key chunks
// (round robin over the split), carrying running max / sum / accumulator as
// in Alg. 1 (tile-wise; the running maximum only moves when a tile's maximum
// exceeds it by more than 8 in the log2 domain).  A chunk's K and V rows are
// loaded whole and staged in the wave's own LDS area, one chunk ahead of the
// arithmetic.  The waves' partial states are merged through LDS and the
// workgroup writes one (unnormalised accumulator, max, sum) triple per query
// head and split.  A second kernel merges the splits of each (batch, query
// head) by their log-sum-exp and applies the final 1/l normalisation; with one
// split the workgroup writes the result itself.  A sequence's own valid keys
// are spread evenly over the splits, so that short sequences of a batch occupy
// their workgroups no longer than they must.
//
// What bounds it: HBM for large caches (16 x 32/8 heads, 8192 keys, D = 128:
// 82 us for 537 MB, 6.5 TB/s against 6.9 for a plain read), and how evenly the
// last round of workgroups fills the chip (see decode_default_splits); for
// small ones the chain launch, lengths, keys, merge, second launch (7 us for
// 32/4 heads, 1537 keys, D = 64).  Loads two chunks ahead (144 and 244
// registers) and 16-wave workgroups at D = 64 gained nothing.
#include "fa_checks.h"
#include "fa_common.h"
#include "fa_internal.h"

namespace fa {
namespace {

constexpr int KPW = 32;        // keys per wave iteration
constexpr int QG = 16;         // query heads per MFMA column block
constexpr int NW = 8;          // waves per workgroup
constexpr float TAU = 8.0f;    // lazy-rescale threshold (log2 units)
constexpr int MIN_KEYS_PER_SPLIT = 256;
constexpr int CUS = 256;                 // compute units of the card
constexpr long long LONG_SPLIT = 4096 * 100;   // keys (hundredths) beyond which one workgroup fills a CU's share of HBM
constexpr int RANKED_KEYS = 512;         // keys per split from which an order by length pays
constexpr int MAX_ROUNDS = 8;            // most rounds of one workgroup per CU that splitting may make

struct DecodeArgs {
    const void *q, *k, *v;
    float *opart, *mpart, *lpart;   // workspace: [B*Hq*S*D], [B*Hq*S], [B*Hq*S]
    void *o;        // written directly when there is one split
    float *lse;
    int out_f32;    // o holds fp32 instead of the input type
    int Hq, Hkv, Nk;
    int G;          // query heads per key/value head
    Divisor S;      // splits
    Divisor nqg;    // 16-head query groups per key/value head
    Divisor nkv;    // key/value heads
    int B, ranked;  // ranked > 0: uneven sequences are taken by length, the first `ranked`
                    // longest first, the others shortest first
    float c;        // |scale| * log2(e)
    unsigned qsign; // sign flip of q for negative scale
    const int *seqlens;   // valid keys per batch element (NULL: Nk for all)
    const int *block_table;   // paged K/V: page of each key block (see Problem)
    Divisor page_size;
    int max_pages, num_pages;
};

template <int D> struct DSmem {
    static constexpr int KS = D + 8;             // K row stride (16-bit elements)
    static constexpr int VS = D + 16;            // V row stride (16-bit elements)
    static constexpr int WAVE = KPW * (KS + VS); // per-wave K and V staging
    static constexpr int MERGE_FLOATS = NW * QG * (D + 2);
    static constexpr int BYTES_STAGE = NW * WAVE * 2;
    static constexpr int BYTES = BYTES_STAGE > MERGE_FLOATS * 4 ? BYTES_STAGE : MERGE_FLOATS * 4;
};

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename TIN, int D, bool PAGED>
__global__ __launch_bounds__(64 * NW, 1) void decode_split_kernel(DecodeArgs a) {
    using S = typename TIN::scalar;
    using V8 = typename TIN::vec8;
    using SM = DSmem<D>;
    constexpr int KST = D / 32;          // QK^T contraction steps (K = 32)
    constexpr int DT = D / 16;           // output row tiles of 16
    constexpr int CPR = D / 8;           // 16-byte chunks per key row
    constexpr int RLOADS = KPW * CPR / 64;   // 16-byte row loads per lane per chunk (K and V each)
    constexpr bool IN_BF16 = __is_same(TIN, bf16_t);

    __shared__ __attribute__((aligned(16))) unsigned char smem[SM::BYTES];

    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = l & 15, lg = l >> 4;            // MFMA column (query) and k-group
    const int bid = blockIdx.x;
    const int u = a.S.div(bid), s = bid - u * a.S.d;
    const int u2 = a.nqg.div(u), qg = u - u2 * a.nqg.d;
    int b = a.nkv.div(u2), len = a.Nk;
    const int g = u2 - b * a.nkv.d;
    // Sequences of uneven length, in grids past one workgroup per CU: longest
    // first, so that the last round is short (64 x 32/8 heads, 512 to 4096 keys,
    // D = 128 119 -> 103 us; 40 of them, D = 64 39.4 -> 36.2); when all start at
    // once, one workgroup for every CU, the others shortest first.  Ranking
    // takes some 0.5 us: below 512 keys a split it is not done (13 x 32/8
    // heads, 1050 keys, D = 64, 4 splits 11.7 us against 12.3 with it)
    if (a.ranked > 0) {
        const Lengths lens(a.seqlens, a.B, l);
        if (lens.uneven()) b = lens.nth_longest(b < a.ranked ? b : a.B - 1 - (b - a.ranked));
        len = lens.of(b);
    } else if (a.seqlens) {
        len = a.seqlens[b];
    }
    const int G = a.G;
    // valid keys of this batch element (a cache of a.Nk rows per element), and
    // its split: the sequence's own keys, spread evenly in multiples of KPW
    const int Nk = __builtin_amdgcn_readfirstlane(min(max(len, 0), a.Nk));
    const unsigned whole = a.S.div(Nk), per = whole + (whole * a.S.d != (unsigned)Nk);   // ceil(Nk / S)
    const long long chunk = (per + (KPW - 1)) & ~(unsigned)(KPW - 1);
    const int k0 = (int)min(s * chunk, (long long)Nk);
    const int k1 = (int)min(k0 + chunk, (long long)Nk);

    // This lane's query head (MFMA column) and its Q operand.
    const int qh = qg * QG + lc;             // index inside the group
    const bool qvalid = qh < G;
    const int h = g * G + qh;
    V8 qf[KST];
    {
        const S *qp = reinterpret_cast<const S *>(a.q) + ((size_t)b * a.Hq + h) * D + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {
            uint4_t u = {0u, 0u, 0u, 0u};
            if (qvalid) u = ld16(qp + 32 * ks);
            u ^= a.qsign;
            qf[ks] = as_vec8<V8>(u);
        }
    }

    const size_t row_elems = (size_t)a.Hkv * D;                   // elements between keys
    const int row_bytes = (int)(row_elems * sizeof(S));
    const size_t head_off = ((size_t)b * a.Nk * a.Hkv + g) * D;   // key 0 of (b, g)

    unsigned short *kst = reinterpret_cast<unsigned short *>(smem) + w * SM::WAVE;
    unsigned short *vst = kst + KPW * SM::KS;
    const _Float16 *vsth = reinterpret_cast<const _Float16 *>(vst);
    // transpose-read lane offset: rows 4*lg + (lc / 4), columns 4 * (lc % 4)
    const int v_lane = (4 * lg + (lc >> 2)) * SM::VS + 4 * (lc & 3);

    float4_t oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt] = float4_t{};
    float m_run = -INFINITY, l_run = 0.f;

    // A chunk's K and V rows are loaded whole (64 lanes cover 64 / CPR
    // complete rows per instruction, the access pattern that streams from HBM
    // fastest) and staged in the wave's own LDS area: K as is (read back in
    // the MFMA operand layout), V as fp16 (read back transposed).  Loads go
    // through a buffer view that ends after the chunk's last key, so that keys
    // past it read as zeros without a branch, and each wait covers exactly the
    // chunk it needs.
    int off[RLOADS];
#pragma unroll
    for (int i = 0; i < RLOADS; ++i) off[i] = (l + 64 * i) / CPR * row_bytes + 16 * ((l + 64 * i) % CPR);
    const int nchunks = (k1 - k0 + KPW - 1) / KPW;
    uint4_t kr[RLOADS], vr[RLOADS];   // the next chunk's rows, in flight
    auto gload = [&](int ch) __attribute__((always_inline)) {
        // first key of the chunk (past the last chunk: an empty view)
        const int kb = k0 + ch * KPW;
        const int n = ch < nchunks ? min(k1 - kb, KPW) : 0;
        const int nrec = n > 0 ? (n - 1) * row_bytes + D * (int)sizeof(S) : 0;
        // its row, contiguous or through the block table (a chunk never
        // crosses a page: chunks start at multiples of 32 keys and pages hold
        // a multiple of 64; page numbers are clamped into the pool)
        size_t rbase = 0;
        if constexpr (PAGED) {
            if (n > 0) {
                const int pi = a.page_size.div(kb);
                const int page = min(max(a.block_table[(size_t)b * a.max_pages + pi], 0), a.num_pages - 1);
                rbase = ((size_t)page * a.page_size.d + (kb - pi * (int)a.page_size.d)) * row_elems + (size_t)g * D;
            }
        } else {
            rbase = head_off + (size_t)(n > 0 ? kb : 0) * row_elems;
        }
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<S *>(reinterpret_cast<const S *>(a.k)) + rbase, (short)0, nrec, 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<S *>(reinterpret_cast<const S *>(a.v)) + rbase, (short)0, nrec, 0x00020000);
        constexpr int NT = 2;   // read once: non-temporal
#pragma unroll
        for (int i = 0; i < RLOADS; ++i) {
            kr[i] = __builtin_bit_cast(uint4_t, __builtin_amdgcn_raw_buffer_load_b128(rk, off[i], 0, NT));
            vr[i] = __builtin_bit_cast(uint4_t, __builtin_amdgcn_raw_buffer_load_b128(rv, off[i], 0, NT));
        }
    };
    auto kvstore = [&]() {
#pragma unroll
        for (int i = 0; i < RLOADS; ++i) {
            const int c = l + 64 * i;
            const int key = c / CPR, cc = c % CPR;
            st16(kst + key * SM::KS + 8 * cc, kr[i]);
            st16(vst + key * SM::VS + 8 * cc, IN_BF16 ? bf16x8_to_f16x8(vr[i]) : vr[i]);
        }
    };

    gload(w);
    for (int ch = w; ch < nchunks; ch += NW) {
        const int kb = k0 + ch * KPW;
        kvstore();
        gload(ch + NW);
        wave_lds_fence();
        // ---- S^T = K Q^T: two 16-key halves, lane owns query lc, keys 4 lg + r
        float4_t s0 = float4_t{}, s1 = float4_t{};
        const unsigned short *kl = kst + lc * SM::KS + 8 * lg;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {
            s0 = mfma16(as_vec8<V8>(*reinterpret_cast<const uint4_t *>(kl + 32 * ks)), qf[ks], s0);
            s1 = mfma16(as_vec8<V8>(*reinterpret_cast<const uint4_t *>(kl + 16 * SM::KS + 32 * ks)),
                        qf[ks], s1);
        }
        const bool masked = kb + KPW > k1;
        if (masked) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s0[r] = (kb + 4 * lg + r < k1) ? s0[r] : -INFINITY;
                s1[r] = (kb + 16 + 4 * lg + r < k1) ? s1[r] : -INFINITY;
            }
        }
        float mx = max3(max3(s0[0], s0[1], s0[2]), max3(s0[3], s1[0], s1[1]), __builtin_fmaxf(s1[2], s1[3]));
        // (by row swaps: an exchange through LDS would also wait for the chunk's
        // other LDS reads; 32/4 heads, 1537 keys, D = 64 6.85 -> 6.66 us, 8 x 16/16,
        // 1200 keys 12.84 -> 12.6, nothing where HBM bounds)
        mx = pair_max(half_max(mx));
        const float m_tile = (mx == -INFINITY) ? -INFINITY : mx * a.c;
        const float m_new = __builtin_fmaxf(m_run, m_tile);
        const bool need = m_new > m_run + TAU;
        if (__builtin_amdgcn_ballot_w64(need)) {
            const float m_next = need ? m_new : m_run;
            const float alpha = need ? exp2_fast(m_run - m_next) : 1.f;
            m_run = m_next;
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[dt] *= alpha;
        }
        const float base = (m_run == -INFINITY) ? 0.f : m_run;
        float p[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = exp2_fast(__builtin_fmaf(s0[r], a.c, -base));
            p[4 + r] = exp2_fast(__builtin_fmaf(s1[r], a.c, -base));
        }
        if (masked) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = (s0[r] == -INFINITY) ? 0.f : p[r];
                p[4 + r] = (s1[r] == -INFINITY) ? 0.f : p[4 + r];
            }
        }
        l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        const half8_t pf = pack_f16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
        // ---- O^T += V^T P^T over the 32 keys (k-group lg: keys 4lg..+3, 16+4lg..+3)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const _Float16 *vp = vsth + v_lane + 16 * dt;
            half8_t va = cat_half8(lds_read_tr16(vp), lds_read_tr16(vp + 16 * SM::VS));
            oacc[dt] = mfma16(va, pf, oacc[dt]);
        }
        wave_lds_fence();   // operand reads of this chunk are done
    }

    // ---- merge the waves' partial states through LDS
    l_run = pair_sum(half_sum(l_run));
    __syncthreads();
    float *mf = reinterpret_cast<float *>(smem);     // [NW][QG][D + 2]
    float *mine = mf + (w * QG + lc) * (D + 2);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[16 * dt + 4 * lg + r] = oacc[dt][r];
    if (lg == 0) {
        mine[D] = m_run;
        mine[D + 1] = l_run;
    }
    __syncthreads();
    // the first 256 threads: query column tid / 16, 16 threads per query, D / 16 columns each
    const int mq = tid >> 4, part = tid & 15;
    const int mh = qg * QG + mq;
    if (mq < QG && mh < G) {
        float M = -INFINITY;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) M = __builtin_fmaxf(M, mf[(ww * QG + mq) * (D + 2) + D]);
        float wgt[NW];
        float L = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const float mw = mf[(ww * QG + mq) * (D + 2) + D];
            wgt[ww] = (mw == -INFINITY) ? 0.f : exp2_fast(mw - M);
            L += wgt[ww] * mf[(ww * QG + mq) * (D + 2) + D + 1];
        }
        const size_t bh = (size_t)b * a.Hq + g * G + mh;
        const bool direct = a.S.d == 1;   // one split: the result itself
        const size_t slot = bh * a.S.d + s;   // (bh itself with one split)
        // as the merge does: a sequence with no valid key (per-sequence lengths),
        // or whose scores are not numbers, gives 0 and -inf
        const bool some = !direct || L > 0.f;
        const float inv = direct ? 1.f / L : 1.f;
        float acc[D / 16];
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
            acc[j] = 0.f;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) acc[j] += wgt[ww] * mf[(ww * QG + mq) * (D + 2) + part + 16 * j];
            acc[j] = some ? acc[j] * inv : 0.f;
        }
        if (!direct || a.out_f32) {
            float *op = (direct ? reinterpret_cast<float *>(a.o) : a.opart) + slot * D + part;
#pragma unroll
            for (int j = 0; j < D / 16; ++j) op[16 * j] = acc[j];
        } else {
            S *op = reinterpret_cast<S *>(a.o) + slot * D + part;
#pragma unroll
            for (int j = 0; j < D / 16; ++j) op[16 * j] = from_f32<S>(acc[j]);
        }
        if (part == 0) {
            if (!direct) {
                a.mpart[slot] = M;
                a.lpart[slot] = L;
            } else if (a.lse) {
                a.lse[bh] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
            }
        }
    }
}

// Merge of the S partial results of one (batch, query head): lse-weighted sum
// of the unnormalised accumulators, final normalisation, log-sum-exp output.
// Splits are taken in groups of 16 whose loads are all issued together (one
// memory round trip per group; the usual split counts fit in one group); the
// running maximum moves once per group.  Every thread of the block handles
// one output column and forms the same maximum and sum.
template <typename TOUT, int D>
__global__ __launch_bounds__(D) void decode_combine_kernel(const float *__restrict__ opart,
                                                          const float *__restrict__ mpart,
                                                          const float *__restrict__ lpart,
                                                          void *o, float *lse, int S) {
    constexpr int CH = 16;
    const int bh = blockIdx.x, t = threadIdx.x;
    const float *mp = mpart + (size_t)bh * S;
    const float *lp = lpart + (size_t)bh * S;
    const float *op = opart + (size_t)bh * S * D + t;
    float M = -INFINITY, L = 0.f, acc = 0.f;
    for (int s0 = 0; s0 < S; s0 += CH) {
        float mv[CH], lv[CH], ov[CH];
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            mv[j] = -INFINITY;
            lv[j] = 0.f;
            ov[j] = 0.f;
            if (s0 + j < S) {
                mv[j] = mp[s0 + j];
                lv[j] = lp[s0 + j];
                ov[j] = op[(size_t)(s0 + j) * D];
            }
        }
        float Mc = M;
#pragma unroll
        for (int j = 0; j < CH; ++j) Mc = __builtin_fmaxf(Mc, mv[j]);
        const float alpha = (M == -INFINITY) ? 0.f : exp2_fast(M - Mc);
        L *= alpha;
        acc *= alpha;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const float w = (mv[j] == -INFINITY) ? 0.f : exp2_fast(mv[j] - Mc);
            L = __builtin_fmaf(w, lv[j], L);
            acc = __builtin_fmaf(w, ov[j], acc);
        }
        M = Mc;
    }
    // a sequence with no valid key (per-sequence lengths), or whose scores are not
    // numbers, gives 0 and -inf
    reinterpret_cast<TOUT *>(o)[(size_t)bh * D + t] = from_f32<TOUT>(L > 0.f ? acc / L : 0.f);
    if (lse && t == 0) lse[bh] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
}

// Workgroups that the chip holds at once.
constexpr long long resident(int D) { return D == 64 ? 2 * CUS : CUS; }

template <typename TIN, typename TOUT, int D>
hipError_t launch_t(const Problem &p, int S, void *ws, hipStream_t stream) {
    DecodeArgs a;
    a.q = p.q; a.k = p.k; a.v = p.v;
    const size_t nslot = (size_t)p.B * p.Hq * S;
    a.opart = reinterpret_cast<float *>(ws);
    a.mpart = a.opart + nslot * D;
    a.lpart = a.mpart + nslot;
    a.o = p.o;
    a.lse = p.lse;
    a.out_f32 = p.out == FA_F32;
    a.Hq = p.Hq; a.Hkv = p.Hkv; a.Nk = p.Nk;
    const int G = p.Hq / p.Hkv, nqg = (G + QG - 1) / QG;
    a.G = G;
    a.S = Divisor(S);
    a.nqg = Divisor(nqg);
    a.nkv = Divisor(p.Hkv);
    a.c = __builtin_fabsf(p.scale) * kLog2e;
    a.qsign = p.scale < 0.f ? 0x80008000u : 0u;
    a.seqlens = p.seqlens;
    a.block_table = p.block_table;
    a.page_size = Divisor(p.block_table ? p.page_size : 1);
    a.max_pages = p.max_pages;
    a.num_pages = p.num_pages;
    const long long nblocks = (long long)p.B * p.Hkv * nqg * S;
    if (nblocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.B = p.B;
    a.ranked = 0;
    if (p.seqlens && p.B > 1 && p.B <= kMaxRanked && nblocks > CUS && p.Nk >= RANKED_KEYS * (long long)S) {
        const long long per_seq = nblocks / p.B;
        a.ranked = nblocks <= resident(D) ? (int)((CUS + per_seq - 1) / per_seq) : p.B;
    }
    if (p.block_table)
        hipLaunchKernelGGL((decode_split_kernel<TIN, D, true>), dim3((unsigned)nblocks), dim3(64 * NW), 0,
                           stream, a);
    else
        hipLaunchKernelGGL((decode_split_kernel<TIN, D, false>), dim3((unsigned)nblocks), dim3(64 * NW), 0,
                           stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    hipLaunchKernelGGL((decode_combine_kernel<TOUT, D>), dim3((unsigned)(p.B * p.Hq)), dim3(D), 0,
                       stream, a.opart, a.mpart, a.lpart, p.o, p.lse, S);
    return hipGetLastError();
}

template <typename TIN, typename TOUT>
hipError_t launch_d(const Problem &p, int S, void *ws, hipStream_t s) {
    return p.D == 64 ? launch_t<TIN, TOUT, 64>(p, S, ws, s) : launch_t<TIN, TOUT, 128>(p, S, ws, s);
}

}  // namespace

bool decode_supported(int Nq, int Hkv, int D, fa_dtype_t in) {
    return Nq == 1 && (D == 64 || D == 128) && (in == FA_F16 || in == FA_BF16) && tile_fits(Hkv, D, KPW);
}

// Split count.  A call has U (batch, key/value head, query group) units and
// runs U S workgroups, as many at once as the chip holds: one per CU at
// D = 128 (143 KB of LDS), two at D = 64.  What counts is that the last round
// is full: 12 units of 2 heads at 6144 keys, D = 128, take 23.6 us with 11
// splits (264 workgroups on 256 CUs) and 18.8 with 10; 9 x 8 at 8839 keys,
// D = 64: 47.2 with 4 (288), 31.5 with 7 (504).  So the candidates are the
// largest counts that fill j rounds of 256, j = 1 .. 8, and one split, and the
// cheapest is taken by a model in keys: a round costs its keys per split (half
// where it leaves a CU one workgroup instead of two: 52 % below 4096 keys, 50
// above, where one streams as fast as two) plus some 250 for the workgroup's
// start and end; more than one split adds the merge kernel (some
// 200) and its loads (4 a split).  The model picks a count within 6 % of the
// best of those measured (a dozen shapes from 24 to 720 units, 512 to 32768
// keys).  At least 256 keys per split (one chunk for each wave).
// Lengths of their own are not known here, and a call with equal ones has the
// bits of one without, so the count is the same.  Over 640 such calls (lengths
// down to an eighth of the cache) it gains 12 % against ceil(256 / U) splits;
// seven are slower by more than 3 %, where D = 128 leaves 176 to 224 workgroups
// and the longest sequences then decide (12 x 32/8, 1684 to 282 keys 15.9 ->
// 18.3; 14 x 32/8, 4067 to 977 31.2 -> 35.7).  Over 1280 calls without lengths
// none is.
// CUS is the whole card's, not the device's: the count must be the same in
// fa_workspace_bytes, which asks no device, and sums must not go by its mode.
int decode_default_splits(int B, int Hq, int Hkv, int Nk, int D) {
    const int G = Hq / Hkv;
    const long long units = (long long)B * Hkv * ((G + QG - 1) / QG);
    long long cap = (Nk + (long long)MIN_KEYS_PER_SPLIT - 1) / MIN_KEYS_PER_SPLIT;
    if (cap > FA_MAX_SPLITS) cap = FA_MAX_SPLITS;
    const long long slots = resident(D);
    long long best = 1, least = 0;
    for (int j = 0; j <= MAX_ROUNDS; ++j) {
        long long S = j == 0 ? 1 : j * (long long)CUS / units;
        if (S > cap) S = cap;
        if (S < 1 || (j > 0 && S == 1)) continue;
        const long long W = units * S, full = W / slots, rest = W % slots;
        const long long keys = 100 * (long long)Nk / S;   // hundredths of a key, as the costs
        long long cost = full * (keys + 25000);
        if (rest > 0) cost += (slots > CUS && rest <= CUS ? keys * (keys > LONG_SPLIT ? 50 : 52) / 100 : keys) + 25000;
        if (S > 1) cost += 20000 + 400 * S;
        if (j == 0 || cost < least) {
            least = cost;
            best = S;
        }
        if (j > 0 && S == cap) break;
    }
    return (int)best;
}

// The most splits of any cache of up to Nk keys.  The count grows with the cache
// (a candidate of more splits has the larger constant part, so one that is
// cheaper at some length stays so), but for the 50 % of long splits: where
// they can apply, the largest candidate.
int decode_most_splits(int B, int Hq, int Hkv, int Nk, int D) {
    if (resident(D) == CUS || Nk <= LONG_SPLIT / 100) return decode_default_splits(B, Hq, Hkv, Nk, D);
    const long long units = (long long)B * Hkv * ((Hq / Hkv + QG - 1) / QG);
    const long long cap = (Nk + (long long)MIN_KEYS_PER_SPLIT - 1) / MIN_KEYS_PER_SPLIT;
    long long S = MAX_ROUNDS * (long long)CUS / units;
    if (S > cap) S = cap;
    if (S > FA_MAX_SPLITS) S = FA_MAX_SPLITS;
    return S < 1 ? 1 : (int)S;
}

size_t decode_workspace_bytes(int B, int Hq, int D, int splits) {
    return (size_t)B * Hq * splits * (size_t)(D + 2) * sizeof(float);
}

hipError_t launch_decode(const Problem &p, int splits, void *ws, hipStream_t stream) {
    if (p.in == FA_F16)
        return p.out == FA_F32 ? launch_d<f16_t, float>(p, splits, ws, stream)
                               : launch_d<f16_t, _Float16>(p, splits, ws, stream);
    return p.out == FA_F32 ? launch_d<bf16_t, float>(p, splits, ws, stream)
                           : launch_d<bf16_t, __bf16>(p, splits, ws, stream);
}

}  // namespace fa
