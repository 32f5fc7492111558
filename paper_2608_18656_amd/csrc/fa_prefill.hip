// fa_prefill.hip -- prefill attention forward on gfx950 matrix cores.
//
// Work split.  A workgroup owns NS (query head, 32-row block) slots that read
// the same key/value head: four, or eight (1 and 2 exist for the packing
// ablation).
// When the group size G = Hq/Hkv allows, up to four of the slots
// are query heads of one key/value group at the same rows -- the GPU form of
// the inter-head packing of Sec. 4.1.1 and the GQA reuse of Sec. 4.1.2 (iv):
// every K/V tile staged in LDS serves all slots of the workgroup, and slots
// of different heads share one causal extent; the other slots are
// consecutive row blocks.  Every wave handles 32 rows and 32 keys of each
// tile.  At D = 64 a slot has two waves (64-key tiles; wave kh takes keys
// 32 kh .. 32 kh + 31) whose states are merged through LDS at the end; at
// D = 128 one wave (32-key tiles).
//
// Per wave and tile, the blocked streaming softmax (Alg. 2 state carry over
// the per-key recurrence of Alg. 1):
//   S^T = K Q^T        32x32x16 MFMA; A = 32 K rows from LDS, B = the wave's
//                      32 query rows, kept in registers for the whole kernel
//   softmax            scores stay in the MFMA result registers; lane l owns
//                      query row l%32 (a row maximum needs one exchange with
//                      lane l^32); scale and log2(e) fold into one
//                      multiply-add ahead of exp2; weights packed to fp16
//   O^T += V^T P^T     32x32x16 fp16 MFMA; P straight from the score registers,
//                      V^T operands read from the row-major V tile with the
//                      transposing LDS read
// Staging.  K tiles, and fp16 V tiles, go from memory to LDS directly (no
// registers, no LDS store instructions); bf16 V passes through registers to
// become fp16.  The transposing read (8 bytes a lane) delivers 249 bytes per
// clock and CU when the four rows that 32 lanes read lie in different quarters
// of the 64 banks, as much as the plain 16-byte read (255), and 64 to 128
// when they do not; LDS stores take 62 (4 bytes a lane) to 79 (16 bytes).  So
// the tiles are laid out for the reads, by swizzling the addresses that a
// lane loads from, and nothing is transposed in the copy.  Against a copy
// through registers that wrote V transposed with 4-byte stores, timed in turn:
// D = 128, 2 x 32/8 heads, 4096 rows, fp16, causal: 299 -> 276 us; D = 64,
// 16/1 heads, 16384 rows, fp16: 597 -> 581 us; 32/8 heads, 2048 rows, bf16:
// 30.3 -> 28.9 us.
// What bounds it.  Large grids run at the card's power limit (1.85 to 2.0 GHz;
// with zeros for data, at 2.35 GHz, D = 128 takes 184 us and the 16384-row
// call 447 us), so what saves energy per tile saves time.  At full clock a
// wave's 32 x 32 block at D = 64 costs about 440 of its SIMD's cycles from
// registers alone: 256 of MFMA, and 35 vector instructions of 4 cycles and 16
// exponentials of 8, which overlap with them only in part.
// The exponent base only moves when a tile's weights against the current base
// grow too large (see the softmax step below), so the accumulator rescale is
// skipped on most tiles; sum and accumulator always share the base, so the
// result is unchanged.
// A wave's steps run in order; latency is hidden by the other waves of the
// SIMD (four-slot layouts: two 8-wave workgroups per CU at D = 64, four waves
// per SIMD within 128 VGPRs; three 4-wave ones at D = 128, three waves per
// SIMD within 168 VGPRs; their barriers are independent).  With three LDS
// stages the tile two steps ahead is loaded during a step.  Matrix
// instructions are issued at raised wave priority.
// Masked scores are -inf and give exactly 0 (the exponent factor is kept
// strictly positive, also for scale = 0).  Keys past the end read as zero
// (buffer loads with the tensor's extent as the range) and are masked.
// Normalisation happens once, after the last tile.
#include <atomic>
#include <type_traits>

#include "fa_checks.h"
#include "fa_common.h"
#include "fa_internal.h"

namespace fa {
namespace {

constexpr int WR = 32;        // query rows per slot
constexpr int NSLOT = 4;      // slots per workgroup where nothing speaks for another number
constexpr int RANKED_KEYS = 512, RANKED_KEYS_EACH = 40;   // cache from which an order by length pays: keys, keys a sequence
constexpr float kMaxLaneSum = 4096.0f;   // largest 16-weight lane sum kept without a rescale

struct PrefillArgs {
    const void *q, *k, *v;
    void *o;
    float *lse;
    int B, Hq, Hkv, Nq, Nk;
    float c;          // max(|scale|, tiny) * log2(e), > 0
    unsigned qsign;   // 0x80008000 to negate q (scale < 0), else 0
    int G;            // query heads per key/value head
    int HW, lgHW;     // query heads per workgroup (1, 2, 4 or 8) and its logarithm
    int nmb;          // row blocks of 32 * (slots / HW) rows
    Divisor per_mb;   // workgroups per row block: B * Hkv * (G / HW)
    Divisor nhg;      // head groups per key/value head (G / HW)
    Divisor nkv;      // key/value heads
    int ranked;       // > 0: uneven sequences are taken by length, the first `ranked` of their row
                      // blocks longest first, the others shortest first
    Divisor per_seq;      // workgroups per sequence and row block: Hkv * (G / HW)
    Divisor row_blocks;   // nmb
    int first;        // row blocks taken longest first, the others shortest first
    const int *seqlens;   // valid keys per batch element (NULL: Nk for all)
    const int *block_table;   // paged K/V: page of each key block (see Problem)
    int page_size, max_pages, num_pages;
};

// Tile shape per head size.  Every wave handles 32 query rows and 32 keys of
// a tile.  D = 64: two waves per slot (64-key tiles, key halves merged at the
// end), 8-wave workgroups of at most 128 VGPRs, two per CU (four waves per
// SIMD).  D = 128: the accumulator (64 VGPRs) and Q (32) leave no room for
// that, so one wave per slot (32-key tiles) and 4-wave workgroups, three per
// CU (three waves per SIMD, from independent workgroups; operands are read
// from LDS in small groups to fit 168 VGPRs).  Three LDS stages (two for
// one- and two-slot workgroups).
// NS, the slots per workgroup (all reading one key/value head, each staged
// tile serving all of them), is 4, or 8 for some large grids (eight_slots); 1
// and 2 exist for the packing ablation (fewer slots stage more per thread, so
// they hold fewer waves per SIMD).
template <int D, int NS = NSLOT> struct Cfg {
    static constexpr int NQ = D == 64 ? 2 : 1;       // waves per slot
    // waves per SIMD (what the registers allow; fewer slots stage more per thread)
    static constexpr int WPE = D == 64 ? (NS >= 4 ? 4 : NS == 2 ? 3 : 2) : (NS >= 4 ? 3 : NS == 2 ? 2 : 1);
    static constexpr int NWG = NS * NQ;              // waves per workgroup
    static constexpr int WPC = NWG >= 4 * WPE ? 1 : 4 * WPE / NWG;   // workgroups per CU (registers)
    static constexpr int BC = 32 * NQ;               // keys per tile
    static constexpr int NT = 64 * NWG;              // threads per workgroup
    static constexpr int NSTAGE = NS >= 4 ? 3 : 2;   // LDS tile stages (small workgroups: two, for room on the CU)
    static constexpr int AHEAD = NSTAGE - 1;         // a tile is loaded this many steps ahead
    static constexpr int KSZ = BC * D;               // K tile: BC rows of D elements, chunks swizzled
    static constexpr int VSZ = BC * D;               // V tile: the same shape
    static constexpr int STAGE = KSZ + VSZ;
    static constexpr int MERGE = NQ > 1 ? NS * (NQ / 2) * ((D / 32) * 16 + 2) * 64 : 0;  // floats
    static constexpr int WORDS = (NSTAGE * STAGE) > (2 * MERGE) ? NSTAGE * STAGE : 2 * MERGE;
    // Staging split: a tile is eight 1 KiB pieces of K and eight of V, 64
    // consecutive 16-byte chunks each.  A wave takes NP pieces of both, or in
    // a 16-wave workgroup one piece of one (waves 0 .. 7 V, 8 .. 15 K).
    static constexpr int PIECES = KSZ * 2 / 1024;
    static constexpr bool SPLIT = NWG > PIECES;
    static constexpr int NP = SPLIT ? 1 : PIECES / NWG;
    static_assert(PIECES == 8 && (SPLIT ? NWG == 2 * PIECES : PIECES % NWG == 0), "staging split");
};

template <typename TIN, typename TOUT, int D, int NS, bool CAUSAL, bool PAGED>
__global__ __launch_bounds__((Cfg<D, NS>::NT)) __attribute__((amdgpu_waves_per_eu((Cfg<D, NS>::WPE), (Cfg<D, NS>::WPE)))) void prefill_kernel(PrefillArgs a) {
    using S = typename TIN::scalar;
    using V8 = typename TIN::vec8;
    using SM = Cfg<D, NS>;
    constexpr int NSLOT = NS;
    constexpr int NQ = SM::NQ, BC = SM::BC, NT = SM::NT, NSTAGE = SM::NSTAGE;
    constexpr int KSTEPS = D / 16;          // QK^T contraction steps
    constexpr int DT = D / 32;              // output column tiles
    constexpr int CPR = D / 8;              // 16-byte chunks per row
    constexpr bool IN_BF16 = __is_same(TIN, bf16_t);

    __shared__ __attribute__((aligned(1024))) unsigned short smem[SM::WORDS];

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63, lq = l & 31, lh = l >> 5;
    const int kh = w / NSLOT, slot = w % NSLOT;   // kh: the wave's 32 keys of a tile
    const int RB = NSLOT >> a.lgHW;
    const int bid = blockIdx.x;
    // Row block of this workgroup.  Latest rows (most keys) first, so that
    // the short causal blocks fill the tail; when the whole grid is resident
    // at once, only one workgroup for every CU in that order and the others
    // shortest first, so that workgroups sharing a CU carry about the same
    // total work (one per CU rather than half of the grid, us: 32/8 heads,
    // D = 64, 1200 rows 21.9 -> 20.1; D = 128, 1100 rows 30.6 -> 29.0, 3000 rows
    // 93.5 -> 89.7).  With lengths of their own that differ, sequences are
    // taken by length and rows within them, in that same pattern: in the order
    // of the batch two workgroups of one sequence share a CU, and the CUs of the
    // long ones finish last (4 x 32/8 heads, 512 rows, 4096 to 1024 keys, D = 64
    // 68 -> 54; 16 such sequences 250 -> 210; 6 of 1024 rows, D = 128 288 -> 250).
    // About equal ones stay in the order of the batch, where workgroups that
    // share a CU share its L1 as well (4 x 4096 keys 83 against 86 by rank), and
    // so do those of short caches, where ranking (0.5 us, 1.5 for 40 and more
    // sequences, ahead of the first load) costs more than it gives (in the
    // order of the batch, which is by length, against ranked, D = 64: 43 x 8/8
    // heads, 32 rows, 256 keys 9.5 / 11.0, 512 12.6 / 13.8, 1024 17.6 / 18.6, but
    // in a random one 21.0 / 18.7; 12 x 32/4, 128 rows, 256 keys 11.9 / 12.1,
    // 512 14.8 / 14.1).  Over 110 batches of 512 to 6000 keys, with 20 to 40
    // keys a sequence, ranking costs 5 % where they come by length and gives 2 in
    // a random order; from 40 on it gives 1 and 5.
    const int q_ = a.per_mb.div(bid);
    int mb = q_ < a.first ? a.nmb - 1 - q_ : q_ - a.first;
    int rest = bid - q_ * a.per_mb.d;
    int b = -1, len = a.Nk;
    if (a.ranked > 0) {
        const Lengths lens(a.seqlens, a.B, l);
        if (lens.uneven()) {
            const int u = a.per_seq.div(bid);
            rest = bid - u * a.per_seq.d;
            const int j = u < a.ranked ? u : a.B * a.nmb - 1 - (u - a.ranked), r = a.row_blocks.div(j);
            mb = a.nmb - 1 - (j - r * a.nmb);
            b = lens.nth_longest(r);
        }
        if (b < 0) b = a.nkv.div(a.nhg.div(rest));
        len = lens.of(b);
    }
    const int bg = a.nhg.div(rest), hg = rest - bg * a.nhg.d;
    const int b0 = a.nkv.div(bg), g = bg - b0 * a.nkv.d;
    if (a.ranked == 0) {
        b = b0;
        if (a.seqlens) len = a.seqlens[b];
    }
    const int G = a.G;
    const int hs = slot & (a.HW - 1), rs = slot >> a.lgHW;
    const int h = g * G + hg * a.HW + hs;
    const int row0_wg = mb * (WR * RB);
    const int row0 = row0_wg + rs * WR;
    const int qi = row0 + lq;
    const int Nq = a.Nq;
    // Valid keys of this batch element: with per-sequence lengths the K/V
    // tensors hold a.Nk rows per batch element of which the first seqlens[b]
    // are valid, and the queries are the sequence's last Nq positions.
    const int Nk = __builtin_amdgcn_readfirstlane(min(max(len, 0), a.Nk));
    const int off = Nk - Nq;

    // Key extents: workgroup, this slot, and keys every row of the slot sees.
    const int last_wg = min(row0_wg + WR * RB, Nq) - 1;
    const int kend_wg = CAUSAL ? min(Nk, last_wg + off + 1) : Nk;
    const bool live = row0 < Nq;
    const int kfree_w = CAUSAL ? min(Nk, row0 + off + 1) : Nk;
    const int ntiles = (kend_wg + BC - 1) / BC;

    // Q rows of this lane (B operand of S^T = K Q^T).
    V8 qf[KSTEPS];
    {
        const int qrow = min(qi, Nq - 1);
        const S *qp = reinterpret_cast<const S *>(a.q) +
                      ((size_t)((size_t)b * Nq + qrow) * a.Hq + h) * D + 8 * lh;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            uint4_t u = ld16(qp + 16 * ks);
            u ^= a.qsign;
            qf[ks] = as_vec8<V8>(u);
        }
    }

    // Tile staging.  K, and fp16 V, go from memory to LDS directly (no
    // registers, no store instructions); bf16 V passes through registers,
    // where it becomes fp16.  A tile's rows lie in LDS without padding, row r's
    // 16-byte chunk c at chunk position c ^ kswz(r) (K) or c ^ vswz(r) (V), so
    // that 16 lanes reading one K chunk of 16 rows, and 32 lanes reading four
    // V rows' 64-byte segments, meet all 64 banks.  A lane's place in LDS is
    // fixed by the load (64 consecutive chunks per instruction), so the swizzle
    // is applied to the address it loads from.  Loads are buffer loads: the
    // tile's first key row is the (scalar) base and each lane keeps a fixed
    // byte offset; chunks past the end of the view become zeros.
    constexpr int NP = SM::NP;
    const bool dok = !SM::SPLIT || w >= SM::PIECES, dov = !SM::SPLIT || w < SM::PIECES;   // wave-uniform
    const size_t row_elems = (size_t)a.Hkv * D;      // elements between consecutive keys
    const int row_bytes = (int)(row_elems * sizeof(S));
    auto kswz = [](int r) { return D == 64 ? (r >> 1) & 7 : r & 15; };
    auto vswz = [](int r) { return D == 64 ? ((r >> 1) & 1) << 2 : (r & 3) << 2; };
    const int piece = SM::SPLIT ? w % SM::PIECES : w;    // first piece; the next ones NT / 64 further
    int koff[NP], voff[NP];                              // tile-relative byte offsets
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int q = 64 * (piece + (NT / 64) * j) + l, r = q / CPR, c = q % CPR;
        koff[j] = r * row_bytes + 16 * (c ^ kswz(r));
        voff[j] = r * row_bytes + 16 * (c ^ vswz(r));
    }
    typedef uint4_t vregs_t[IN_BF16 ? NP : 1];
    vregs_t vr;   // bf16: the next tile's V chunks, in flight during a step
    // Scalar state of the next tile to load: the address of its first key row
    // in K and V, which advances by one tile per load, and its number.  The
    // buffer view of a tile ends after its last valid key (keys past it read
    // as zero): a full tile's extent for the first Nk / BC tiles, then that of
    // the remaining keys, if any (one tile's extent fits 31 bits: tile_fits).
    const size_t head0 = ((size_t)b * a.Nk * a.Hkv + g) * D;
    const S *ktile = reinterpret_cast<const S *>(a.k) + (PAGED ? 0 : head0);
    const S *vtile = reinterpret_cast<const S *>(a.v) + (PAGED ? 0 : head0);
    const int tile_bytes = (BC - 1) * row_bytes + D * (int)sizeof(S);
    const int full_tiles = Nk / BC;
    const int last_bytes = Nk % BC ? (Nk % BC - 1) * row_bytes + D * (int)sizeof(S) : 0;
    int tload = 0;
    // paged K/V: the pool of pages, at head g.  Tiles are loaded in order
    // and a page holds a whole number of tiles, so the page index and the
    // offset inside the page advance without a division.  The wave holds 64
    // table entries, one per lane, and the next 64, read with vector loads
    // through a view of this sequence's row of the table (entries past the row
    // read as zero): no scalar load (whose counter the LDS reads share) is in
    // flight during a step, and no wait for an entry stands between the loads
    // of two tiles, where it would wait for the tiles as well (with the entry
    // of the following page loaded alone, 5 x 32/4 heads, 61 rows, 7680 keys,
    // D = 64, pages of 64 took 115 us against 78 for contiguous keys).
    const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int *>(PAGED ? a.block_table + (size_t)b * a.max_pages : nullptr), (short)0,
        PAGED ? a.max_pages * 4 : 0, 0x00020000);
    const size_t page_elems = (size_t)a.page_size * row_elems;
    int pidx = 0, poff = 0;   // page index and key offset of the next tile
    int tcur = 0, tnx = 0;    // lane i: table entries of pages 64 (pidx / 64) + i and 64 further
    if constexpr (PAGED) {
        tcur = __builtin_amdgcn_raw_buffer_load_b32(trs, 4 * l, 0, 0);
        tnx = __builtin_amdgcn_raw_buffer_load_b32(trs, 4 * (64 + l), 0, 0);
    }
    const unsigned lds0 = lds_address(smem);
    // the next tile (they are loaded in order) into stage `stage`; bf16 V into vr
    auto gload_to = [&](vregs_t &vr, int stage) __attribute__((always_inline)) {
        if constexpr (PAGED) {
            // the tile's rows sit in one page (pages hold a multiple of 64
            // keys, tiles start at multiples of BC): at the start of a page
            // the address comes from the table (page numbers clamped into the
            // pool), within it the address advances by one tile per load
            if (poff == 0) {
                if (pidx > 0 && pidx % 64 == 0) {
                    tcur = tnx;
                    tnx = __builtin_amdgcn_raw_buffer_load_b32(trs, 4 * (pidx + 64 + l), 0, 0);
                }
                const int page = min(max(__builtin_amdgcn_readlane(tcur, pidx % 64), 0), a.num_pages - 1);
                const size_t t = (size_t)g * D + (size_t)page * page_elems;
                ktile = reinterpret_cast<const S *>(a.k) + t;
                vtile = reinterpret_cast<const S *>(a.v) + t;
            }
        }
        const int nrec = tload < full_tiles ? tile_bytes : last_bytes;
        ++tload;
        const unsigned dst = lds0 + stage * (2 * SM::STAGE) + 1024 * piece;
        if (dok) {
#pragma unroll
            for (int j = 0; j < NP; ++j)
                load_lds16(ktile, nrec, dst + 1024 * (NT / 64) * j, koff[j]);
        }
        if (dov) {
            const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<S *>(vtile), (short)0, nrec, 0x00020000);
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                if constexpr (IN_BF16)
                    vr[j] = __builtin_bit_cast(uint4_t, __builtin_amdgcn_raw_buffer_load_b128(rv, voff[j], 0, 0));
                else
                    load_lds16(vtile, nrec, dst + 2 * SM::KSZ + 1024 * (NT / 64) * j, voff[j]);
            }
        }
        ktile += BC * (size_t)row_elems;
        vtile += BC * (size_t)row_elems;
        if constexpr (PAGED) {
            poff += BC;
            const bool cross = poff == a.page_size;   // wave-uniform
            poff = cross ? 0 : poff;
            pidx += cross ? 1 : 0;
        }
    };
    // bf16 V of a loaded tile, as fp16, into its stage
    auto vstore_from = [&](const vregs_t &vr, unsigned short *stage) __attribute__((always_inline)) {
        if constexpr (IN_BF16) {
            if (dov) {
#pragma unroll
                for (int j = 0; j < NP; ++j)
                    st16(stage + SM::KSZ + 512 * (piece + (NT / 64) * j) + 8 * l, bf16x8_to_f16x8(vr[j]));
            }
        }
    };

    float16_t oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[dt] = float16_t{};
    float m_run = -INFINITY;   // exponent base (log2 domain), same in lanes l and l^32
    float l_run = 0.f;         // this lane's part of the row sum
    float nbase = 0.f;         // -m_run, or 0 while the row has no base
    float lim = -INFINITY;     // largest lane sum kept without a rescale; below any sum while the row has no base

    // LDS offsets (elements) of the lane's operands.  K: chunk 2 kk + lh of row
    // 32 kh + lq.  V: the transposing read gives a lane four keys of one column;
    // lane i of each 16 addresses row i / 4 of four, columns 4 (i % 4) .. + 3 of
    // 16, and the group of 16 picks the column half; k-step j takes keys 16 j +
    // 4 lh .. + 3 and 16 j + 8 + 4 lh .. + 3, the order of the weights.
    const int k_row = (32 * kh + lq) * D, k_sw = 8 * (lh ^ kswz(lq));
    auto kat = [&](const unsigned short *stage, int kk) {
        return as_vec8<V8>(*reinterpret_cast<const uint4_t *>(stage + k_row + ((16 * kk) ^ k_sw)));
    };
    const int v_j = l & 15;
    const int v_row = SM::KSZ + (32 * kh + 4 * lh + (v_j >> 2)) * D + 16 * ((l >> 4) & 1) + 4 * (v_j & 3);
    const int v_sw = 8 * vswz(v_j >> 2);
    auto vat = [&](const unsigned short *stage, int dt, int j) {
        const _Float16 *p = reinterpret_cast<const _Float16 *>(stage) + v_row + ((32 * dt) ^ v_sw) + 16 * D * j;
        return cat_half8(lds_read_tr16(p), lds_read_tr16(p + 8 * D));
    };
    auto stage_at = [&](int r) { return smem + r * SM::STAGE; };

    // K operands of this wave's 32 keys of the tile held in `stage`
    auto kread = [&](const unsigned short *stage, V8 (&ka)[KSTEPS]) {
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
            ka[kk] = kat(stage, kk);
    };
    // S^T = K Q^T.  Matrix instructions are issued at raised wave priority:
    // the SIMD then starts a wave's next MFMA as soon as the matrix core is
    // free and fills the gaps with the other waves' vector work.
    auto qk = [&](const V8 (&ka)[KSTEPS]) {
        float16_t s = float16_t{};
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) s = mfma32(ka[kk], qf[kk], s);
        __builtin_amdgcn_s_setprio(0);
        return s;
    };
    auto scores = [&](const unsigned short *stage) {
        V8 ka[KSTEPS];
        kread(stage, ka);
        return qk(ka);
    };

    // V^T operands of one tile for this wave (k-step order: dt, j)
    auto vread = [&](const unsigned short *stage, half8_t (&va)[KSTEPS]) {
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
            va[kk] = vat(stage, kk >> 1, kk & 1);
    };
    // O^T += V^T P^T with the weights of one tile (k-step j = keys 16 j .. 16 j
    // + 15 of the wave's half)
    auto pv = [&](const half8_t &p0, const half8_t &p1, const half8_t (&va)[KSTEPS]) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            oacc[dt] = mfma32(va[2 * dt], p0, oacc[dt]);
            oacc[dt] = mfma32(va[2 * dt + 1], p1, oacc[dt]);
        }
        __builtin_amdgcn_s_setprio(0);
    };

    // Grouped operand reads for D = 128: two k-steps per group, the next
    // group read from LDS while the current one multiplies, so that at most
    // four operand words are live instead of one per k-step (this keeps the
    // kernel within the 168 VGPRs of three waves per SIMD).
    auto scores_jit = [&](const unsigned short *stage) {
        float16_t s = float16_t{};
        V8 cur0, cur1, nxt0, nxt1;
        cur0 = kat(stage, 0);
        cur1 = kat(stage, 1);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int g = 0; g < KSTEPS / 2; ++g) {
            if (g + 1 < KSTEPS / 2) {
                nxt0 = kat(stage, 2 * (g + 1));
                nxt1 = kat(stage, 2 * (g + 1) + 1);
            }
            s = mfma32(cur0, qf[2 * g], s);
            s = mfma32(cur1, qf[2 * g + 1], s);
            __builtin_amdgcn_sched_barrier(0);
            cur0 = nxt0;
            cur1 = nxt1;
        }
        __builtin_amdgcn_s_setprio(0);
        return s;
    };
    auto pv_jit = [&](const half8_t &p0, const half8_t &p1, const unsigned short *stage) {
        half8_t cur0, cur1, nxt0, nxt1;
        cur0 = vat(stage, 0, 0);
        cur1 = vat(stage, 0, 1);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            if (dt + 1 < DT) {
                nxt0 = vat(stage, dt + 1, 0);
                nxt1 = vat(stage, dt + 1, 1);
            }
            oacc[dt] = mfma32(cur0, p0, oacc[dt]);
            oacc[dt] = mfma32(cur1, p1, oacc[dt]);
            __builtin_amdgcn_sched_barrier(0);
            cur0 = nxt0;
            cur1 = nxt1;
        }
        __builtin_amdgcn_s_setprio(0);
    };

    // hide keys of tile t that some row of the wave must not see
    auto mask = [&](float16_t &s, int t) {
        const int kw = t * BC + 32 * kh;        // first key of this wave's half
        if (kw + 32 > kfree_w) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kw + 8 * (r >> 2) + 4 * lh + (r & 3);
                const bool vis = key < Nk && (!CAUSAL || key <= qi + off);
                s[r] = vis ? s[r] : -INFINITY;
            }
        }
    };

    // p = 2^(s c + nbase) for the 16 scores of the lane, packed to f16 in the
    // key order of the two PV k-steps
    auto exp_pack = [&](const float16_t &s, float nbase, half8_t &p0, half8_t &p1) {
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = exp2_fast(__builtin_fmaf(s[r], a.c, nbase));
        p0 = pack_f16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
        p1 = pack_f16x8(p[8], p[9], p[10], p[11], p[12], p[13], p[14], p[15]);
    };

    // row sum += the 16 f16 weights of the lane, in fp32 (dot products with (1, 1))
    auto add_sum = [&](float l, const half8_t &p0, const half8_t &p1) {
        const half2_t one = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            l = __builtin_amdgcn_fdot2(half2_t{p0[2 * i], p0[2 * i + 1]}, one, l, false);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            l = __builtin_amdgcn_fdot2(half2_t{p1[2 * i], p1[2 * i + 1]}, one, l, false);
        return l;
    };
    // Online softmax of one tile.  The weights are first formed against the
    // current base and kept if the lane's 16 weights add at most 4096 to its
    // row sum (every weight then fits f16 with room to spare and no rescale is
    // due; the row maximum is never formed).  Only when some row outgrows its
    // base that far (or a row has no base yet) is the row maximum taken, the
    // accumulator and row sum rescaled to it and the weights recomputed.  The
    // row sum adds, in fp32, the f16 weights that also feed the matrix product.
    auto softmax = [&](const float16_t &s, half8_t &p0, half8_t &p1) {
        exp_pack(s, nbase, p0, p1);
        const float l_old = l_run;
        l_run = add_sum(l_run, p0, p1);
        const bool over = !(l_run <= l_old + lim);
        if (__builtin_amdgcn_ballot_w64(over) != 0) {
            float mx = max3(s[0], s[1], s[2]);
            mx = max3(mx, s[3], s[4]);
            mx = max3(mx, s[5], s[6]);
            mx = max3(mx, s[7], s[8]);
            mx = max3(mx, s[9], s[10]);
            mx = max3(mx, s[11], s[12]);
            mx = max3(mx, s[13], s[14]);
            mx = __builtin_fmaxf(mx, s[15]);
            mx = pair_max(mx);
            const float m_new = __builtin_fmaxf(m_run, mx * a.c);
            const float alpha = (m_new == -INFINITY) ? 1.f : exp2_fast(m_run - m_new);
            m_run = m_new;
            nbase = (m_new == -INFINITY) ? 0.f : -m_new;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) oacc[dt] *= alpha;
            exp_pack(s, nbase, p0, p1);
            l_run = add_sum(l_old * alpha, p0, p1);
            lim = (m_new == -INFINITY) ? -INFINITY : kMaxLaneSum;
        }
    };

    // Tile loop: one tile per step, in order -- scores, softmax, PV -- and one
    // barrier.  The latencies of a step are hidden by the waves of the other
    // workgroups on the CU, whose barriers are independent of this one's.
    // Tile i + AHEAD is loaded during step i, into the stage that tile i - 1
    // (two stages: the other one) has left.  With three stages the loads have
    // the whole next step as well: step i waits for tile i + 1's, and writes its
    // bf16 V, after its own scores.  With two, at its end.
    constexpr int AHEAD = SM::AHEAD;
    if (ntiles > 0) {
        vregs_t v0;
        gload_to(v0, 0);
        if (AHEAD == 2 && ntiles > 1) gload_to(vr, 1);
        vstore_from(v0, stage_at(0));
        if (AHEAD == 2 && ntiles > 1)
            lds_loads_done<SM::SPLIT ? NP : 2 * NP>();   // all but those of tile 1
        else
            lds_loads_done<0>();
    }
    lds_barrier();
    auto step = [&](int i, auto R) {   // R: stage of tile i (i % NSTAGE)
        constexpr int r = decltype(R)::value;
        // the next tile's loads are issued after the K operand reads (their
        // scalar set-up then overlaps the LDS latency, and at D = 128 their
        // registers are not live across the QK^T product)
        float16_t s = D == 128 ? scores_jit(stage_at(r)) : scores(stage_at(r));
        if (AHEAD == 2 && i + 1 < ntiles) {
            lds_loads_done<0>();   // tile i + 1, loaded since the previous step
            vstore_from(vr, stage_at((r + 1) % NSTAGE));
        }
        const bool more = i + AHEAD < ntiles;
        if (more) gload_to(vr, (r + AHEAD) % NSTAGE);
        mask(s, i);
        half8_t p0, p1;
        half8_t va[KSTEPS];
        // D = 64: the V operands are read before the softmax, so that their
        // LDS latency is not on the step's critical path
        if constexpr (D == 64) vread(stage_at(r), va);
        softmax(s, p0, p1);
        if constexpr (D == 128) {
            pv_jit(p0, p1, stage_at(r));
        } else {
            pv(p0, p1, va);
        }
        if (AHEAD == 1) {
            if (more) vstore_from(vr, stage_at((r + AHEAD) % NSTAGE));
            lds_loads_done<0>();
        }
        lds_barrier();
    };
    for (int i = 0; i < ntiles; i += NSTAGE) {   // unrolled over the stages: their offsets are constants
        step(i, std::integral_constant<int, 0>{});
        if (i + 1 < ntiles) step(i + 1, std::integral_constant<int, 1>{});
        if constexpr (NSTAGE > 2) {
            if (i + 2 < ntiles) step(i + 2, std::integral_constant<int, 2>{});
        }
    }
    __syncthreads();   // the merge below reuses the stage memory

    // ---- merge the two key halves of each slot through LDS
    float *mf = reinterpret_cast<float *>(smem);
    constexpr int NV = DT * 16 + 2;
    float *mine = mf + (slot * NV) * 64 + l;
    if (NQ == 2 && kh == 1) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[(dt * 16 + r) * 64] = oacc[dt][r];
        mine[(DT * 16) * 64] = m_run;
        mine[(DT * 16 + 1) * 64] = l_run;
    }
    if (NQ == 2) __syncthreads();
    if (kh != 0 || !live) return;
    if (NQ == 2) {
        const float m1 = mine[(DT * 16) * 64];
        const float l1 = mine[(DT * 16 + 1) * 64];
        const float M = __builtin_fmaxf(m_run, m1);
        const float a0 = (m_run == -INFINITY) ? 0.f : exp2_fast(m_run - M);
        const float a1 = (m1 == -INFINITY) ? 0.f : exp2_fast(m1 - M);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                oacc[dt][r] = a0 * oacc[dt][r] + a1 * mine[(dt * 16 + r) * 64];
        l_run = a0 * l_run + a1 * l1;
        m_run = M;
    }
    const float l_tot = pair_sum(l_run);
    // a row with no visible key (only with per-sequence lengths) gives 0 and
    // a log-sum-exp of -inf
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (qi < Nq) {
        TOUT *op = reinterpret_cast<TOUT *>(a.o) + ((size_t)((size_t)b * Nq + qi) * a.Hq + h) * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            if constexpr (sizeof(TOUT) == 4) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *reinterpret_cast<float4_t *>(op + 32 * dt + 8 * i + 4 * lh) =
                        float4_t{oacc[dt][4 * i] * inv, oacc[dt][4 * i + 1] * inv,
                                 oacc[dt][4 * i + 2] * inv, oacc[dt][4 * i + 3] * inv};
            } else {
                // a lane has half of each 8-column chunk, lane l ^ 32 the other:
                // of every two chunks the pair exchanges halves, so that each
                // stores one chunk of 16 bytes (8-byte stores of the halves took
                // 2960 cycles of a D = 128 workgroup's end, these 1800: 4 x 16/2
                // heads, 135 rows, fp16 9.35 -> 7.98 us; 333 rows, bf16 13.1 ->
                // 12.1; D = 64, 100 rows 7.3 -> 6.8)
                typedef TOUT t4 __attribute__((ext_vector_type(4)));
                typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    uint2_t u[2];
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        t4 x;
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = from_f32<TOUT>(oacc[dt][4 * (i + n) + e] * inv);
                        u[n] = __builtin_bit_cast(uint2_t, x);
                    }
                    auto lo = __builtin_amdgcn_permlane32_swap(u[0][0], u[1][0], false, false);
                    auto hi = __builtin_amdgcn_permlane32_swap(u[0][1], u[1][1], false, false);
                    st16(op + 32 * dt + 8 * (i + lh), uint4_t{lo[0], hi[0], lo[1], hi[1]});
                }
            }
        }
        if (a.lse && lh == 0)
            a.lse[((size_t)b * a.Hq + h) * Nq + qi] = l_tot > 0.f ? (m_run + log2f(l_tot)) * kLn2 : -INFINITY;
    }
}

// Compute units of the current device (cached per device; 0 if unknown).
int cu_count() {
    static std::atomic<int> cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0 && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
        cached[dev].store(n, std::memory_order_relaxed);
    return n;
}

// Query heads per workgroup of `slots` slots: the most of one key/value group,
// up to 4, that fill the slots evenly.
int default_heads(int slots, int G) {
    int hw = 1;
    for (int c = 2; c <= (slots < 4 ? slots : 4); c *= 2)
        if (slots % c == 0 && G % c == 0) hw = c;
    return hw;
}

// Whether a D = 64 call takes eight slots per workgroup (one 16-wave workgroup
// per CU) where the caller leaves the choice, rather than four (two of 8
// waves).  Eight stage each tile half as often and run a full CU 4 to 5 %
// faster; four end more evenly, and one's start and end go under in the other's
// steps.  Calls whose workgroups all take about the same time, not causal or few
// rows against many keys, compare rounds: a last round that leaves four-slot
// workgroups alone on their CUs costs them 0.58 of a full one (4 against 8, us,
// 32/8 heads, bf16: 1056 rows 24.8 / 23.3; 1400 rows 28.9 / 26.9; 2048 rows 47.9 /
// 45.6; 2500 rows 77.8 / 92.9; 5920 rows 342.9 / 329.6; 8192 rows 631 / 605; 16/1
// heads, 3000 rows 54.0 / 48.1; fp16, 16384 rows 1245 / 1198; bf16, 9000 rows 417.6
// / 453.7; causal, 4 x 1024 rows against 4096 keys 141.7 / 134.2, 5 x 1000 against
// 5000 216 / 228), and a round's start and end cost eight the time of some 90
// keys more, 32 where there is one round (over 1600 calls of 16 to 6000 keys the
// choice is on average 0.1 % off the better one; without those keys 2.1, at most
// 42: 49 x 32/8, 57 rows 13.7 / 15.4; 62 x 32/8, 189 rows 47.7 / 63.7; 14 x 32/4,
// 67 rows 8.5 / 10.0; 7 x 32/8, 1406 rows 143.9 / 153.7).  A K/V that the memory
// side's 256 MB do not hold comes from HBM for every workgroup that reads it:
// eight where they are half as many, and two rounds or more (97 x 16/16 heads,
// 172 rows, 2228 keys 401 / 322; 84 x 16/16, 506 rows, 1233 keys 419 / 338; at 290
// to 330 MB -10 to +9 %; not for uneven lengths in order, 33 x 16/16, 439 rows,
// 2978 to 2233 keys 223 / 256).
// Square causal calls end on short workgroups in any case: eight from four full
// rounds and 7168 rows on, where four heads share a workgroup (32/8, 8192 rows
// 314 / 307; 2 x 32/8, 7200 rows 483 / 476; 16/1 16384, fp16 628 / 621; but 2 x
// 32/8, 4700 rows 220 / 228; 29 x 32/4, 290 rows 35.7 / 46.2; and 2 x 16/16 heads,
// 5000 rows 137 / 146).  Lengths of their own are not known here.  Where they are
// equal, eight gain as much (16 x 32/8 heads, 512 rows against 4096 keys 370 /
// 348; 32 x 16/2, 256 rows 205 / 184), and long uneven ones lose at most 1 % (the
// first call with 614 keys and more 180 / 181); short ones would lose up to 12 %
// (16 x 512 rows against up to 1024 keys 64.5 / 72.5, against 2048 99.8 / 104.1,
// where equal ones gain 1.4 %), and so would those of one round, whose long and
// short workgroups then no longer share CUs (4 x 512 rows against 2048 to 4096
// keys 62.7 / 69.2): eight from 2048 keys and two rounds on.
bool eight_slots(const Problem &p, bool causal) {
    if (p.D != 64 || p.hw > 0 || p.block_table) return false;
    const long long cus = cu_count();
    if (cus == 0) return false;
    const int G = p.Hq / p.Hkv;
    auto groups = [&](int slots) {
        const int hw = default_heads(slots, G), rows = WR * slots / hw;
        return ((long long)p.Nq + rows - 1) / rows * p.B * p.Hkv * (G / hw);
    };
    const long long four = groups(4), eight = groups(8);
    const bool square = causal && p.Nk < 4LL * p.Nq;
    const long long kv_bytes = 256LL * p.B * p.Hkv * p.Nk;
    if (!square && eight >= 2 * cus && four == 2 * eight && kv_bytes > 335000000 && (!p.seqlens || p.B > kMaxRanked))
        return true;
    if (p.seqlens && (p.Nk < 2048 || eight < 2 * cus)) return false;
    if (square) return G % 4 == 0 && four >= 8 * cus && p.Nk >= 7168;
    const long long rest = four % (2 * cus);
    const long long cost4 = four / (2 * cus) * 1000 + (rest == 0 ? 0 : rest <= cus ? 580 : 1000);
    return (eight + cus - 1) / cus * (955 + 1000 * (eight <= cus ? 32 : 90) / p.Nk) < cost4;
}

template <typename TIN, typename TOUT, int D, int NS, bool CAUSAL>
hipError_t launch_t(const Problem &p, hipStream_t stream) {
    using SM = Cfg<D, NS>;
    PrefillArgs a;
    a.q = p.q; a.k = p.k; a.v = p.v; a.o = p.o; a.lse = p.lse;
    a.B = p.B; a.Hq = p.Hq; a.Hkv = p.Hkv; a.Nq = p.Nq; a.Nk = p.Nk;
    a.seqlens = p.seqlens;
    a.block_table = p.block_table;
    a.page_size = p.page_size;
    a.max_pages = p.max_pages;
    a.num_pages = p.num_pages;
    // A zero scale keeps a tiny positive factor: every visible exponent is then
    // exactly 0 in fp32, and masked (-inf) scores still give 0.
    a.c = __builtin_fmaxf(__builtin_fabsf(p.scale), 1e-30f) * kLog2e;
    a.qsign = p.scale < 0.f ? 0x80008000u : 0u;
    const int G = p.Hq / p.Hkv;
    // query heads per workgroup: the requested packing, else the default
    a.HW = p.hw > 0 ? p.hw : default_heads(NS, G);
    const int RB = NS / a.HW;
    a.nmb = (p.Nq + WR * RB - 1) / (WR * RB);
    const long long nblocks = (long long)a.nmb * p.B * p.Hkv * (G / a.HW);
    if (nblocks <= 0) return hipSuccess;
    if (nblocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    a.G = G;
    a.lgHW = a.HW == 8 ? 3 : a.HW == 4 ? 2 : a.HW == 2 ? 1 : 0;
    a.nhg = Divisor(G / a.HW);
    a.nkv = Divisor(p.Hkv);
    a.per_mb = Divisor((unsigned)p.B * p.Hkv * (G / a.HW));   // <= nblocks
    const int cus = cu_count();
    const bool at_once = nblocks <= (long long)SM::WPC * cus;   // every workgroup is resident from the start
    a.first = p.causal && at_once ? (cus + (int)a.per_mb.d - 1) / (int)a.per_mb.d : a.nmb;
    a.ranked = 0;
    a.row_blocks = Divisor(a.nmb);
    if (p.seqlens && p.B > 1 && p.B <= kMaxRanked && nblocks > cus && p.Nk >= RANKED_KEYS &&
        p.Nk >= RANKED_KEYS_EACH * (long long)p.B) {
        const int per_seq = p.Hkv * (G / a.HW);
        a.per_seq = Divisor(per_seq);
        a.ranked = at_once ? (cus + per_seq - 1) / per_seq : a.nmb * p.B;
    }
    if constexpr (NS == NSLOT) {
        if (p.block_table) {
            hipLaunchKernelGGL((prefill_kernel<TIN, TOUT, D, NS, CAUSAL, true>), dim3((unsigned)nblocks),
                               dim3(SM::NT), 0, stream, a);
            return hipGetLastError();
        }
    } else if (p.block_table) {
        return hipErrorInvalidValue;   // paged K/V takes the default slots
    }
    hipLaunchKernelGGL((prefill_kernel<TIN, TOUT, D, NS, CAUSAL, false>), dim3((unsigned)nblocks),
                       dim3(SM::NT), 0, stream, a);
    return hipGetLastError();
}

template <typename TIN, typename TOUT, int D, bool CAUSAL>
hipError_t launch_s(const Problem &p, hipStream_t s) {
    switch (p.slots) {
    case 1: return launch_t<TIN, TOUT, D, 1, CAUSAL>(p, s);
    case 2: return launch_t<TIN, TOUT, D, 2, CAUSAL>(p, s);
    case 4: return launch_t<TIN, TOUT, D, 4, CAUSAL>(p, s);
    case 8: return launch_t<TIN, TOUT, D, 8, CAUSAL>(p, s);
    default:
        return eight_slots(p, CAUSAL) ? launch_t<TIN, TOUT, D, 8, CAUSAL>(p, s) : launch_t<TIN, TOUT, D, NSLOT, CAUSAL>(p, s);
    }
}

template <typename TIN, typename TOUT>
hipError_t launch_d(const Problem &p, hipStream_t s) {
    if (p.D == 64) return p.causal ? launch_s<TIN, TOUT, 64, true>(p, s)
                                   : launch_s<TIN, TOUT, 64, false>(p, s);
    return p.causal ? launch_s<TIN, TOUT, 128, true>(p, s) : launch_s<TIN, TOUT, 128, false>(p, s);
}

}  // namespace

bool prefill_supported(int Hkv, int D, fa_dtype_t in) {
    return (D == 64 || D == 128) && (in == FA_F16 || in == FA_BF16) && tile_fits(Hkv, D, D == 64 ? Cfg<64>::BC : Cfg<128>::BC);
}

hipError_t launch_prefill(const Problem &p, hipStream_t stream) {
    if (p.in == FA_F16)
        return p.out == FA_F32 ? launch_d<f16_t, float>(p, stream)
                               : launch_d<f16_t, _Float16>(p, stream);
    return p.out == FA_F32 ? launch_d<bf16_t, float>(p, stream) : launch_d<bf16_t, __bf16>(p, stream);
}

}  // namespace fa
