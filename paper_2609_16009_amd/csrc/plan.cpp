// Host-side argument checks and the GEMV partition.  Pure functions: no HIP calls, no device
// access, so they run (and are tested) on a machine without a GPU.
//
// The partition plays the role of Algorithm 2's init stage (Section IV-E), which splits a
// [K, N] weight into kParts K-slices x fractalNum 16-column fractals and spreads them evenly over
// at most 2P vector units.  Here the unit of work is a K-slice of a column panel (64 to 512
// columns; one 16-byte chunk per lane per row).  Panel width and K-split count follow rules
// fitted to measurements on MI355X over the decode shapes (see the comments below).
#include <algorithm>
#include <cstdlib>

#include "nmm_internal.h"

namespace nmm {
namespace {

constexpr int64_t kLimit = int64_t(1) << 31;

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t rup(int64_t a, int64_t b) { return cdiv(a, b) * b; }

int next_pow2(int64_t v) {
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

// The partition's tuning constants are fixed in the library, so a plan (and with it the order of
// every sum) depends on the sizes alone, and for an [N, K] weight on its leading dimensions too.  Only a library built with -DNMM_TUNING_ENV, for tuning
// sweeps, lets the environment override them; the library as built for use reads no environment.
int64_t tuned(const char* name, int64_t dflt) {
#ifdef NMM_TUNING_ENV
    const char* s = std::getenv(name);
    if (!s || !*s) return dflt;
    char* end = nullptr;
    long long v = std::strtoll(s, &end, 10);
    return (end && *end == '\0' && v > 0) ? v : dflt;
#else
    (void)name;
    return dflt;
#endif
}

bool tuned_set(const char* name) {
#ifdef NMM_TUNING_ENV
    return std::getenv(name) != nullptr;
#else
    (void)name;
    return false;
#endif
}

int m_tile_for(int64_t M) {
    if (M <= 1) return 1;
    if (M <= 2) return 2;
    if (M <= 4) return 4;
    if (M <= 8) return 8;
    return kMaxMTile;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

nmm_status validate_workspace(const void* ws, size_t bytes, size_t need) {
    if (need == 0) return NMM_OK;
    if (!ws || bytes < need || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0) return NMM_ERR_WORKSPACE;
    return NMM_OK;
}

nmm_status validate_gemv(const GemvArgs& a, int path) {
    if (path != NMM_PATH_AUTO && path != NMM_PATH_GEMV && path != NMM_PATH_MFMA) return NMM_ERR_PATH;
    if (a.dt != NMM_F16 && a.dt != NMM_BF16) return NMM_ERR_DTYPE;
    if (a.batch < 0 || a.M < 0 || a.K < 0 || a.N < 0) return NMM_ERR_SHAPE;
    if (a.M >= kLimit || a.K >= kLimit || a.N >= kLimit) return NMM_ERR_SHAPE;
    if (a.ldx < 0 || a.ldw < 0 || a.ldy < 0 || a.ldx >= kLimit || a.ldw >= kLimit || a.ldy >= kLimit)
        return NMM_ERR_SHAPE;
    if (a.sx < 0 || a.sw < 0 || a.sy < 0) return NMM_ERR_SHAPE;
    if (a.batch == 0 || a.M == 0 || a.N == 0) return NMM_OK;          // nothing is touched
    if (!a.y && !a.ybf) return NMM_ERR_NULL;                         // some output is required
    if (a.y && a.ldy < a.N) return NMM_ERR_SHAPE;
    if (a.ybf && (a.ybf_ldm < 0 || a.ybf_ldm >= kLimit)) return NMM_ERR_SHAPE;
    if (a.ybf && (a.ybf_group <= 0 || a.ybf_keep <= 0 || a.ybf_keep > a.ybf_group)) return NMM_ERR_ARG;
    if (a.ybf_away != 0 && a.ybf_away != 1) return NMM_ERR_ARG;
    if ((a.y && (reinterpret_cast<uintptr_t>(a.y) & 3u)) || (reinterpret_cast<uintptr_t>(a.ybf) & 1u))
        return NMM_ERR_ALIGN;
    if (a.K == 0) return NMM_OK;                                      // y = 0; x and W unused
    if (!a.x || !a.w) return NMM_ERR_NULL;
    if (a.ldx < a.K || a.ldw < a.N) return NMM_ERR_SHAPE;
    if (!aligned16(a.x) || !aligned16(a.w) || a.ldx % 8 || a.ldw % 8 || a.sx % 8 || a.sw % 8)
        return NMM_ERR_ALIGN;
    const int64_t extent = ((a.K - 1) * a.ldw + rup(a.N, 8)) * 2;    // bytes of one W
    if (extent >= kLimit) return NMM_ERR_SHAPE;
    // bytes of x one row block reads (blocks are at most 32 rows)
    const int64_t x_extent = ((std::min<int64_t>(a.M, 32) - 1) * a.ldx + rup(a.K, 8)) * 2;
    if (x_extent >= kLimit) return NMM_ERR_SHAPE;
    return NMM_OK;
}

// Panels and K-slices of a single 1- or 2-row product of up to 100 MB: chunks per panel, slices and
// row-steps in flight.  Measured on MI355X at one row over panels of 8 to 64 chunks, 4 to 16 steps and
// grids of 64 to 512 (against 128-byte panels and the power-of-two split that larger weights take):
//  * no K-split where 150 to 256 panels of some width cover the row (from 129 on for 16 and 32 chunks): nothing is
//    handed over (W_UQ [1536, 24576] 192 panels 14.5 us, [1536, 12288] 10.5; [700, 20000] 157 panels 8.7 against
//    12.8; [1536, 18432] 144 panels 14.0 against 16.5; [1280, 34000] 133 panels of 32 21.5, 266 of 16 23.3);
//  * else panels of 16 chunks (256 bytes: whole lines, also where rows start inside one) and as many
//    slices, up to 8, as keep one workgroup per CU: [3000, 3000] 8.5 against 11.1, [4099, 5003] 11.8
//    against 15.6, [4096, 7168] 13.5 against 15.5, [8192, 4096] 14.7 against 16.8, [1536, 6144] 8.1
//    against 9.4;
//  * panels of 8 chunks where that would need more slices, whose gather is a serial tail ([7168, 576] 14 slices of 9
//    panels 6.9, of 5 wider ones 7.4; [7168, 2112] level);
//  * no split of K up to 512 either ([512, 512] 4.4, two slices 4.9); rows past 256 panels of 32 chunks take 16, or
//    64 where K has few steps or they fit one round ([512, 70000] 16.2, 64 chunks 17.2, 8 chunks 16.5; [64, 80000] 64
//    chunks 4.9, 8 chunks 8.5; [256, 131072] 64 chunks 12.8, 16 chunks 13.5, 8 chunks 15.7);
//  * up to 12 MB about 144 workgroups, as the streams are short ([4096, 1024] 128 of them 6.9, 256 8.2; [2048, 2048]
//    level), and at most 4 slices of the wider panels.
// Eight row-steps in flight serve a split K and a short one as well as sixteen or better ([512, 512] 4.4 and 4.5,
// [64, 512] 3.2 and 3.9: at 8 chunks 16 steps are 512 rows).  A long unsplit stream keeps sixteen (W_UQ 15.2, eight
// 15.6), panels of 32 chunks in fewer than 150 workgroups only for two rows ([1280, 36000] one row 20.3 with eight
// and 21.1 with sixteen, two rows 23.9 and 20.8), which below K = 768 take twice the workgroups and four steps
// instead ([260, 34000] 7.8 against 8.6, [520, 33280] 10.7 and 11.8).
struct NarrowChoice {
    int cw = 0, ks = 1, unroll = 8;
};
NarrowChoice narrow_plan(int mt, int64_t K, int64_t chunks, int64_t w_bytes) {
    NarrowChoice c;
    for (int cw : {32, 16, 8}) {
        const int64_t panels = cdiv(chunks, cw);
        if (panels < (cw == 8 ? 150 : 129) || panels > 256) continue;
        c.cw = cw;
        if (panels >= 150) {
            if (K >= 1024) c.unroll = 16;
        } else if (cw == 32 && mt == 2) {
            if (K < 768) c.cw = 16;
            c.unroll = K < 768 ? 4 : 16;
        }
        return c;
    }
    const int64_t widest = cdiv(chunks, kPanelChunks);
    if (K <= 512) {
        c.cw = cdiv(chunks, 32) <= 256 ? 8 : K < 128 || (widest > 200 && widest <= 256) ? kPanelChunks : 16;
        return c;
    }
    const bool small = w_bytes <= int64_t(12) << 20;
    const int64_t want = small ? 144 : 256;
    const int64_t wide = want / cdiv(chunks, 16);
    c.cw = wide <= (small ? 4 : 10) ? 16 : 8;
    c.ks = static_cast<int>(std::max<int64_t>(1, c.cw == 16 ? std::min<int64_t>(8, wide) : std::min<int64_t>(16, want / cdiv(chunks, 8))));
    return c;
}

// The matrix-core partition: 128-column panels, K-slices of whole 64-row stages, x tiles of
// 16 or 32 rows.  As many slices as keep the grid within one workgroup per CU: a part-filled second
// round costs more than shorter slices save (measured on MI355X at 4 / 32 rows, floor(256 / panels)
// slices against the power of two nearest it: [4096, 5120] 6 slices 11.8 / 13.6 us against 8 14.1 /
// 17.7, [1024, 2560] 8 slices 6.6 / 8.5 against 16 8.8 / 14.2, [4096, 8960] 3 slices 15.7 / 18.3
// against 4 18.9 / 23.2; where the two agree, W_O's 4 and [8192, 8192]'s, nothing changes).
nmm_status plan_mfma(int64_t M, int64_t K, int64_t N, GemvPlan* p) {
    GemvPlan q;
    q.path = NMM_PATH_MFMA;
    q.mt = M <= 16 ? 16 : 32;
    q.mblocks = static_cast<int>(std::max<int64_t>(1, cdiv(M, q.mt)));
    q.unroll = 1;
    q.cw_full = kMfmaPanelCols / 8;
    q.n_full = static_cast<int>(cdiv(N, kMfmaPanelCols));
    if (M == 0 || N == 0 || K == 0) {
        *p = q;
        return NMM_OK;
    }
    const int64_t panels = int64_t(q.mblocks) * q.n_full;
    const int64_t want = tuned("NMM_GEMV_TARGET", kMfmaTargetGrid);
    // a short K takes at most 8 slices ([1536, 1536] at 4 / 32 rows 6.5 / 7.8 us, 12 slices 6.7 / 9.5; [512, 512] 5.1 /
    // 6.1, 2 slices 5.3 / 6.3; four would be 4.6 / 5.6 there)
    const int64_t ks_cap = tuned("NMM_GEMV_MAXSPLIT", K < kMfmaShortK ? 8 : 16);
    int64_t ks_want = std::max<int64_t>(1, want / panels);
    // no more slices than nmm_gemv_noalloc's scratch holds (170 panels of 32 rows: two)
    const int64_t slice_bytes = panels * q.mt * kMfmaPanelCols * 4;
    const int64_t fits = (int64_t(NMM_NOALLOC_SCRATCH_BYTES) - kTicketBytes) / slice_bytes;
    // 129 to 170 panels on a long K: three slices, two workgroups per CU side by side.  At 4 / 32 rows [4096, 16512]
    // 26.8 / 30.8 us against 30.0 / 31.8 with one, [2560, 20480] 20.7 / 24.6 against 22.4 / 26.0, [2048, 16512] 16.1 /
    // 19.5 against 16.5 / 17.7; two slices lose to one wherever the grid has over 128 panels ([2048, 22400], 175 panels,
    // 20.4 / 23.5 against 18.3 / 19.9; [4096, 16512] 32.9 / 38.8), and five to two at 86 to 89 ([2048, 11136] 13.2 / 16.5
    // against 12.2 / 14.6)
    if (ks_want == 1 && 2 * want / panels == 3 && fits >= 3 && K >= (q.mt == 16 ? kMfmaLongK : kMfmaLongK32)) ks_want = 3;
    ks_want = std::max<int64_t>(1, std::min(std::min(ks_want, ks_cap), fits));
    int64_t r = rup(cdiv(K, ks_want), kMfmaStageRows);
    int64_t k = cdiv(K, r);
    if (panels > kMaxTickets) {
        k = 1;
        r = rup(K, kMfmaStageRows);
    }
    q.ks_full = static_cast<int>(k);
    q.rows_full = static_cast<int>(r);
    q.ks_max = q.ks_full;
    q.items = q.n_full * q.ks_full;
    q.grid = int64_t(q.mblocks) * q.items;
    if (q.split()) {
        q.n_tickets = panels;
        q.part_floats = panels * q.ks_max * int64_t(q.mt) * kMfmaPanelCols;
        q.ws_bytes = static_cast<size_t>(kTicketBytes + q.part_floats * 4);
    }
    *p = q;
    return NMM_OK;
}

nmm_status plan_gemv(int64_t batch, int64_t M, int64_t K, int64_t N, int dt, int path, GemvPlan* p,
                     int unroll) {
    if (!p) return NMM_ERR_NULL;
    if (dt != NMM_F16 && dt != NMM_BF16) return NMM_ERR_DTYPE;
    if (path != NMM_PATH_AUTO && path != NMM_PATH_GEMV && path != NMM_PATH_MFMA) return NMM_ERR_PATH;
    if (batch < 0 || M < 0 || K < 0 || N < 0 || M >= kLimit || K >= kLimit || N >= kLimit)
        return NMM_ERR_SHAPE;
    GemvPlan q;
    // AUTO for a single matrix: the streaming GEMV for one row, the matrix cores from
    // kMfmaMinMDefault rows on.  At two rows the matrix-core launch wins only where its plan needs no
    // K-split: its split-K tail costs as much as the GEMV's second row or more.  Measured on MI355X: W_UQ [1536,
    // 24576] (one slice) 15.3 against 16.2 us; W_O [16384, 7168] (4 slices) 39.5 against 39.6; down
    // [7168, 2112] (15 slices) 10.6 against 9.9.  A batch has the streaming plan; whether its
    // launch takes the matrix cores instead is heads_on_mfma's.
    if (path == NMM_PATH_AUTO) {
        const int64_t mfma_min_m = tuned("NMM_MFMA_MIN_M", kMfmaMinMDefault);
        path = NMM_PATH_GEMV;
        if (batch <= 1 && M >= mfma_min_m) {
            path = NMM_PATH_MFMA;
        } else if (batch <= 1 && M == 2 && K > 0 && N > 0) {
            GemvPlan m;
            if (plan_mfma(M, K, N, &m) == NMM_OK && m.ks_full == 1) path = NMM_PATH_MFMA;
        }
    }
    if (path == NMM_PATH_MFMA) {
        if (batch > 1) return NMM_ERR_PATH;
        return plan_mfma(M, K, N, p);
    }
    q.path = NMM_PATH_GEMV;
    q.mt = m_tile_for(M);
    q.mblocks = static_cast<int>(std::max<int64_t>(1, cdiv(M, q.mt)));
    const int64_t chunks = cdiv(N, 8);
    const int64_t mats = std::max<int64_t>(batch, 1) * q.mblocks;
    const int64_t w_bytes = mats * K * chunks * 16;
    // Measured on MI355X: 1- and 2-row tiles stream best with about one workgroup per compute unit.
    // Weights up to 100 MB ("deep") choose panels and slices by narrow_plan below; larger ones take panels
    // up to 512 columns with 8 row-steps in flight.  Taller tiles keep 4 in flight and more workgroups.
    const bool narrow_m = q.mt <= 2;
    const bool deep = narrow_m && w_bytes <= int64_t(100) << 20;
    const NarrowChoice nc = deep && mats == 1 && K > 0 && N > 0 ? narrow_plan(q.mt, K, chunks, w_bytes) : NarrowChoice{};
    q.unroll = unroll > 0 ? unroll : static_cast<int>(tuned("NMM_GEMV_UNROLL", nc.cw ? nc.unroll : deep ? 16 : narrow_m ? 8 : 4));
    if (q.unroll != 2 && q.unroll != 4 && q.unroll != 8 && q.unroll != 16) q.unroll = 8;
    if (q.unroll == 16 && q.mt > 2) q.unroll = 8;                  // 16 only for 1- and 2-row tiles
    const int U = q.unroll;
    // Panel width (measured on MI355X over the decode shapes): as wide as possible, up to 32
    // chunks (64 for 16-row tiles and for 1-2-row tiles of weights over 100 MB), while the launch
    // still has >= 24 panels in total and every row is split into >= 2 panels; never narrower
    // than 8 chunks (128-byte row segments).
    int min_cw = static_cast<int>(tuned("NMM_GEMV_MINCW", 8));
    if (min_cw > kPanelChunks || (min_cw & (min_cw - 1))) min_cw = 8;
    int cw = static_cast<int>(tuned("NMM_GEMV_MAXCW", (q.mt >= 16 || (narrow_m && !deep)) ? 64 : 32));
    if (cw > kPanelChunks || (cw & (cw - 1)) || cw < min_cw) cw = std::max(min_cw, 32);
    // Workgroups wanted: one per ~100 KB of W, between 256 and 768 (fewer leave HBM idle; more
    // only add split-K gather work); 256 for the deep-prefetch plans.
    const int64_t want = tuned("NMM_GEMV_TARGET",
                                 narrow_m ? 256 : std::max<int64_t>(256, std::min<int64_t>(768, w_bytes / 100000)));
    while (cw > min_cw && (mats * cdiv(chunks, cw) < 24 || chunks < 2 * cw)) cw /= 2;
    // deep plans of a batch trade K-slices for narrower panels while twice the panels still fit the target
    if (nc.cw && !tuned_set("NMM_GEMV_MAXCW")) cw = nc.cw;
    else if (deep && U == 16 && !tuned_set("NMM_GEMV_MAXCW"))
        while (cw > min_cw && 2 * mats * cdiv(chunks, cw) <= want) cw /= 2;
    // K-slices per panel: the power of two nearest want / panels, capped (fewer for tall row
    // tiles, whose partial sums are MT times larger)
    const int64_t ks_cap = tuned("NMM_GEMV_MAXSPLIT", q.mt >= 8 ? 8 : 16);
    q.cw_full = cw;
    q.n_full = static_cast<int>(chunks / cw);
    q.tail_chunks = static_cast<int>(chunks % cw);
    if (q.tail_chunks) {
        // the staged x slice of a tail item must fit the LDS budget: rows_tail * mt * 4 bytes,
        // with rows_tail >= kWaves * (64 / tail_cw) * U
        int lds_cw = 1;
        while (int64_t(kWaves) * (kPanelChunks / lds_cw) * U * q.mt * 4 > kXStageBytes) lds_cw <<= 1;
        q.tail_cw = std::max(next_pow2(q.tail_chunks), lds_cw);
    }
    if (batch == 0 || M == 0 || N == 0 || K == 0) {
        q.items = 0;
        q.grid = 0;
        *p = q;
        return NMM_OK;
    }

    const int64_t rstep_full = int64_t(kWaves) * (kPanelChunks / q.cw_full);   // rows per WG step
    const int64_t rstep_tail = q.tail_chunks ? int64_t(kWaves) * (kPanelChunks / q.tail_cw) : 1;
    const int64_t panels_all = mats * (q.n_full + (q.tail_chunks ? 1 : 0));
    int64_t ks_want = 1;
    {
        const double ratio = double(want) / double(std::max<int64_t>(panels_all, 1));
        if (nc.cw && !tuned_set("NMM_GEMV_TARGET")) {
            ks_want = nc.ks;
        } else if (tuned("NMM_GEMV_KS_ANY", 0) > 0) {
            ks_want = std::max<int64_t>(1, std::min<int64_t>(ks_cap, int64_t(ratio + 0.5)));
        } else {
            while (ks_want < ks_cap && double(ks_want) * 1.41421356 < ratio) ks_want *= 2;   // nearest power of two
            ks_want = std::min(ks_want, ks_cap);
            // one or two rows: not more than one workgroup per CU ([10000, 9001], 36 panels: 7 slices 30.8
            // us, 8 slices 41.9).  Where that leaves over 30 % of the CUs idle, a last panel of up to a quarter's width,
            // whose workgroups end early, does not count ([800, 65600], 128 panels and 8 chunks: two slices 20.1,
            // one 23.6; but [4096, 16512], 32 panels and 16 chunks at two rows: 7 slices 26.4, 8 slices 27.9)
            if (narrow_m && mats == 1 && ks_want * panels_all > want) {
                const int64_t fit = std::max<int64_t>(1, want / panels_all);
                const bool idle = fit * panels_all * 10 < want * 7;
                ks_want = idle && q.tail_chunks && 4 * q.tail_chunks <= q.cw_full ? std::max<int64_t>(1, want / q.n_full) : fit;
            }
        }
    }

    auto slice = [&](int64_t rstep, int& ks, int& rows) {
        const int64_t unit = rstep * U;
        const int64_t cap = std::max<int64_t>(unit, (kXStageBytes / (4 * q.mt * rstep)) / U * unit);
        int64_t r = std::min<int64_t>(std::min<int64_t>(rup(cdiv(K, ks_want), unit), cap), rup(K, unit));
        int64_t k = cdiv(K, r);
        r = std::min<int64_t>(cap, rup(cdiv(K, k), unit));   // rebalance the slices
        k = cdiv(K, r);
        ks = static_cast<int>(k);
        rows = static_cast<int>(r);
    };
    if (q.n_full) slice(rstep_full, q.ks_full, q.rows_full);
    if (q.tail_chunks) slice(rstep_tail, q.ks_tail, q.rows_tail);
    const int64_t panels = q.n_full + (q.tail_chunks ? 1 : 0);
    if (mats * panels > kMaxTickets) {
        // more panels than arrival counters: give every panel a single K-slice instead
        auto whole = [&](int64_t rstep, int& ks, int& rows) {
            const int64_t unit = rstep * U;
            ks = 1;
            rows = static_cast<int>(rup(K, unit));
        };
        if (q.n_full) whole(rstep_full, q.ks_full, q.rows_full);
        if (q.tail_chunks) whole(rstep_tail, q.ks_tail, q.rows_tail);
        if (std::max(q.rows_full, q.rows_tail) * int64_t(q.mt) * 4 > kXStageBytes) return NMM_ERR_SHAPE;
    }
    q.ks_max = std::max(q.ks_full, q.ks_tail);
    q.items = q.n_full * q.ks_full + (q.tail_chunks ? q.ks_tail : 0);
    q.grid = batch * q.mblocks * int64_t(q.items);
    if (q.split()) {
        q.n_tickets = mats * panels;
        q.part_floats = mats * panels * q.ks_max * int64_t(q.mt) * kPanelCols;
        q.ws_bytes = static_cast<size_t>(kTicketBytes + q.part_floats * 4);
    }
    *p = q;
    return NMM_OK;
}


// Whether AUTO gives a batch to the matrix cores.  Measured on MI355X (batches of 8 / 32 / 128 heads):
//  * from two rows on: [128, 512] at 2 rows 3.3 / 3.7 / 6.7 us against 4.8 / 5.1 / 6.8 for the GEMV, at
//    4 rows 3.4 / 3.7 / 6.7 against 7.2 / 8.8 / 8.8, at 16 rows 3.5 / 3.9 / 7.6 against 15 / 21 / 21;
//    [512, 128] at 4 rows 4.5 / 4.7 / 6.1 against 7.0 / 7.6 / 8.2;
//  * at one row where K is short and the grid small, so that the GEMV has little to stream: [128, 512]
//    3.3 / 3.7 against 4.2 / 4.5 for 8 and 32 heads, but 7 % slower than the GEMV for 128; [512, 128] 2 to 7 % slower
//    for 8 and 32 heads, level for 128.
// All of K is one workgroup's, so a long K with few workgroups stays on the GEMV, which splits it.
bool heads_on_mfma(int64_t batch, int64_t M, int64_t K, int64_t N) {
    if (batch <= 1 || M <= 0 || K <= 0 || N <= 0) return false;
    const int64_t groups = batch * cdiv(N, kHeadsCols);          // workgroups per row block
    if (groups * cdiv(M, 16) >= kLimit / kThreads) return false;
    if (M == 1) return K <= 256 && groups <= 512;
    return K <= kHeadsLongK || groups >= 256;
}

// ---------------------------------------------------------------------------------------------
// The transposed-weight GEMV.  x's K-slice is staged in LDS as 16-bit values (at most
// kXStageBytes), so a slice holds at most 16384 / mt values of k; rows are dealt so that at
// least one workgroup per CU streams (4 r rows each, r at most 8).  The kernel runs one row (mt 1);
// the plans of more rows, which the matrix cores take, still say which sizes are refused and what
// workspace a call brings.
// ---------------------------------------------------------------------------------------------
nmm_status validate_gemv_nt(const GemvArgs& a) {
    if (a.dt != NMM_F16 && a.dt != NMM_BF16) return NMM_ERR_DTYPE;
    if (a.M < 0 || a.K < 0 || a.N < 0 || a.M >= kLimit || a.K >= kLimit || a.N >= kLimit) return NMM_ERR_SHAPE;
    if (a.ldx < 0 || a.ldw < 0 || a.ldy < 0 || a.ldx >= kLimit || a.ldw >= kLimit || a.ldy >= kLimit)
        return NMM_ERR_SHAPE;
    if (a.M == 0 || a.N == 0) return NMM_OK;
    if (!a.y) return NMM_ERR_NULL;
    if (a.ldy < a.N) return NMM_ERR_SHAPE;
    if (reinterpret_cast<uintptr_t>(a.y) & 3u) return NMM_ERR_ALIGN;
    if (a.K == 0) return NMM_OK;
    if (!a.x || !a.w) return NMM_ERR_NULL;
    if (a.ldx < a.K || a.ldw < a.K) return NMM_ERR_SHAPE;
    if (!aligned16(a.x) || !aligned16(a.w) || a.ldx % 8 || a.ldw % 8) return NMM_ERR_ALIGN;
    const int64_t extent = ((a.N - 1) * a.ldw + rup(a.K, 8)) * 2;     // bytes of Wt
    if (extent >= kLimit) return NMM_ERR_SHAPE;
    const int64_t x_extent = ((std::min<int64_t>(a.M, 4) - 1) * a.ldx + rup(a.K, 8)) * 2;
    if (x_extent >= kLimit) return NMM_ERR_SHAPE;
    return NMM_OK;
}

nmm_status plan_gemv_nt(int64_t M, int64_t K, int64_t N, NtPlan* p) {
    NtPlan q;
    q.mt = M <= 1 ? 1 : M <= 2 ? 2 : 4;
    q.mblocks = static_cast<int>(std::max<int64_t>(1, cdiv(M, q.mt)));
    if (M == 0 || N == 0 || K == 0) {
        *p = q;
        return NMM_OK;
    }
    const int64_t slice_max = kXStageBytes / 2 / q.mt;          // 16384, 8192 or 4096 (16-bit x in LDS)
    int64_t ks = cdiv(K, slice_max);
    const int64_t slice = rup(cdiv(K, ks), 512);
    ks = cdiv(K, slice);
    q.slice_k = static_cast<int>(slice);
    q.ks = static_cast<int>(ks);
    const int64_t target_rb = std::max<int64_t>(1, 256 / (ks * q.mblocks));
    // at most 8 rows per wave: short rows (small K) then spread over more workgroups, which
    // measured faster for W_UQ's [24576, 1536] (768 workgroups) than 24 rows per wave
    int r = static_cast<int>(std::min<int64_t>(8, std::max<int64_t>(1, N / (4 * target_rb))));
    r = static_cast<int>(std::min<int64_t>(32, std::max<int64_t>(1, tuned("NMM_NT_ROWS", r))));
    // rows per load step (rgroup) times steps in flight is 8 loads per lane: two rows per step keep
    // four steps in flight and read x from LDS once for two loads (W_O [7168, 16384] 39.0 us against
    // 41.7 with eight rows and one step, 49.7 with one row).  One row per wave (small N) keeps one.
    q.rgroup = r < 2 ? 1 : q.mt == 1 ? 2 : 4;
    q.r = (r + q.rgroup - 1) / q.rgroup * q.rgroup;
    const int64_t rb = cdiv(N, 4 * q.r);
    if (rb >= kLimit) return NMM_ERR_SHAPE;
    q.row_blocks = static_cast<int>(rb);
    q.grid = int64_t(q.mblocks) * rb * ks;
    if (q.grid >= kLimit) return NMM_ERR_SHAPE;
    if (ks > 1) {
        q.n_tickets = int64_t(q.mblocks) * rb;
        if (q.n_tickets > kMaxTickets) return NMM_ERR_SHAPE;
        q.ws_bytes = size_t(kTicketBytes) + size_t(q.grid) * q.mt * 4 * q.r * 4;
    }
    *p = q;
    return NMM_OK;
}

// The matrix-core form of the transposed-weight product, or false where the one-row GEMV is the
// better one.  Measured on MI355X (GPU time, W rotated over three copies):
//  * from two rows on always: W_O [7168, 16384] at 2 / 4 / 16 / 32 rows 41 / 44 / 40 / 47 us against
//    50 / 53 / 172 / 329 for the GEMV (in blocks of 4 rows); [576, 7168] 7.4 / 7.7 / 10.4 / 13.6
//    against 7.9 / 16.9 / 19.2 / 26.9; [512, 512] 3.0 / 3.1 / 3.2 / 3.9 against 4.1 / 4.8 / 5.7 / 5.7;
//  * one row up to K = 2048: [512, 512] 3.0 against 3.8, [1536, 1536] 3.9 against 4.6, W_UQ
//    [24576, 1536] 14.6 against 14.8, [7168, 2048] 8.5 against 8.7; past that the GEMV's 1 KB rows
//    win where rows are few or not 256-byte aligned ([576, 7168] 5.6 against 7.5, [5003, 4099] 11.4
//    against 12.0) and the two are within 5 % elsewhere.
bool plan_mfma_nt(const GemvArgs& a, NtMfmaPlan* p) {
    const int64_t M = a.M, K = a.K, N = a.N;
    if (M < 1 || K < 1 || N < 1 || (M == 1 && K > kMfmaNtOneRowK)) return false;
    NtMfmaPlan q;
    q.xr = M <= 4 ? 1 : M <= 8 ? 2 : M <= 16 ? 4 : 8;
    // x rows of a block are addressed through one 32-bit buffer resource (4 rows always fit)
    if (((std::min<int64_t>(M, 4 * q.xr) - 1) * a.ldx + rup(K, 8)) * 2 >= kLimit) q.xr = 1;
    q.mblocks = static_cast<int>(cdiv(M, 4 * q.xr));
    // two 16-row tiles of Wt per wave halve the x traffic from L2, which counts from 16 rows on: W_O 10 % faster than
    // with one at 16 rows and 16 % at 32 (40 and 47 us), [5003, 4099] 19 % at 32 (19.1); while the
    // grid still has over half a workgroup per CU (at fewer [2112, 7168] is a third slower with two)
    q.nt = q.xr >= 4 && cdiv(N, 32) >= 150 ? 2 : 1;
    q.row_blocks = static_cast<int>(cdiv(N, 16 * q.nt));
    // one workgroup per CU at most: a third group in flight (up to 8 rows; [2112, 7168] 5 % faster at 4); with more workgroups than CUs the smaller ring lets more of them share a CU (W_UQ at one
    // row 15 % faster)
    q.depth = q.row_blocks <= 256 && q.xr <= 2 ? 3 : 2;
    // Rows whose 16 nt-row blocks lie a multiple of 256 KB apart meet on the same memory channels when
    // all workgroups walk k in step, so block b starts its walk b * rot rounds on.  The shift that helps
    // lies 2^9 or 2^7 (not 2^8) under the block stride: a stride of 512 KB takes 1 round of 1 KB, 256 KB
    // takes 2 (at 4 rows [7168, 16384] 13 % faster than without, [4096, 16384] 17 %, [8192, 8192] 3 %; the other shift
    // makes them 31, 46 and 42 % slower).
    const int64_t stride = int64_t(16) * q.nt * a.ldw * 2;
    q.rot = stride % (1 << 19) == 0 ? 1 : stride % (1 << 18) == 0 ? 2 : 0;
    q.grid = rup(q.row_blocks, 8) * q.mblocks;
    if (q.grid > int64_t(0xFFFFFFFF) / kThreads) return false;   // a launch has fewer than 2^32 threads
    *p = q;
    return true;
}

}  // namespace nmm
