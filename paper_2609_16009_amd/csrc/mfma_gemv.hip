// Narrow MatMul on the matrix cores for larger M (gfx950): y[M,N] = x[M,K] . W[K,N] with M in
// tiles of 16 or 32 rows, W row-major [K,N] (bf16 or fp16), fp32 accumulation.
//
// Once x has enough rows the streaming GEMV runs out of vector ALU (it spends 2*M flops per
// weight element against HBM's ~1 byte per element), while the product stays HBM-bound for
// the matrix cores far beyond M = 32.  The paper's narrow-dimension conditions (Condition 2,
// Section III-A; Conditions 4-5, Section V) are about where the split between the two units
// lies; on MI355X it is measured, and nmm_gemv's AUTO path switches here above it.
//
//  * A workgroup (4 waves) owns one 128-column panel of W and one K-slice.
//  * W streams in stages of 64 rows x 128 columns (16 KB) together with the stage's 64 k of the
//    x tile (the MFMA A operand, 2-4 KB): each thread keeps two stages of 16-byte chunks in
//    flight, stores the oldest to a double-buffered LDS stage and reloads its registers in
//    place.  The waves read their v_mfma_f32_16x16x32 B operands back with ds_read_b64_tr_b16,
//    the gfx950 transposing LDS read (the B operand needs 8 consecutive k of one column; W rows
//    hold consecutive columns).  x travels with W instead of being staged for the whole slice
//    up front, so no workgroup waits for its x before its W stream starts and the slice length
//    is not bounded by LDS.
//  * Wave w owns the column tiles 2w and 2w+1 of the panel, so no cross-wave reduction is needed.  W
//    is the A operand and x the B operand, so a lane ends with 4 consecutive columns of one row and
//    stores 16 bytes at a time.
//  * Sums: the two MFMAs of a stage (at 32 rows the four of two stages) chain in fp32 from zero and are
//    added in fp64; the K-slices are added in fp64 as well.  Relative 2-norm error for K of 512 to 16384: up to 16
//    rows 4.9e-8 to 5.7e-8 in bf16 and 6.2e-8 to 7.0e-8 in fp16, 32 rows 6.5e-8 to 7.0e-8 and 8.0e-8 to 8.6e-8; one
//    fp32 chain over K: 2.3e-7 at K = 1536, 8.0e-7 at 16384.
//  * K-slices are combined like the GEMV's: device-scope stores of the slice's M rows (not of the
//    whole 16- or 32-row tile), a ticket per panel, and the last workgroup sums the slices in order,
//    16 bytes a load.  The tail is what bounds short weights: [7168, 2112] at 3 rows 10.7 us (13.9
//    with 4-byte partials of all 16 rows and 16 slices), [7168, 576] 7.8 (10.3).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "handoff.h"
#include "nmm_internal.h"
#include "out4.h"

namespace nmm {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __fp16 fp16x4 __attribute__((__vector_size__(4 * sizeof(__fp16))));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef __attribute__((address_space(3))) fp16x4 lds_f16x4;

constexpr int kRsrcWord3 = 0x00020000;
constexpr int kLoadNT = 2;
constexpr int kDevice = 16;                    // sc1: device scope (past the XCD's L2)
constexpr uint32_t kOutOfRange = 0x80000000u;
constexpr int kWStride = kMfmaPanelCols + 8;   // LDS row stride of a W stage (elements)
constexpr int kXStride = kMfmaStageRows + 8;   // LDS row stride of an x stage (elements)
// A gather of up to kFewSlices slices has a kernel of its own: batches of 16 (8 at 32 rows) add zeros for the
// slices that are not there, in fp64, and take 130 registers for the loads ([3072, 22912], 2 slices, at 4 / 16
// rows 29.1 / 31.2 us with them, 27.4 / 29.8 without; [1536, 12288] at 16 rows 11.5 and 10.8).
constexpr int kMaxSlices = 16, kFewSlices = 4;
constexpr int kMfmaDepth = 2;                  // stages in flight per thread (2-4 measured alike)

struct MParams {
    const uint16_t* x;
    int64_t ldx;
    const uint16_t* w;
    float* y;              // fp32 output (may be null when ybf is set)
    int64_t ldy;
    uint16_t* ybf;         // optional bf16 output, ybf[m * ldyb + n]
    int64_t ldyb;
    int away;              // bf16 rounding: 0 nearest-even, 1 ties away from zero
    float* part;
    unsigned* tickets;
    int M, K, N;
    uint32_t row_bytes, w_extent;
    int panels, ks, rows, items, mblocks;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, kRsrcWord3);
}

template <int DT>
__device__ __forceinline__ f32x4 mfma(i32x4 a, i32x4 b, f32x4 c) {
    if constexpr (DT == NMM_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// A operand (W transposed) of one 16-column tile for 32 k-rows starting at `row0` of the LDS stage: lane
// (g = lane/16, j = lane%16) receives W[row0 + 8g .. + 7][col0 + j] via two transposing reads.
template <int DT>
__device__ __forceinline__ i32x4 load_w(const uint16_t* wst, int row0, int col0, int g, int j) {
    const uint16_t* base = wst + (row0 + 8 * g + (j >> 2)) * kWStride + col0 + 4 * (j & 3);
    uint2 lo, hi;
    if constexpr (DT == NMM_BF16) {
        lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(base)));
        hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(base + 4 * kWStride)));
    } else {
        lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_f16x4*)(base)));
        hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_f16x4*)(base + 4 * kWStride)));
    }
    return i32x4{int(lo.x), int(lo.y), int(hi.x), int(hi.y)};
}

// SLICES: the gather's batch is at most this many K-slices (0: one slice, nothing handed over).  TALL (one
// slice): x is the A operand, and a lane ends with 4 consecutive rows of one column instead.
template <int DT, int MT, int D, bool BF, int SLICES, bool TALL>
__global__ __launch_bounds__(kThreads) void mfma_gemv_kernel(const MParams p) {
    // two stage buffers, each a W tile [64][kWStride] followed by an x tile [MT][kXStride]
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    __shared__ int s_last;
    constexpr int MTILES = MT / 16;
    constexpr bool SPLIT = SLICES > 0;
    static_assert(!(SPLIT && TALL), "partial sums are stored in rows");
    constexpr int kStage = kMfmaStageRows * kWStride + MT * kXStride;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;

    const uint32_t bid = blockIdx.x;
    const int item = static_cast<int>(bid % uint32_t(p.items));
    const int mb = static_cast<int>(bid / uint32_t(p.items));
    const int panel = SPLIT ? item / p.ks : item, slice = SPLIT ? item - panel * p.ks : 0;
    const int m0 = mb * MT, k0 = slice * p.rows, n0 = panel * kMfmaPanelCols;
    const int stages = (min(p.rows, p.K - k0) + kMfmaStageRows - 1) / kMfmaStageRows;
    const int mrows = min(MT, p.M - m0);

    // ---- W: thread t takes chunk t%16 of rows t/16 + 16q (q < 4) of a stage.
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.w, p.w_extent);
    const int wc = tid & 15, wr0 = tid >> 4;
    const int chunks_valid = min(16, (p.N - n0 + 7) / 8);
    auto w_off = [&](int st, int q) -> uint32_t {
        const int row = k0 + st * kMfmaStageRows + wr0 + 16 * q;
        return (st < stages && row < p.K && wc < chunks_valid) ? uint32_t(row) * p.row_bytes + uint32_t(n0 / 8 + wc) * 16u
                                                              : kOutOfRange;
    };
    // ---- x: thread t takes chunk t%8 (8 k) of row t/8 of the stage's 64 k; rows past M or
    // chunks past K read zeros, and elements past K inside the last chunk are cleared on the way
    // to LDS (the padding of a row is read but never used).
    const int xm = tid >> 3, xc = tid & 7;
    const __amdgpu_buffer_rsrc_t xr =
        make_rsrc(p.x + int64_t(m0) * p.ldx, uint32_t(((mrows - 1) * p.ldx + (p.K + 7) / 8 * 8) * 2));
    const int xk_left = p.K - (k0 + 8 * xc);   // elements of this thread's chunk of stage 0 inside K
    auto x_off = [&](int st) -> uint32_t {
        const int left = xk_left - st * kMfmaStageRows;
        return (st < stages && xm < mrows && left > 0) ? uint32_t((xm * p.ldx + k0 + st * kMfmaStageRows + 8 * xc) * 2)
                                                      : kOutOfRange;
    };

    // D stages in flight: the registers of stage s go to LDS and are then reloaded with stage
    // s + D in place (no register copies, so the stream never drains); past the slice they read
    // zeros without touching memory.
    i32x4 wreg[D][4], xreg[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
        for (int q = 0; q < 4; ++q) wreg[d][q] = __builtin_amdgcn_raw_buffer_load_b128(wr, w_off(d, q), 0, kLoadNT);
        xreg[d] = __builtin_amdgcn_raw_buffer_load_b128(xr, x_off(d), 0, 0);
    }

    double acc[MTILES][2][4];
#pragma unroll
    for (int mt = 0; mt < MTILES; ++mt)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[mt][t][i] = 0.0;

    // one stage: registers to LDS buffer (s & 1), reload with stage s + D, then the MFMAs.  A
    // wave that writes buffer (s & 1) has passed the barrier of stage s - 1, so every wave has
    // finished reading stage s - 2 from it.
    f32x4 part[MTILES][2];
    auto stage = [&](int s, i32x4 (&wd)[4], i32x4& xd, bool first, bool last) {
        uint16_t* wst = smem + (s & 1) * kStage;
        uint16_t* xst = wst + kMfmaStageRows * kWStride;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            *reinterpret_cast<i32x4*>(wst + (wr0 + 16 * q) * kWStride + 8 * wc) = wd[q];
            wd[q] = __builtin_amdgcn_raw_buffer_load_b128(wr, w_off(s + D, q), 0, kLoadNT);
        }
        if (tid < MT * 8) {
            i32x4 v = xd;
            if (p.K & 7) {
                const int left = xk_left - s * kMfmaStageRows;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] &= (2 * e + 1 < left) ? -1 : (2 * e < left ? 0x0000FFFF : 0);
            }
            *reinterpret_cast<i32x4*>(xst + xm * kXStride + 8 * xc) = v;
        }
        xd = __builtin_amdgcn_raw_buffer_load_b128(xr, x_off(s + D), 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        // the 32-row steps of a chain run in fp32 from zero, then add to the fp64 sums
#pragma unroll
        for (int kk = 0; kk < kMfmaStageRows / 32; ++kk) {
            i32x4 x[MTILES];
#pragma unroll
            for (int mt = 0; mt < MTILES; ++mt)
                x[mt] = *reinterpret_cast<const i32x4*>(xst + (16 * mt + j) * kXStride + 32 * kk + 8 * g);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const i32x4 w = load_w<DT>(wst, 32 * kk, 16 * (2 * wave + t), g, j);
#pragma unroll
                for (int mt = 0; mt < MTILES; ++mt)
                    part[mt][t] = mfma<DT>(TALL ? x[mt] : w, TALL ? w : x[mt], kk == 0 && first ? f32x4{0.f, 0.f, 0.f, 0.f} : part[mt][t]);
            }
        }
        if (last) {
#pragma unroll
            for (int mt = 0; mt < MTILES; ++mt)
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[mt][t][i] += double(part[mt][t][i]);
        }
    };
    // a chain is one stage, or the D stages of an iteration for 32 rows, whose sums are twice as many
    constexpr bool kLong = MTILES == 2;
    int s0 = 0;
    for (; s0 + D <= stages; s0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) stage(s0 + d, wreg[d], xreg[d], !kLong || d == 0, !kLong || d == D - 1);
    }
#pragma unroll
    for (int d = 0; d + 1 < D; ++d)
        if (s0 + d < stages) stage(s0 + d, wreg[d], xreg[d], true, true);

    // ---- outputs: lane (g, j) holds columns 4 g .. + 3 of row j of its tiles
    const int64_t pbase = ((int64_t(mb) * p.panels + panel) * p.ks) * (int64_t(MT) * kMfmaPanelCols);
    const bool wide = wide_f32(p.y, p.ldy, 0), wide_b = BF && wide_bf16(p.ybf, p.ldyb, 0);
    auto put = [&](int m, int n, const f32x4 f) {
        const float v[4] = {f[0], f[1], f[2], f[3]};
        if (!BF || p.y) put4(p.y + int64_t(m) * p.ldy, n, p.N, v, wide);
        if constexpr (BF) put4(p.ybf + int64_t(m) * p.ldyb, n, p.N, v, p.away, wide_b);
    };
    auto value = [&](int mt, int t) {
        return f32x4{float(acc[mt][t][0]), float(acc[mt][t][1]), float(acc[mt][t][2]), float(acc[mt][t][3])};
    };
    if constexpr (!SPLIT) {
        if constexpr (TALL) {
#pragma unroll
            for (int mt = 0; mt < MTILES; ++mt)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const f32x4 v = value(mt, t);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int ml = 16 * mt + 4 * g + i, n = n0 + 16 * (2 * wave + t) + j;
                        if (ml >= mrows || n >= p.N) continue;
                        if (!BF || p.y) p.y[int64_t(m0 + ml) * p.ldy + n] = v[i];
                        if constexpr (BF) p.ybf[int64_t(m0 + ml) * p.ldyb + n] = to_bf16_mode(v[i], p.away);
                    }
                }
            return;
        }
#pragma unroll
        for (int mt = 0; mt < MTILES; ++mt)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                if (16 * mt + j < mrows) put(m0 + 16 * mt + j, n0 + 16 * (2 * wave + t) + 4 * g, value(mt, t));
        return;
    }
    // the slice's real rows, 16 bytes a store, at device scope: piece o of a slice is columns
    // 4 (o % kQuads) .. + 3 of row o / kQuads
    constexpr int kQuads = kMfmaPanelCols / 4, kSlicePieces = MT * kQuads;
    const __amdgpu_buffer_rsrc_t pr = make_rsrc(p.part + pbase, uint32_t(p.ks) * kSlicePieces * 16u);
#pragma unroll
    for (int mt = 0; mt < MTILES; ++mt)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int o = (16 * mt + j) * kQuads + 4 * (2 * wave + t) + g;
            if (16 * mt + j < mrows)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, value(mt, t)), pr,
                                                       uint32_t(slice * kSlicePieces + o) * 16u, 0, kDevice);
        }
    // same hand-off as the GEMV: completed device-scope stores, one ticket, ordered gather
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
        s_last = arrive(p.tickets + int64_t(mb) * p.panels + panel, unsigned(p.ks));
    }
    __syncthreads();
    if (!s_last) return;
    // every piece of the panel sums its slices in slice order in fp64; the loads of PER pieces x QB
    // slices are all in flight before any is added (rows past M load nothing)
    constexpr int PER = kSlicePieces / kThreads;            // pieces per thread (2 or 4)
    constexpr int QB = SLICES < 32 / PER ? SLICES : 32 / PER;   // slices per batch
    const int n_out = mrows * kQuads;
    double sum[PER][4];
#pragma unroll
    for (int r = 0; r < PER; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[r][i] = 0.0;
    for (int q0 = 0; q0 < p.ks; q0 += QB) {
        f32x4 v[PER][QB];
#pragma unroll
        for (int r = 0; r < PER; ++r)
#pragma unroll
            for (int u = 0; u < QB; ++u) {
                const int o = tid + r * kThreads;
                const uint32_t off = (o < n_out && q0 + u < p.ks) ? uint32_t((q0 + u) * kSlicePieces + o) * 16u : kOutOfRange;
                v[r][u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(pr, off, 0, kDevice));
            }
#pragma unroll
        for (int r = 0; r < PER; ++r)
#pragma unroll
            for (int u = 0; u < QB; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[r][i] += double(v[r][u][i]);
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int o = tid + r * kThreads;
        if (o < n_out)
            put(m0 + o / kQuads, n0 + 4 * (o % kQuads),
                f32x4{float(sum[r][0]), float(sum[r][1]), float(sum[r][2]), float(sum[r][3])});
    }
}

template <int DT, int MT, bool BF>
void launch_bf(const MParams& mp, int64_t grid, size_t lds, hipStream_t s) {
    const dim3 g(static_cast<uint32_t>(grid)), block(kThreads);
    if (mp.ks > kFewSlices) {
        hipLaunchKernelGGL((mfma_gemv_kernel<DT, MT, kMfmaDepth, BF, kMaxSlices, false>), g, block, lds, s, mp);
    } else if (mp.ks > 1) {
        hipLaunchKernelGGL((mfma_gemv_kernel<DT, MT, kMfmaDepth, BF, kFewSlices, false>), g, block, lds, s, mp);
    } else if ((!mp.y || wide_f32(mp.y, mp.ldy, 0)) && (!BF || wide_bf16(mp.ybf, mp.ldyb, 0))) {
        hipLaunchKernelGGL((mfma_gemv_kernel<DT, MT, kMfmaDepth, BF, 0, false>), g, block, lds, s, mp);
    } else {
        // rows that take no wide store: 16 lanes store 64 bytes of a row, where four columns a lane would be four
        // stores of every fourth column ([1022, 33335] at 13 / 32 rows 23.9 / 25.8 us against 25.0 / 28.0)
        hipLaunchKernelGGL((mfma_gemv_kernel<DT, MT, kMfmaDepth, BF, 0, true>), g, block, lds, s, mp);
    }
}

template <int DT, int MT>
void launch_mt(const MParams& mp, int64_t grid, size_t lds, hipStream_t s) {
    if (mp.ybf) launch_bf<DT, MT, true>(mp, grid, lds, s);
    else launch_bf<DT, MT, false>(mp, grid, lds, s);
}

}  // namespace

size_t mfma_lds_bytes(const GemvPlan& p) {
    return size_t(2) * (kMfmaStageRows * kWStride + p.mt * kXStride) * 2;
}

nmm_status launch_mfma(const GemvArgs& a, const GemvPlan& p, unsigned* tickets, float* part, void* stream) {
    MParams mp{};
    mp.x = static_cast<const uint16_t*>(a.x);
    mp.ldx = a.ldx;
    mp.w = static_cast<const uint16_t*>(a.w);
    mp.y = a.y;
    mp.ldy = a.ldy;
    mp.ybf = static_cast<uint16_t*>(a.ybf);
    mp.ldyb = a.ybf_ldm;
    mp.away = a.ybf_away;
    mp.part = part;
    mp.tickets = tickets;
    mp.M = static_cast<int>(a.M);
    mp.K = static_cast<int>(a.K);
    mp.N = static_cast<int>(a.N);
    mp.row_bytes = static_cast<uint32_t>(a.ldw * 2);
    mp.w_extent = static_cast<uint32_t>(((a.K - 1) * a.ldw + (a.N + 7) / 8 * 8) * 2);
    mp.panels = p.n_full;
    mp.ks = p.ks_full;
    mp.rows = p.rows_full;
    mp.items = p.items;
    mp.mblocks = p.mblocks;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t lds = mfma_lds_bytes(p);
    if (a.dt == NMM_BF16) {
        if (p.mt == 16) launch_mt<NMM_BF16, 16>(mp, p.grid, lds, s);
        else launch_mt<NMM_BF16, 32>(mp, p.grid, lds, s);
    } else {
        if (p.mt == 16) launch_mt<NMM_F16, 16>(mp, p.grid, lds, s);
        else launch_mt<NMM_F16, 32>(mp, p.grid, lds, s);
    }
    return hipGetLastError() == hipSuccess ? NMM_OK : NMM_ERR_HIP;
}

}  // namespace nmm
