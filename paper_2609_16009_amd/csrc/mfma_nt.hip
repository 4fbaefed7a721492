// The transposed-weight product on the matrix cores (gfx950): y[M,N] = x[M,K] . Wt[N,K]^T for Wt
// row-major [N, K] (a torch Linear weight), x in blocks of 4, 8, 16 or 32 rows, fp32 out.
//
// The streaming form (gemv_nt_kernel) reads Wt once per block of 4 rows of x and spends 2 M flops a
// weight on the vector units.  Here Wt is read once per 32 rows:
//  * A workgroup owns 16 or 32 rows of Wt and all of K; its 4 waves share K in groups of 128 (256
//    bytes of each row), dealt round robin, so together they walk each row in order.  No K-split
//    across workgroups, so no workspace and no second pass: the waves' sums meet in LDS.
//  * Both operands of v_mfma_f32_16x16x32 want 8 consecutive k of one row per lane, which is what rows
//    of Wt and x hold, but loading fragments straight from memory (16 rows x 64 bytes an instruction)
//    takes a CU in at about a quarter of the rate of whole row pieces (W_O [7168, 16384] at 16 rows 68
//    us).  So both are staged: LDS-direct loads of 4 rows x 256 bytes each, into a ring private to the
//    wave (2 or 3 groups in flight, no barrier in the loop), with the chunks of a row permuted so that a
//    fragment read has no bank conflict.  The weight is the A operand and x the B operand, so a lane
//    ends with 4 consecutive n of one m.
//  * Sums: a chain of two MFMAs in fp32, then added in fp64 (the vector units are idle), waves
//    added in fp64 in wave order, one rounding to fp32 at the end.  One fp32 chain over K loses
//    precision with its length (relative 2-norm error 2.3e-7 at K = 1536, 8.0e-7 at 16384, against
//    7.1e-8 and 1.3e-7 for fp32 FMAs over 64 lanes); this form measures 4.7e-8 to 5.1e-8 in bf16 and
//    6.1e-8 to 6.6e-8 in fp16 for K of 512 to 16384.
//  * Bound by the weight's bytes up to about 16 rows (W_O 40 to 44 us, 5.3 to 5.9 TB/s), then also by x from
//    L2, which every workgroup reads whole: 47 us at 32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "nmm_internal.h"

namespace nmm {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kRsrcWord3 = 0x00020000;
constexpr int kLoadNT = 2;
constexpr uint32_t kOutOfRange = 0x80000000u;
constexpr int kNtWaves = 4;
constexpr int kRowBytes = kMfmaNtGroup * 2;     // bytes of one row in a group: 16 chunks
constexpr int kQuad = 4 * kRowBytes;            // one LDS-direct load: 4 rows of a group
constexpr int kTilePitch = 4 * 68;              // doubles of one 16 x 16 tile in LDS: [g][j][i], padded per g

struct NtMParams {
    const uint16_t* x;
    int64_t ldx;
    const uint16_t* wt;
    uint32_t row_bytes, w_extent;
    float* y;
    int64_t ldy;
    int M, K, N;
    int row_blocks, mblocks, rot;
};

template <int DT>
__device__ __forceinline__ f32x4 mfma(i32x4 a, i32x4 b, f32x4 c) {
    if constexpr (DT == NMM_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// The first `left` of a chunk's 8 values, zeros after them.
__device__ __forceinline__ i32x4 keep_first(i32x4 v, int left) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] &= (2 * e + 1 < left) ? -1 : (2 * e < left ? 0x0000FFFF : 0);
    return v;
}

// The fragments of two MFMA steps from LDS: once at most VM of the wave's loads are outstanding, F
// fragments at addresses a and b each (fragment f at byte offset OFF + 4096 f, the x fragments of the
// last MT at XOFF + 4096 f from ax and bx), complete when this returns.  The loads that fill LDS are
// LDS-direct: the compiler would wait for all of them before any read that may alias, so the wait
// and the reads are written out.
template <int VM, int NT, int MT, int OFF, int XOFF>
__device__ __forceinline__ void read_pair(i32x4 (&w0)[NT], i32x4 (&w1)[NT], i32x4 (&x0)[MT], i32x4 (&x1)[MT], uint32_t a,
                                          uint32_t b, uint32_t ax, uint32_t bx) {
    static_assert(VM < 64 && OFF + 4096 * NT < 65536 && XOFF + 4096 * MT < 65536, "immediate fields");
    if constexpr (NT == 1 && MT == 1)
        asm volatile("s_waitcnt vmcnt(%8)\n\tds_read_b128 %0, %4 offset:%9\n\tds_read_b128 %1, %5 offset:%9\n\t"
                     "ds_read_b128 %2, %6 offset:%10\n\tds_read_b128 %3, %7 offset:%10\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(w0[0]), "=&v"(w1[0]), "=&v"(x0[0]), "=&v"(x1[0])
                     : "v"(a), "v"(b), "v"(ax), "v"(bx), "n"(VM), "n"(OFF), "n"(XOFF) : "memory");
    else if constexpr (NT == 2 && MT == 1)
        asm volatile("s_waitcnt vmcnt(%10)\n\tds_read_b128 %0, %6 offset:%11\n\tds_read_b128 %1, %7 offset:%11\n\t"
                     "ds_read_b128 %2, %6 offset:%12\n\tds_read_b128 %3, %7 offset:%12\n\t"
                     "ds_read_b128 %4, %8 offset:%13\n\tds_read_b128 %5, %9 offset:%13\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(w0[0]), "=&v"(w1[0]), "=&v"(w0[1]), "=&v"(w1[1]), "=&v"(x0[0]), "=&v"(x1[0])
                     : "v"(a), "v"(b), "v"(ax), "v"(bx), "n"(VM), "n"(OFF), "n"(OFF + 4096), "n"(XOFF) : "memory");
    else if constexpr (NT == 1 && MT == 2)
        asm volatile("s_waitcnt vmcnt(%10)\n\tds_read_b128 %0, %6 offset:%11\n\tds_read_b128 %1, %7 offset:%11\n\t"
                     "ds_read_b128 %2, %8 offset:%12\n\tds_read_b128 %3, %9 offset:%12\n\t"
                     "ds_read_b128 %4, %8 offset:%13\n\tds_read_b128 %5, %9 offset:%13\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(w0[0]), "=&v"(w1[0]), "=&v"(x0[0]), "=&v"(x1[0]), "=&v"(x0[1]), "=&v"(x1[1])
                     : "v"(a), "v"(b), "v"(ax), "v"(bx), "n"(VM), "n"(OFF), "n"(XOFF), "n"(XOFF + 4096) : "memory");
    else
        asm volatile("s_waitcnt vmcnt(%12)\n\tds_read_b128 %0, %8 offset:%13\n\tds_read_b128 %1, %9 offset:%13\n\t"
                     "ds_read_b128 %2, %8 offset:%14\n\tds_read_b128 %3, %9 offset:%14\n\t"
                     "ds_read_b128 %4, %10 offset:%15\n\tds_read_b128 %5, %11 offset:%15\n\t"
                     "ds_read_b128 %6, %10 offset:%16\n\tds_read_b128 %7, %11 offset:%16\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(w0[0]), "=&v"(w1[0]), "=&v"(w0[1]), "=&v"(w1[1]), "=&v"(x0[0]), "=&v"(x1[0]), "=&v"(x0[1]), "=&v"(x1[1])
                     : "v"(a), "v"(b), "v"(ax), "v"(bx), "n"(VM), "n"(OFF), "n"(OFF + 4096), "n"(XOFF), "n"(XOFF + 4096) : "memory");
}

// XR: row quads of x staged (1, 2, 4 or 8: x rows up to 4 XR); NT: 16-row tiles of Wt; NW waves; D
// groups in flight per wave (2 or 3).
template <int DT, int XR, int NT, int NW, int D>
__global__ __launch_bounds__(64 * NW) void mfma_nt_kernel(const NtMParams p) {
    constexpr int MT = XR > 4 ? 2 : 1;               // 16-row tiles of x
    constexpr int kLoads = 4 * NT + XR;              // loads of a group per wave
    constexpr int kSlot = kLoads * kQuad;            // LDS bytes of a group
    constexpr size_t kRing = size_t(NW) * D * kSlot, kRed = size_t(NW) * NT * MT * kTilePitch * 8;
    static_assert(kRing <= 160 * 1024 && kRed <= 160 * 1024, "LDS of a CU");
    __shared__ __attribute__((aligned(256))) uint8_t smem[kRing > kRed ? kRing : kRed];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;

    // the row blocks of x over one block of Wt rows sit 8 workgroup ids apart, on one XCD
    const int bid = blockIdx.x;
    const int rb = (bid & 7) + 8 * (bid / (8 * p.mblocks));
    const int mb = (bid >> 3) % p.mblocks;
    if (rb >= p.row_blocks) return;
    const int n0 = rb * 16 * NT, m0 = mb * 4 * XR;
    const int mrows = min(4 * XR, p.M - m0);

    const __amdgpu_buffer_rsrc_t wr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(p.wt), (short)0, (int)p.w_extent, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(p.x + int64_t(m0) * p.ldx), (short)0,
        int(uint32_t((int64_t(mrows - 1) * p.ldx + (p.K + 7) / 8 * 8) * 2)), kRsrcWord3);
    // Load q of a group covers rows 4 q .. 4 q + 3, lane l the slot l % 16 of row 4 q + l / 16.  Slot c
    // of row r holds the row's chunk c ^ (r % 16), so that the 16 rows of a fragment read lie in 16
    // different 16-byte columns of LDS.
    uint32_t off[kLoads];      // byte offset of the lane's chunk in group 0; out of range past N or M
    int kc[4];                 // its first k in group 0, by row quad of a tile
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
        const bool is_w = q < 4 * NT;
        const int r = 4 * (is_w ? q : q - 4 * NT) + g;
        const int c = j ^ (r & 15);
        if (q < 4) kc[q] = 8 * c;
        const bool ok = is_w ? n0 + r < p.N : r < mrows;
        off[q] = ok ? uint32_t(is_w ? int64_t(n0 + r) * p.row_bytes : int64_t(r) * p.ldx * 2) + 16u * c : kOutOfRange;
    }
    uint8_t* const ring = smem + wave * (D * kSlot);
    auto load_group = [&](int group, uint8_t* slot) {
        const int kg = group * kMfmaNtGroup;
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const int qq = q < 4 * NT ? q & 3 : (q - 4 * NT) & 3;
            const uint32_t o = (kg + kc[qq] < p.K) ? off[q] + uint32_t(kg) * 2u : kOutOfRange;
            if (q < 4 * NT)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_void*)(slot + q * kQuad), 16, o, 0, 0, kLoadNT);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void*)(slot + q * kQuad), 16, o, 0, 0, 0);
        }
    };

    const int groups = (p.K + kMfmaNtGroup - 1) / kMfmaNtGroup;
    const int rounds = (groups + NW - 1) / NW;   // the same for every wave; groups past K are zeros
    // round r takes groups (r + start) % rounds of the walk (one past the last: nothing to load)
    const int start = (rb * p.rot) % rounds;
    auto group_of = [&](int r) {
        const int rr = r + start < rounds ? r + start : r + start - rounds;
        return r < rounds ? wave + rr * NW : groups;
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load_group(group_of(d), ring + d * kSlot);

    double sum[NT][MT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[t][mt][i] = 0.0;

    // LDS addresses of the lane's fragment of step 0: row j, chunk g; step s flips bits 6 and 7
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>((lds_void*)ring));
    const uint32_t wa = base + uint32_t(j * kRowBytes + ((g ^ j) * 16));
    const int jx = XR < 4 ? (j & (4 * XR - 1)) : j;
    const uint32_t xa = base + uint32_t(jx * kRowBytes + ((g ^ jx) * 16));

    auto consume = [&](auto dc, int r) {
        constexpr int d = decltype(dc)::value;
        constexpr int kOff = d * kSlot, kXOff = kOff + 4 * NT * kQuad;
        const int group = group_of(r);
        const bool ragged = (group + 1) * kMfmaNtGroup > p.K;
        auto half = [&](auto hc) {
            constexpr int h = decltype(hc)::value;
            i32x4 w0[NT], w1[NT], x0[MT], x1[MT];
            read_pair<(D - 1) * kLoads, NT, MT, kOff, kXOff>(w0, w1, x0, x1, wa ^ (128u * h), wa ^ (128u * h + 64u),
                                                             xa ^ (128u * h), xa ^ (128u * h + 64u));
            if (ragged) {   // clear what lies past K
                const int l0 = p.K - (group * kMfmaNtGroup + 64 * h + 8 * g), l1 = l0 - 32;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    w0[t] = keep_first(w0[t], l0);
                    w1[t] = keep_first(w1[t], l1);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    x0[mt] = keep_first(x0[mt], l0);
                    x1[mt] = keep_first(x1[mt], l1);
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    f32x4 a = mfma<DT>(w0[t], x0[mt], f32x4{0.f, 0.f, 0.f, 0.f});
                    a = mfma<DT>(w1[t], x1[mt], a);
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[t][mt][i] += double(a[i]);
                }
        };
        half(std::integral_constant<int, 0>{});
        half(std::integral_constant<int, 1>{});
        load_group(group_of(r + D), ring + kOff);
    };
    for (int r = 0; r < rounds; r += D) {
        consume(std::integral_constant<int, 0>{}, r);
        if (r + 1 < rounds) consume(std::integral_constant<int, 1>{}, r + 1);
        if constexpr (D > 2) {
            if (r + 2 < rounds) consume(std::integral_constant<int, 2>{}, r + 2);
        }
    }

    // the waves' sums through LDS (the rings' last loads have landed), lane (g, j) holding n = 4 g + i,
    // m = j of each tile
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    double* const red = reinterpret_cast<double*>(smem);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            double* dst = red + (wave * NT * MT + t * MT + mt) * kTilePitch + g * 68 + j * 4;
            *reinterpret_cast<f64x2*>(dst) = f64x2{sum[t][mt][0], sum[t][mt][1]};
            *reinterpret_cast<f64x2*>(dst + 2) = f64x2{sum[t][mt][2], sum[t][mt][3]};
        }
    __syncthreads();
    for (int o = tid; o < 16 * NT * mrows; o += 64 * NW) {
        const int nl = o % (16 * NT), ml = o / (16 * NT);
        const double* src = red + ((nl >> 4) * MT + (ml >> 4)) * kTilePitch + ((nl >> 2) & 3) * 68 + (ml & 15) * 4 + (nl & 3);
        double v = src[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += src[w * NT * MT * kTilePitch];
        if (n0 + nl < p.N) p.y[int64_t(m0 + ml) * p.ldy + n0 + nl] = float(v);
    }
}

template <int DT, int XR>
void launch_xr(const NtMParams& np, const NtMfmaPlan& q, hipStream_t s) {
    const dim3 grid(static_cast<uint32_t>(q.grid)), block(64 * kNtWaves);
    if constexpr (XR >= 4) {
        if (q.nt == 2) {
            hipLaunchKernelGGL((mfma_nt_kernel<DT, XR, 2, kNtWaves, 2>), grid, block, 0, s, np);
            return;
        }
    } else {
        if (q.depth == 3) {
            hipLaunchKernelGGL((mfma_nt_kernel<DT, XR, 1, kNtWaves, 3>), grid, block, 0, s, np);
            return;
        }
    }
    hipLaunchKernelGGL((mfma_nt_kernel<DT, XR, 1, kNtWaves, 2>), grid, block, 0, s, np);
}

}  // namespace

nmm_status launch_mfma_nt(const GemvArgs& a, const NtMfmaPlan& q, void* stream) {
    NtMParams np{};
    np.x = static_cast<const uint16_t*>(a.x);
    np.ldx = a.ldx;
    np.wt = static_cast<const uint16_t*>(a.w);
    np.row_bytes = static_cast<uint32_t>(a.ldw * 2);
    np.w_extent = static_cast<uint32_t>(((a.N - 1) * a.ldw + (a.K + 7) / 8 * 8) * 2);
    np.y = a.y;
    np.ldy = a.ldy;
    np.M = static_cast<int>(a.M);
    np.K = static_cast<int>(a.K);
    np.N = static_cast<int>(a.N);
    np.row_blocks = q.row_blocks;
    np.mblocks = q.mblocks;
    np.rot = q.rot;
    hipStream_t s = static_cast<hipStream_t>(stream);
#define NMM_NTM_XR(DTV)                              \
    do {                                             \
        switch (q.xr) {                              \
            case 1: launch_xr<DTV, 1>(np, q, s); break; \
            case 2: launch_xr<DTV, 2>(np, q, s); break; \
            case 4: launch_xr<DTV, 4>(np, q, s); break; \
            default: launch_xr<DTV, 8>(np, q, s); break; \
        }                                            \
    } while (0)
    if (a.dt == NMM_BF16) NMM_NTM_XR(NMM_BF16);
    else NMM_NTM_XR(NMM_F16);
#undef NMM_NTM_XR
    return hipGetLastError() == hipSuccess ? NMM_OK : NMM_ERR_HIP;
}

}  // namespace nmm
