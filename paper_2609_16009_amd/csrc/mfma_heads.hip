// Batched narrow MatMul on the matrix cores (gfx950): y_b[M,N] = x_b[M,K] . W_b[K,N] for the per-head
// products of several tokens, W_b row-major, fp32 (and optionally bf16) out.
//
// The streaming GEMV spends 2 M flops a weight on the vector units and reads x from LDS for every
// row: 128 heads x [4, 128] . [128, 512] took 8.8 us and 16 rows 21.3, against 6.1 us for one row.  Here
//  * A workgroup (4 waves) owns 64 columns of one matrix and all of K, so nothing is handed over
//    between workgroups and no workspace is needed; its waves take groups of 32 rows in turn.
//  * A group's W rows (4 KB) and its 32 k of x go to a ring in LDS private to the wave, by LDS-direct
//    loads of 8 rows x 128 bytes: no barrier in the loop, D groups in flight per wave (all of a head's,
//    up to K = 512).  The 16-byte chunks of a row are permuted so that the reads have no bank conflict.
//  * The A operand of v_mfma_f32_16x16x32 is W transposed, read by ds_read_b64_tr_b16, gfx950's
//    transposing LDS read (an operand needs 8 consecutive k of one column; W rows hold consecutive
//    columns); x is the B operand, so a lane ends with 4 consecutive n of one m.
//  * Sums: every MFMA starts from zero and is added in fp64 (the vector units are idle); the waves'
//    sums, rounded to fp32, meet in LDS.  Relative 2-norm error 3.9e-8 to 4.7e-8 in bf16 and 5.1e-8 to 5.7e-8
//    in fp16 (fp32 FMAs: 5e-8 to 7e-8).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "nmm_internal.h"
#include "out4.h"

namespace nmm {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kRsrcWord3 = 0x00020000;
constexpr int kLoadNT = 2;
constexpr uint32_t kOutOfRange = 0x80000000u;
constexpr int kGroup = 32;                      // rows of W per group
constexpr int kRowBytes = kHeadsCols * 2;       // bytes of a panel's row: 8 chunks
constexpr int kWLoads = kGroup / 8;             // LDS-direct loads of a group's W rows (8 rows each)
constexpr int kLoadBytes = 1024;
constexpr int kTiles = kHeadsCols / 16;         // 16-column tiles of a panel
constexpr int kTilePitch = 4 * 68;              // floats of one 16 x 16 tile in LDS: [g][j][i], padded per g
constexpr int kQuads = kHeadsCols / 4;      // 4-column pieces of a panel's row

struct HParams {
    const uint16_t* x;
    int64_t ldx, sx;
    const uint16_t* w;
    int64_t sw;
    float* y;              // fp32 output (may be null when ybf is set)
    int64_t ldy, sy;
    uint16_t* ybf;         // optional bf16 output, ybf[b * ybf_sb + m * ldyb + n]
    int64_t ldyb, ybf_sb;
    int away;              // bf16 rounding: 0 nearest-even, 1 ties away from zero
    int M, K, N;
    uint32_t row_bytes, w_extent;
    int panels, mblocks;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, kRsrcWord3);
}

template <int DT>
__device__ __forceinline__ f32x4 mfma(i32x4 a, i32x4 b) {
    const f32x4 c = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (DT == NMM_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Fragments from LDS: once at most VM of the wave's loads are outstanding, the transposed fragments of
// four column tiles (halves of 4 k each at a0 .. a3, OFF and OFF + 4 rows), complete when this
// returns.  The loads that fill LDS are LDS-direct: the compiler would wait for all of them before any
// read that may alias, so the wait and the reads are written out.
template <int VM, int OFF>
__device__ __forceinline__ void read_w4(i32x4 (&w)[4], uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3) {
    static_assert(VM < 64 && OFF + 4 * kRowBytes < 65536, "immediate fields");
    u32x2 l0, l1, l2, l3, h0, h1, h2, h3;
    asm volatile("s_waitcnt vmcnt(%12)\n\t"
                 "ds_read_b64_tr_b16 %0, %8 offset:%13\n\tds_read_b64_tr_b16 %1, %8 offset:%14\n\t"
                 "ds_read_b64_tr_b16 %2, %9 offset:%13\n\tds_read_b64_tr_b16 %3, %9 offset:%14\n\t"
                 "ds_read_b64_tr_b16 %4, %10 offset:%13\n\tds_read_b64_tr_b16 %5, %10 offset:%14\n\t"
                 "ds_read_b64_tr_b16 %6, %11 offset:%13\n\tds_read_b64_tr_b16 %7, %11 offset:%14\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(l0), "=&v"(h0), "=&v"(l1), "=&v"(h1), "=&v"(l2), "=&v"(h2), "=&v"(l3), "=&v"(h3)
                 : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(VM), "n"(OFF), "n"(OFF + 4 * kRowBytes) : "memory");
    w[0] = i32x4{int(l0.x), int(l0.y), int(h0.x), int(h0.y)};
    w[1] = i32x4{int(l1.x), int(l1.y), int(h1.x), int(h1.y)};
    w[2] = i32x4{int(l2.x), int(l2.y), int(h2.x), int(h2.y)};
    w[3] = i32x4{int(l3.x), int(l3.y), int(h3.x), int(h3.y)};
}

// The x fragments of a group, likewise.
template <int VM, int OFF, int MT>
__device__ __forceinline__ void read_x(i32x4 (&x)[MT], uint32_t a) {
    static_assert(VM < 64 && OFF + MT * kLoadBytes < 65536, "immediate fields");
    if constexpr (MT == 1)
        asm volatile("s_waitcnt vmcnt(%2)\n\tds_read_b128 %0, %1 offset:%3\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(x[0]) : "v"(a), "n"(VM), "n"(OFF) : "memory");
    else
        asm volatile("s_waitcnt vmcnt(%3)\n\tds_read_b128 %0, %2 offset:%4\n\tds_read_b128 %1, %2 offset:%5\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(x[0]), "=&v"(x[1]) : "v"(a), "n"(VM), "n"(OFF), "n"(OFF + kLoadBytes) : "memory");
}

template <int DT, int MT, int D, bool BF>
__global__ __launch_bounds__(kThreads) void mfma_heads_kernel(const HParams p) {
    constexpr int kLoads = kWLoads + MT;            // loads of a group per wave
    constexpr int kSlot = kLoads * kLoadBytes;      // LDS bytes of a group
    constexpr int kRing = kWaves * D * kSlot, kRed = kWaves * kTiles * MT * kTilePitch * 4;
    __shared__ __attribute__((aligned(256))) uint8_t smem[kRing > kRed ? kRing : kRed];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, j = lane & 15;

    const uint32_t bid = blockIdx.x;
    const int panel = static_cast<int>(bid % uint32_t(p.panels));
    const uint32_t bm = bid / uint32_t(p.panels);
    const int mb = static_cast<int>(bm % uint32_t(p.mblocks));
    const int64_t b = bm / uint32_t(p.mblocks);
    const int m0 = mb * 16 * MT, n0 = panel * kHeadsCols;
    const int groups = (p.K + kGroup - 1) / kGroup;
    const int rounds = (groups + kWaves - 1) / kWaves;   // the same for every wave; rows past K are zeros
    const int mrows = min(16 * MT, p.M - m0);

    // W: load q of a group covers rows 8 q .. 8 q + 7, lane l the slot l % 8 of row 8 q + l / 8.  Slot s of
    // row r holds the row's chunk s ^ f(r), f(r) = 2 ((r >> 1 & 1) + 2 (r >> 3 & 1)): the 8 rows x 32
    // bytes of half a transposing read lie in 16 different 16-byte columns.
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.w + b * p.sw, p.w_extent);
    const int chunks_valid = min(8, (p.N - n0 + 7) / 8);
    const int wr0 = lane >> 3;
    uint32_t w_off[2];      // byte offset of the lane's chunk in row wr0 of the matrix, by q & 1
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int c = (lane & 7) ^ (2 * (((wr0 >> 1) & 1) + 2 * h));
        w_off[h] = c < chunks_valid ? uint32_t(wr0) * p.row_bytes + uint32_t(n0) * 2u + 16u * c : kOutOfRange;
    }
    // x: load t covers rows 16 t + l / 4 of the tile, slot l % 4; slot s of row r holds the chunk
    // s ^ (r >> 2 & 3) of its 32 k.  Rows past M read zeros.
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x + b * p.sx + int64_t(m0) * p.ldx,
                                                uint32_t((int64_t(mrows - 1) * p.ldx + (p.K + 7) / 8 * 8) * 2));
    const int xr0 = lane >> 2, xc = (lane & 3) ^ ((xr0 >> 2) & 3);
    uint32_t x_off[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
        x_off[t] = 16 * t + xr0 < mrows ? uint32_t((int64_t(16 * t + xr0) * p.ldx + 8 * xc) * 2) : kOutOfRange;

    uint8_t* const ring = smem + wave * (D * kSlot);
    auto load_group = [&](int r, uint8_t* slot) {
        const int k = (wave + r * kWaves) * kGroup;
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            const uint32_t o = x_off[t] == kOutOfRange || k + 8 * xc >= p.K ? kOutOfRange : x_off[t] + uint32_t(k) * 2u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void*)(slot + (kWLoads + t) * kLoadBytes), 16, o, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < kWLoads; ++q) {
            const uint32_t o = w_off[q & 1] == kOutOfRange || k + 8 * q + wr0 >= p.K ? kOutOfRange
                                                                                  : w_off[q & 1] + uint32_t(k + 8 * q) * p.row_bytes;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_void*)(slot + q * kLoadBytes), 16, o, 0, 0, kLoadNT);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load_group(d, ring + d * kSlot);

    double sum[kTiles][MT][4];
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[t][mt][i] = 0.0;

    // LDS addresses of the lane's fragments: row 8 g + j / 4 (and 4 rows on), columns 4 (j % 4) .. + 3 of
    // a tile; tile t flips bits 5 and 6.  x: row j, chunk g.
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>((lds_void*)ring));
    const uint32_t wa = base + uint32_t((8 * g + (j >> 2)) * kRowBytes + 16 * ((2 * ((j >> 3) + 2 * (g & 1))) ^ ((j & 3) >> 1)) + 8 * (j & 1));
    const uint32_t xa = base + uint32_t(kWLoads * kLoadBytes + j * 64 + 16 * (g ^ ((j >> 2) & 3)));

    auto consume = [&](auto dc, int r) {
        constexpr int d = decltype(dc)::value, kOff = d * kSlot, kWait = (D - 1) * kLoads;
        i32x4 xf[MT];
        read_x<kWait, kOff, MT>(xf, xa);
        const int left = p.K - ((wave + r * kWaves) * kGroup + 8 * g);
        if ((p.K & 7) != 0 && (wave + r * kWaves + 1) * kGroup > p.K) {   // clear the chunk that holds K past it
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int e = 0; e < 4; ++e) xf[mt][e] &= (2 * e + 1 < left) ? -1 : (2 * e < left ? 0x0000FFFF : 0);
        }
#pragma unroll
        for (int t0 = 0; t0 < kTiles; t0 += 4) {
            i32x4 wf[4];
            read_w4<kWait, kOff>(wf, wa ^ (32u * t0), wa ^ (32u * (t0 + 1)), wa ^ (32u * (t0 + 2)), wa ^ (32u * (t0 + 3)));
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const f32x4 a = mfma<DT>(wf[t], xf[mt]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[t0 + t][mt][i] += double(a[i]);
                }
        }
        load_group(r + D, ring + kOff);
    };
    for (int r = 0; r < rounds; r += D) {
        consume(std::integral_constant<int, 0>{}, r);
        if constexpr (D > 1) {
            if (r + 1 < rounds) consume(std::integral_constant<int, 1>{}, r + 1);
        }
        if constexpr (D > 2) {
            if (r + 2 < rounds) consume(std::integral_constant<int, 2>{}, r + 2);
            if (r + 3 < rounds) consume(std::integral_constant<int, 3>{}, r + 3);
        }
    }

    // ---- the waves' sums through LDS (the rings' last loads have landed): lane (g, j) holds columns
    // 4 g .. + 3 of row j of each tile
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<f32x4*>(red + ((wave * kTiles + t) * MT + mt) * kTilePitch + g * 68 + j * 4) =
                f32x4{float(sum[t][mt][0]), float(sum[t][mt][1]), float(sum[t][mt][2]), float(sum[t][mt][3])};
    __syncthreads();
    // output piece o: columns 4 (o % kQuads) .. + 3 of row o / kQuads
    const int n_out = mrows * kQuads;
    const bool wide = wide_f32(p.y, p.ldy, p.sy), wide_b = BF && wide_bf16(p.ybf, p.ldyb, p.ybf_sb);
    for (int o = tid; o < n_out; o += kThreads) {
        const int ml = o / kQuads, q = o % kQuads;
        const float* src = red + ((q >> 2) * MT + (ml >> 4)) * kTilePitch + (q & 3) * 68 + (ml & 15) * 4;
        double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(src + w * kTiles * MT * kTilePitch);
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] += double(v[i]);
        }
        const float v[4] = {float(s[0]), float(s[1]), float(s[2]), float(s[3])};
        const int m = m0 + ml, n = n0 + 4 * q;
        if (!BF || p.y) put4(p.y + b * p.sy + int64_t(m) * p.ldy, n, p.N, v, wide);
        if constexpr (BF) put4(p.ybf + b * p.ybf_sb + int64_t(m) * p.ldyb, n, p.N, v, p.away, wide_b);
    }
}

template <int DT, int MT, int D>
void launch_mt(const HParams& mp, int64_t grid, hipStream_t s) {
    if (mp.ybf)
        hipLaunchKernelGGL((mfma_heads_kernel<DT, MT, D, true>), dim3(static_cast<uint32_t>(grid)), dim3(kThreads), 0, s, mp);
    else
        hipLaunchKernelGGL((mfma_heads_kernel<DT, MT, D, false>), dim3(static_cast<uint32_t>(grid)), dim3(kThreads), 0, s, mp);
}

template <int DT, int MT>
void launch_d(const HParams& mp, int64_t grid, hipStream_t s) {
    // groups in flight per wave: all of them up to four
    const int rounds = (mp.K + kGroup * kWaves - 1) / (kGroup * kWaves);
    if (rounds == 1) launch_mt<DT, MT, 1>(mp, grid, s);
    else if (rounds == 2) launch_mt<DT, MT, 2>(mp, grid, s);
    else launch_mt<DT, MT, 4>(mp, grid, s);
}

}  // namespace

nmm_status launch_mfma_heads(const GemvArgs& a, void* stream) {
    HParams mp{};
    mp.x = static_cast<const uint16_t*>(a.x);
    mp.ldx = a.ldx;
    mp.sx = a.sx;
    mp.w = static_cast<const uint16_t*>(a.w);
    mp.sw = a.sw;
    mp.y = a.y;
    mp.ldy = a.ldy;
    mp.sy = a.sy;
    mp.ybf = static_cast<uint16_t*>(a.ybf);
    mp.ldyb = a.ybf_ldm;
    mp.ybf_sb = a.ybf_sb;
    mp.away = a.ybf_away;
    mp.M = static_cast<int>(a.M);
    mp.K = static_cast<int>(a.K);
    mp.N = static_cast<int>(a.N);
    mp.row_bytes = static_cast<uint32_t>(a.ldw * 2);
    mp.w_extent = static_cast<uint32_t>(((a.K - 1) * a.ldw + (a.N + 7) / 8 * 8) * 2);
    const int mt = a.M <= 16 ? 16 : 32;
    mp.panels = static_cast<int>((a.N + kHeadsCols - 1) / kHeadsCols);
    mp.mblocks = static_cast<int>((a.M + mt - 1) / mt);
    const int64_t grid = a.batch * mp.mblocks * mp.panels;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (a.dt == NMM_BF16) {
        if (mt == 16) launch_d<NMM_BF16, 1>(mp, grid, s);
        else launch_d<NMM_BF16, 2>(mp, grid, s);
    } else {
        if (mt == 16) launch_d<NMM_F16, 1>(mp, grid, s);
        else launch_d<NMM_F16, 2>(mp, grid, s);
    }
    return hipGetLastError() == hipSuccess ? NMM_OK : NMM_ERR_HIP;
}

}  // namespace nmm
