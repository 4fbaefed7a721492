// Four consecutive columns of one output row.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bf16_cast.h"

namespace nmm {

// Whether the fp32 rows and the bf16 rows of an output take one wide store per four columns: only
// where every row starts on that boundary (the ABI asks for 4- and 2-byte alignment only).
__host__ __device__ __forceinline__ bool wide_f32(const float* y, int64_t ldy, int64_t sy) {
    return ((reinterpret_cast<uintptr_t>(y) | uintptr_t(ldy * 4) | uintptr_t(sy * 4)) & 15u) == 0;
}
__host__ __device__ __forceinline__ bool wide_bf16(const uint16_t* y, int64_t ldy, int64_t sy) {
    return ((reinterpret_cast<uintptr_t>(y) | uintptr_t(ldy * 2) | uintptr_t(sy * 2)) & 7u) == 0;
}

// v to row[n .. n + 3], columns at or past N left alone.
__device__ __forceinline__ void put4(float* row, int n, int N, const float (&v)[4], bool wide) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    if (wide && n + 4 <= N) {
        *reinterpret_cast<f32x4*>(row + n) = f32x4{v[0], v[1], v[2], v[3]};
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (n + i < N) row[n + i] = v[i];
}
__device__ __forceinline__ void put4(uint16_t* row, int n, int N, const float (&v)[4], int away, bool wide) {
    uint16_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = to_bf16_mode(v[i], away);
    if (wide && n + 4 <= N) {
        *reinterpret_cast<uint2*>(row + n) =
            uint2{uint32_t(h[0]) | (uint32_t(h[1]) << 16), uint32_t(h[2]) | (uint32_t(h[3]) << 16)};
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (n + i < N) row[n + i] = h[i];
}

}  // namespace nmm
