// Rows of w floats read four at a time by kernels of a padded width.
#pragma once

#include <hip/hip_runtime.h>

namespace deeppcr {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// EXACT (w = the padded width): plain 16-byte loads.  Otherwise rows start on
// any 4-byte boundary: buffer loads, which the hardware bounds-checks per
// element against the `floats` given and fills with zeros beyond them.
template <bool EXACT>
struct Src {
    const float* p;
    __device__ __forceinline__ Src(const float* q, unsigned) : p(q) {}
    __device__ __forceinline__ f4 at(unsigned off) const {
        return *reinterpret_cast<const f4*>(p + off);
    }
    __device__ __forceinline__ float one(unsigned off) const { return p[off]; }
};
template <>
struct Src<false> {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Src(const float* q, unsigned floats)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(q), 0, floats * 4u, 0x00027000)) {}
    __device__ __forceinline__ f4 at(unsigned off) const {
        return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off * 4u, 0, 0));
    }
    __device__ __forceinline__ float one(unsigned off) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off * 4u, 0, 0));
    }
};

// Elements i .. i + N - 1 of the row of w starting at float `row` of src;
// zeros beyond the row's end.
template <int N, bool EXACT>
__device__ __forceinline__ void load_row(const Src<EXACT>& src, unsigned row, int i, int w,
                                         float (&v)[N]) {
#pragma unroll
    for (int q = 0; q < N; q += 4) {
        const f4 x = src.at(row + i + q);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[q + e] = EXACT || i + q + e < w ? x[e] : 0.f;
    }
}
template <int N, bool EXACT>
__device__ __forceinline__ void store_row(float* p, int i, int w, const float (&v)[N]) {
    if constexpr (EXACT) {
#pragma unroll
        for (int q = 0; q < N; q += 4)
            *reinterpret_cast<f4*>(p + i + q) = f4{v[q], v[q + 1], v[q + 2], v[q + 3]};
    } else {
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (i + q < w) p[i + q] = v[q];
    }
}

}  // namespace
}  // namespace deeppcr
