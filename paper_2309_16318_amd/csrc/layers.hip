// Layer evaluation, Jacobian assembly, Newton update and gradient kernels of
// the DeepPCR hot path.
//
// Layers (App. A.1, Eqs. 7-9, post-activation form; App. A.3 with a skip of
// length one), sigma in {tanh, logistic sigmoid, ReLU}:
//   plain    : f_l(z) = sigma(W_l z + b_l),          J_l = diag(sigma') W_l
//   residual : f_l(z) = z + alpha sigma(W_l z + b_l), J_l = I + alpha diag(sigma') W_l
#include "internal.h"

namespace deeppcr {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

__device__ inline float wave_sum(float v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ inline unsigned wave_umax(unsigned v) {
    for (int off = 32; off > 0; off >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, off, 64));
    return v;
}

// ---------------------------------------------------------------- forward
// Bound by the latency of reading W_0 and by its stores: up to 16 lanes share a
// row and the rows go out 16 bytes at a time (B 256, L 256, w 32: 15.2 us with
// a wave per row, single words and a division each, now 7.6-9; B 16, L 1024,
// w 128: 35 -> 14.7).
__global__ __launch_bounds__(kThreads) void initial_guess_kernel(
    const float* __restrict__ W, const float* __restrict__ bias, const float* __restrict__ z0,
    float* __restrict__ Z, int L, int w, int layer, float alpha, int rows_per_block) {
    const int chunks = (L + rows_per_block - 1) / rows_per_block;
    const int b = blockIdx.x / chunks;
    const int l0 = (blockIdx.x % chunks) * rows_per_block;
    const int t = threadIdx.x;
    __shared__ float zp[kMaxWidth];
    __shared__ __align__(16) float f0[kMaxWidth];
    for (int i = t; i < w; i += kThreads) zp[i] = z0[(long long)b * w + i];
    __syncthreads();
    // the lanes of a row together: as many as fit, at most 16
    int lanes = 16;
    while (lanes > 1 && lanes * w > kThreads) lanes >>= 1;
    for (int i = t / lanes; i < w; i += kThreads / lanes) {
        float acc = 0.f;
#pragma unroll 4
        for (int j = t % lanes; j < w; j += lanes) acc = fmaf(W[(long long)i * w + j], zp[j], acc);
        for (int off = lanes >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        float d;
        const float y = activate(layer, acc + bias[i], &d);
        if (t % lanes == 0) f0[i] = layer_residual(layer) ? fmaf(alpha, y, zp[i]) : y;
    }
    __syncthreads();
    const int rows = min(L, l0 + rows_per_block) - l0;
    float* out = Z + ((long long)b * L + l0) * w;
    auto repeat = [&](auto* dst, const auto* src, int n) {
        int i = t % n;
        const int step = kThreads % n;
        for (int k = t; k < rows * n; k += kThreads) {
            dst[k] = src[i];
            i += step;
            if (i >= n) i -= n;
        }
    };
    if (w % 4 == 0)
        repeat(reinterpret_cast<float4*>(out), reinterpret_cast<const float4*>(f0), w / 4);
    else
        repeat(out, f0, w);
}

__global__ __launch_bounds__(kThreads) void update_reduce_kernel(
    float* __restrict__ Z, const float* __restrict__ x, long long n, unsigned* __restrict__ red) {
    unsigned mx = 0u, mz = 0u;
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (long long)gridDim.x * kThreads) {
        const float dx = x[i];
        const float z = Z[i] + dx;
        Z[i] = z;
        mx = max(mx, __float_as_uint(fabsf(dx)));
        mz = max(mz, __float_as_uint(fabsf(z)));
    }
    mx = wave_umax(mx);
    mz = wave_umax(mz);
    __shared__ unsigned sx[kWaves], sz[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        sx[wave] = mx;
        sz[wave] = mz;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned a = sx[0], c = sz[0];
        for (int i = 1; i < kWaves; ++i) {
            a = max(a, sx[i]);
            c = max(c, sz[i]);
        }
        const int slot = blockIdx.x % kRedShards;
        atomicMax(red + kRedDZ + slot, a);
        atomicMax(red + kRedZ + slot, c);
    }
}

// --------------------------------------------------------------- backward
__global__ __launch_bounds__(kThreads) void dz0_kernel(
    const float* __restrict__ W, const float* __restrict__ dscale, const float* __restrict__ Lambda,
    float* __restrict__ dz0, int L, int w, int layer) {
    const int b = blockIdx.x;
    const int t = threadIdx.x;
    __shared__ float g[kMaxWidth];
    const float* lam = Lambda + (long long)b * L * w;  // row l = 0
    const float* dsc = dscale + (long long)b * L * w;
    for (int k = t; k < w; k += kThreads) g[k] = dsc[k] * lam[k];
    __syncthreads();
    for (int i = t; i < w; i += kThreads) {
        float acc = 0.f;
        for (int k = 0; k < w; ++k) acc = fmaf(W[(long long)k * w + i], g[k], acc);
        dz0[(long long)b * w + i] = layer_residual(layer) ? lam[i] + acc : acc;
    }
}

constexpr int kWgradBC = 32;  // batch rows staged per LDS chunk

// PRE = false: g = dscale * Lambda and the layer inputs as they are (the
// post-activation MLP of Eq. 10).  PRE = true: g = Lambda and sigma(layer
// input) with activation act (the pre-activation layers of the ResNet).
template <bool PRE>
__global__ __launch_bounds__(kThreads) void wgrad_kernel(
    const float* __restrict__ z0, const float* __restrict__ Z, const float* __restrict__ dscale,
    const float* __restrict__ Lambda, float* __restrict__ dW, float* __restrict__ db, int B, int L,
    int w, int act) {
    const int l = blockIdx.x;
    const int t = threadIdx.x;
    __shared__ float g[kWgradBC][kMaxWidth];
    __shared__ float zp[kWgradBC][kMaxWidth];
    constexpr int kAcc = kMaxWidth * kMaxWidth / kThreads;
    float acc[kAcc];
#pragma unroll
    for (int q = 0; q < kAcc; ++q) acc[q] = 0.f;
    float dbacc = 0.f;
    const int nout = w * w;
    for (int b0 = 0; b0 < B; b0 += kWgradBC) {
        const int nb = min(kWgradBC, B - b0);
        for (int idx = t; idx < nb * w; idx += kThreads) {
            const int bb = idx / w, i = idx - (idx / w) * w;
            const long long rowi = ((long long)(b0 + bb) * L + l) * w + i;
            const float zin = (l == 0) ? z0[(long long)(b0 + bb) * w + i] : Z[rowi - w];
            if constexpr (PRE) {
                float d;
                g[bb][i] = Lambda[rowi];
                zp[bb][i] = activate(2 * act, zin, &d);
            } else {
                g[bb][i] = dscale[rowi] * Lambda[rowi];
                zp[bb][i] = zin;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kAcc; ++q) {
            const int idx = t + q * kThreads;
            if (idx < nout) {
                const int i = idx / w, j = idx - (idx / w) * w;
                float a = acc[q];
                for (int bb = 0; bb < nb; ++bb) a = fmaf(g[bb][i], zp[bb][j], a);
                acc[q] = a;
            }
        }
        if (t < w) {
            for (int bb = 0; bb < nb; ++bb) dbacc += g[bb][t];
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kAcc; ++q) {
        const int idx = t + q * kThreads;
        if (idx < nout) dW[(long long)l * nout + idx] = acc[q];
    }
    if (t < w) db[(long long)l * w + t] = dbacc;
}

// The same sums for w = 16, 32, 64, 128, one workgroup per layer: thread
// (ti, tj) of a 16 x 16 grid owns the (w/16) x (w/16) tile of dW_l at rows
// ti w/16.. and columns tj w/16..; per staged batch row it reads its rows of
// g and columns of the layer input from LDS once and forms their outer
// product in registers (the index arithmetic is done once, outside the
// batch loop).
template <int W, bool PRE>
__global__ __launch_bounds__(kThreads) void wgrad_tile_kernel(
    const float* __restrict__ z0, const float* __restrict__ Z, const float* __restrict__ dscale,
    const float* __restrict__ Lambda, float* __restrict__ dW, float* __restrict__ db, int B, int L,
    int act) {
    constexpr int RT = W / 16;  // rows and columns of the tile of a thread
    const int l = blockIdx.x;
    const int t = threadIdx.x;
    const int i0 = (t >> 4) * RT, j0 = (t & 15) * RT;
    __shared__ float g[kWgradBC][W];
    __shared__ float zp[kWgradBC][W];
    float acc[RT][RT];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int c = 0; c < RT; ++c) acc[a][c] = 0.f;
    float dbacc = 0.f;
    for (int b0 = 0; b0 < B; b0 += kWgradBC) {
        const int nb = min(kWgradBC, B - b0);
        for (int idx = t; idx < nb * W; idx += kThreads) {
            const int bb = idx / W, i = idx % W;
            const long long rowi = ((long long)(b0 + bb) * L + l) * W + i;
            const float zin = (l == 0) ? z0[(long long)(b0 + bb) * W + i] : Z[rowi - W];
            if constexpr (PRE) {
                float d;
                g[bb][i] = Lambda[rowi];
                zp[bb][i] = activate(2 * act, zin, &d);
            } else {
                g[bb][i] = dscale[rowi] * Lambda[rowi];
                zp[bb][i] = zin;
            }
        }
        __syncthreads();
        for (int bb = 0; bb < nb; ++bb) {
            float gi[RT], zj[RT];
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                gi[a] = g[bb][i0 + a];
                zj[a] = zp[bb][j0 + a];
            }
#pragma unroll
            for (int a = 0; a < RT; ++a)
#pragma unroll
                for (int c = 0; c < RT; ++c) acc[a][c] = fmaf(gi[a], zj[c], acc[a][c]);
        }
        if (t < W)
            for (int bb = 0; bb < nb; ++bb) dbacc += g[bb][t];
        __syncthreads();
    }
    float* dWl = dW + (long long)l * W * W;
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int c = 0; c < RT; ++c) dWl[(i0 + a) * W + j0 + c] = acc[a][c];
    if (t < W) db[(long long)l * W + t] = dbacc;
}

// The same sums for w <= 8: one thread per element (l, i, j) of dW (and of db
// for j = 0), the batch summed in the same order, so the results equal
// wgrad_kernel's.
template <bool PRE>
__global__ __launch_bounds__(kThreads) void wgrad_small_kernel(
    const float* __restrict__ z0, const float* __restrict__ Z, const float* __restrict__ dscale,
    const float* __restrict__ Lambda, float* __restrict__ dW, float* __restrict__ db, int B, int L,
    int w, int act) {
    const long long o = (long long)blockIdx.x * kThreads + threadIdx.x;  // (l w + i) w + j
    if (o >= (long long)L * w * w) return;
    const int j = (int)(o % w);
    const long long li = o / w;
    const int i = (int)(li % w);
    const long long l = li / w;
    float acc = 0.f, dbacc = 0.f;
    for (int b = 0; b < B; ++b) {
        const long long row = ((long long)b * L + l) * w;
        const float gi = PRE ? Lambda[row + i] : dscale[row + i] * Lambda[row + i];
        const float zin = (l == 0) ? z0[(long long)b * w + j] : Z[row - w + j];
        float zpj = zin;
        if constexpr (PRE) {
            float d;
            zpj = activate(2 * act, zin, &d);
        }
        acc = fmaf(gi, zpj, acc);
        dbacc += gi;
    }
    dW[o] = acc;
    if (j == 0) db[l * w + i] = dbacc;
}

__global__ __launch_bounds__(kThreads) void residual_kernel(const float* __restrict__ F,
                                                           const float* __restrict__ Z,
                                                           float* __restrict__ r, long long n,
                                                           unsigned* __restrict__ red) {
    // four elements per thread and step, one atomic per workgroup of at most
    // 1024: a wave's atomic each for one element per thread took 22 us at
    // n = 2^20 (the slots share 16 cache lines), against 4 for the data
    typedef float v4 __attribute__((ext_vector_type(4)));
    unsigned mr = 0u;
    const long long n4 = n / 4;
    const long long step = (long long)gridDim.x * kThreads;
    const long long k0 = (long long)blockIdx.x * kThreads + threadIdx.x;
    for (long long k = k0; k < n4; k += step) {
        const v4 v = reinterpret_cast<const v4*>(F)[k] - reinterpret_cast<const v4*>(Z)[k];
        reinterpret_cast<v4*>(r)[k] = v;
#pragma unroll
        for (int e = 0; e < 4; ++e) mr = max(mr, __float_as_uint(fabsf(v[e])));
    }
    for (long long k = 4 * n4 + k0; k < n; k += step) {
        const float v = F[k] - Z[k];
        r[k] = v;
        mr = max(mr, __float_as_uint(fabsf(v)));
    }
    mr = wave_umax(mr);
    __shared__ unsigned sr[kWaves];
    if ((threadIdx.x & 63) == 0) sr[threadIdx.x >> 6] = mr;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kWaves; ++i) mr = max(mr, sr[i]);
        atomicMax(red + kRedF + (int)(blockIdx.x % kRedShards), mr);
    }
}

__global__ __launch_bounds__(kThreads) void zero_words_kernel(unsigned* __restrict__ p, int n) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// The Newton stopping measures for the host: max |dZ|, max |Z| and max |F|,
// each the max over its kRedShards slots, go to out[0..2], then seq to
// out[3] after a system-scope fence, so that a host that reads seq in out[3]
// (host-mapped memory) also reads the maxima.  One workgroup of kRedShards
// threads, one slot of each measure per thread.
__global__ __launch_bounds__(kRedShards) void measures_kernel(const unsigned* __restrict__ red,
                                                              unsigned* out, unsigned seq) {
    __shared__ unsigned part[3][kRedShards / 64];
    const int t = threadIdx.x;
    unsigned v[3] = {red[kRedDZ + t], red[kRedZ + t], red[kRedF + t]};
#pragma unroll
    for (int j = 0; j < 3; ++j)
        for (int off = 32; off > 0; off >>= 1) v[j] = max(v[j], (unsigned)__shfl_xor((int)v[j], off, 64));
    if ((t & 63) == 0)
        for (int j = 0; j < 3; ++j) part[j][t >> 6] = v[j];
    __syncthreads();
    if (t == 0) {
        for (int j = 0; j < 3; ++j) {
            unsigned m = part[j][0];
            for (int q = 1; q < kRedShards / 64; ++q) m = max(m, part[j][q]);
            out[j] = m;
        }
        __threadfence_system();
        __hip_atomic_store(out + 3, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ __launch_bounds__(kThreads) void copy_rows_kernel(VecSrc src, VecDst dst, int L, int w) {
    const long long row = blockIdx.x;
    const int l = (int)(row % L);
    const int b = (int)(row / L);
    const float* s = src.base + b * src.bstride + (long long)l * src.rstride;
    float* d = dst.base + b * dst.bstride + (long long)l * dst.rstride;
    for (int i = threadIdx.x; i < w; i += kThreads) d[i] = s[i];
}

}  // namespace

hipError_t launch_forward_eval(const float* W, const float* bias, const float* z0,
                               const float* Z, float* A, float* r, unsigned* red,
                               int B, int L, int w, int layer, float alpha,
                               hipStream_t stream) {
    if (small_width(w))
        return launch_eval_small(false, W, bias, z0, Z, nullptr, A, r, nullptr, red, B, L, w,
                                 layer, alpha, stream);
    if (!wide_width(w)) return hipErrorInvalidValue;
    return launch_forward_eval_wide(W, bias, z0, Z, A, r, red, B, L, w, layer, alpha, stream);
}

hipError_t launch_initial_guess(const float* W, const float* bias, const float* z0, float* Z,
                                int B, int L, int w, int layer, float alpha,
                                hipStream_t stream) {
    if (wide_width(w))
        return launch_initial_guess_wide(W, bias, z0, Z, B, L, w, layer, alpha, stream);
    const int rows_per_block = 64;
    const int chunks = (L + rows_per_block - 1) / rows_per_block;
    hipLaunchKernelGGL(initial_guess_kernel, dim3((unsigned)((long long)B * chunks)),
                       dim3(kThreads), 0, stream, W, bias, z0, Z, L, w, layer, alpha,
                       rows_per_block);
    return hipGetLastError();
}

hipError_t launch_update_reduce(float* Z, const float* x, long long n, unsigned* red,
                                hipStream_t stream) {
    long long blocks = (n + kThreads * 8 - 1) / (kThreads * 8);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(update_reduce_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, Z,
                       x, n, red);
    return hipGetLastError();
}

hipError_t launch_backward_assemble(const float* W, const float* bias, const float* z0,
                                    const float* Z, const float* G, float* A, float* rrev,
                                    float* dscale, int B, int L, int w, int layer,
                                    float alpha, hipStream_t stream) {
    if (small_width(w))
        return launch_eval_small(true, W, bias, z0, Z, G, A, rrev, dscale, nullptr, B, L, w,
                                 layer, alpha, stream);
    if (!wide_width(w)) return hipErrorInvalidValue;
    return launch_backward_assemble_wide(W, bias, z0, Z, G, A, rrev, dscale, B, L, w, layer,
                                         alpha, stream);
}

hipError_t launch_dz0(const float* W, const float* dscale, const float* Lambda, float* dz0,
                      int B, int L, int w, int layer, hipStream_t stream) {
    if (wide_width(w)) return launch_dz0_wide(W, dscale, Lambda, dz0, B, L, w, layer, stream);
    hipLaunchKernelGGL(dz0_kernel, dim3((unsigned)B), dim3(kThreads), 0, stream, W, dscale,
                       Lambda, dz0, L, w, layer);
    return hipGetLastError();
}

template <bool PRE>
hipError_t launch_wgrad_any(const float* z0, const float* Z, const float* dscale,
                            const float* Lambda, float* dW, float* db, int B, int L, int w,
                            int act, hipStream_t stream) {
    const dim3 grid((unsigned)L), blk(kThreads);
    switch (w) {
        case 16: hipLaunchKernelGGL((wgrad_tile_kernel<16, PRE>), grid, blk, 0, stream, z0, Z, dscale, Lambda, dW, db, B, L, act); break;
        case 32: hipLaunchKernelGGL((wgrad_tile_kernel<32, PRE>), grid, blk, 0, stream, z0, Z, dscale, Lambda, dW, db, B, L, act); break;
        case 64: hipLaunchKernelGGL((wgrad_tile_kernel<64, PRE>), grid, blk, 0, stream, z0, Z, dscale, Lambda, dW, db, B, L, act); break;
        case 128: hipLaunchKernelGGL((wgrad_tile_kernel<128, PRE>), grid, blk, 0, stream, z0, Z, dscale, Lambda, dW, db, B, L, act); break;
        default:
            if (w <= 8) {
                const long long n = (long long)L * w * w;
                hipLaunchKernelGGL((wgrad_small_kernel<PRE>), dim3((unsigned)((n + kThreads - 1) / kThreads)), blk, 0, stream, z0, Z, dscale, Lambda, dW, db, B, L, w, act);
            } else {
                hipLaunchKernelGGL((wgrad_kernel<PRE>), grid, blk, 0, stream, z0, Z, dscale, Lambda, dW, db, B, L, w, act);
            }
            break;
    }
    return hipGetLastError();
}

hipError_t launch_wgrad(const float* z0, const float* Z, const float* dscale,
                        const float* Lambda, float* dW, float* db, int B, int L, int w,
                        hipStream_t stream) {
    if (wide_width(w)) return launch_wgrad_wide(z0, Z, dscale, Lambda, dW, db, B, L, w, stream);
    return launch_wgrad_any<false>(z0, Z, dscale, Lambda, dW, db, B, L, w, 0, stream);
}

hipError_t launch_wgrad_pre(const float* z0, const float* Z, const float* Lambda, float* dW,
                            float* db, int B, int L, int w, int act, hipStream_t stream) {
    return launch_wgrad_any<true>(z0, Z, nullptr, Lambda, dW, db, B, L, w, act, stream);
}

hipError_t launch_residual(const float* F, const float* Z, float* r, long long n, unsigned* red,
                           hipStream_t stream) {
    long long blocks = (n + 4 * kThreads - 1) / (4 * kThreads);
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(residual_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, F, Z, r,
                       n, red);
    return hipGetLastError();
}

hipError_t launch_zero_words(unsigned* p, int n, hipStream_t stream) {
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, stream, p, n);
    return hipGetLastError();
}

hipError_t launch_measures(const unsigned* red, unsigned* out, unsigned seq, hipStream_t stream) {
    hipLaunchKernelGGL(measures_kernel, dim3(1), dim3(kRedShards), 0, stream, red, out, seq);
    return hipGetLastError();
}

hipError_t launch_copy_rows(const VecSrc& src, const VecDst& dst, int B, int L, int w,
                            hipStream_t stream) {
    hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)((long long)B * L)), dim3(kThreads), 0,
                       stream, src, dst, L, w);
    return hipGetLastError();
}

}  // namespace deeppcr
