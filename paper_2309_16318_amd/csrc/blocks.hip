// The block-bidiagonal solve of Eq. 3 on stored blocks, widths 4 to 128, by
// reduction over row chunks: the cyclic reduction of Sec. 3 with chunks of m
// rows in the place of pairs.
//
//   block_up    for every chunk but the last, x_end = P x_in + q: q by
//               substitution from x_in = 0 and, in every chunk but the
//               first, P as the product of the chunk's blocks;
//   the chunk ends are a system of the same form with 1/m of the rows,
//               reduced again or, once short, substituted by block_down;
//   block_down  substitution inside every chunk from its x_in.
//
// A block is read twice, and one block product is formed per row; the PCR
// levels read and write every block once per pair of levels and form a
// product per row and level.
//
// Widths are padded to WP = 16, 32, 64 or 128.  All products are float32
// MFMAs whose operands need no rearrangement: a lane of v_mfma_f32_16x16x4
// (32x32x2) holds rows 4 g + e (8 q + 4 h + e) of its column of a result, and
// as the right operand of the next product it supplies just these rows if
// instruction e (4 q + e) takes k = 4 g + e (8 q + 4 h + e), which the left
// operand's 16-byte loads of the block's rows match.  So the running product
// never leaves its registers, and a wave needs no other wave's columns.
#include "internal.h"
#include "rows.h"
#include "strip.h"

#include <type_traits>

namespace deeppcr {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));

template <bool EXACT>
__device__ __forceinline__ Src<EXACT> block_at(const BlockSrc& A, int b, int m, int w) {
    return Src<EXACT>(A.base + b * A.bstride + (long long)m * A.rstride, (unsigned)(w * w));
}

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f16v mfma2(float a, float b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

template <int I, int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<I + 1, N>(f);
    }
}

// ---------------------------------------------------------------- w <= 16
// One wave per chunk, the next 8 rows' blocks and right-hand sides requested
// ahead (one 16-byte piece of each per lane).
constexpr int kAhead16 = 8;

// rows 4 g .. 4 g + 3 of a vector
template <bool EXACT>
__device__ __forceinline__ f4 vec16(const float* p, int w, int g) {
    if constexpr (EXACT) return *reinterpret_cast<const f4*>(p + 4 * g);
    f4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = p[4 * g + e < w ? 4 * g + e : 0];
        v[e] = 4 * g + e < w ? x : 0.f;
    }
    return v;
}
template <bool EXACT>
__device__ __forceinline__ void put16(float* p, int w, int g, f4 v) {
    if constexpr (EXACT) {
        *reinterpret_cast<f4*>(p + 4 * g) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (4 * g + e < w) p[4 * g + e] = v[e];
    }
}

// LAYER: the blocks of MLP layers formed from the weights A (shared by the
// systems) and d, J = diag(d) W (+ I), instead of stored ones; transposed,
// only row 0 has a right-hand side.
template <bool TRANS, bool EXACT, bool LAYER>
__device__ __forceinline__ f4 block16(const BlockSrc& A, const LayerScale& y, int b, int m, int w,
                                      int i, int g) {
    const Src<EXACT> s = block_at<EXACT>(A, b, m, w);
    f4 v;
    if constexpr (!TRANS) {
        v = s.at(i * w + 4 * g);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = s.one((4 * g + e) * w + i);
    }
    if constexpr (!EXACT)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (TRANS ? i : 4 * g + e) < w ? v[e] : 0.f;
    if constexpr (LAYER) {
        const float* d = y.d + b * y.bstride + m * y.rstride;
        const float di = TRANS ? 0.f : d[EXACT || i < w ? i : 0];
        f4 dk = {di, di, di, di};
        if constexpr (TRANS) dk = vec16<EXACT>(d, w, g);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = fmaf(dk[e], v[e], y.residual && 4 * g + e == i ? 1.f : 0.f);
    }
    return v;
}
// A x in two halves, the order of least rounding (the right-hand side, the
// largest term as a rule, is added last) and of the shorter dependent chain.
__device__ __forceinline__ f4 product16(f4 a, f4 x) {
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const f4 s0 = mfma4(a[1], x[1], mfma4(a[0], x[0], zero));
    const f4 s1 = mfma4(a[3], x[3], mfma4(a[2], x[2], zero));
    return s0 + s1;
}

template <bool TRANS, bool EXACT, bool LAYER>
__global__ __launch_bounds__(64) void block_up16(BlockSrc A, LayerScale y, VecSrc r,
                                                 float* __restrict__ P, float* __restrict__ q,
                                                 int L, int w_, int Lc, int C) {
    constexpr int NB = kAhead16;
    const int w = EXACT ? 16 : w_;
    const int lane = threadIdx.x, i = lane & 15, g = lane >> 4;
    const int c = blockIdx.x % (C - 1), b = blockIdx.x / (C - 1);
    const int m0 = c * Lc, m1 = min(L, m0 + Lc);
    const float* rb = r.base + b * r.bstride;
    f4 x = {0.f, 0.f, 0.f, 0.f}, p;
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = 4 * g + e == i ? 1.f : 0.f;
    int m = m0;
    if (c == 0) x = vec16<EXACT>(rb + (long long)(m++) * r.rstride, w, g);
    f4 a[NB], rr[NB];
    auto request = [&](int row, int s) {
        const int mm = min(row, m1 - 1);
        a[s] = block16<TRANS, EXACT, LAYER>(A, y, b, mm, w, i, g);
        if constexpr (LAYER && TRANS)
            rr[s] = f4{0.f, 0.f, 0.f, 0.f};
        else
            rr[s] = vec16<EXACT>(rb + (long long)mm * r.rstride, w, g);
    };
    if (m < m1)
#pragma unroll
        for (int s = 0; s < NB; ++s) request(m + s, s);
    for (; m < m1; m += NB) {
#pragma unroll
        for (int s = 0; s < NB; ++s) {
            if (m + s >= m1) break;
            if (c > 0) {
                f4 pn = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e) pn = mfma4(a[s][e], p[e], pn);
                p = pn;
            }
            x = rr[s] + product16(a[s], x);
            request(m + s + NB, s);
        }
    }
    const long long o = (long long)b * (C - 1) + c;
    if (i == 0) put16<EXACT>(q + o * w, w, g, x);
    if (c > 0 && i < w)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (EXACT || 4 * g + e < w) P[o * w * w + (4 * g + e) * w + i] = p[e];
}

// UPD: out is the Newton iterate; the solution is added to it and max |x|,
// max |Z + x| go to the kRedDZ, kRedZ slots of red.
__device__ __forceinline__ void reduce_maxima(unsigned* red, unsigned mx, unsigned mz) {
    for (int off = 32; off > 0; off >>= 1) {
        mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
        mz = max(mz, (unsigned)__shfl_xor((int)mz, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        const int slot = (blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64) % kRedShards;
        atomicMax(red + kRedDZ + slot, mx);
        atomicMax(red + kRedZ + slot, mz);
    }
}

template <bool TRANS, bool EXACT, bool UPD, bool LAYER>
__global__ __launch_bounds__(64) void block_down16(BlockSrc A, LayerScale y, VecSrc r, VecDst out,
                                                   const float* __restrict__ xe,
                                                   const float* __restrict__ P, unsigned* red,
                                                   int L, int w_, int Lc, int C) {
    constexpr int NB = kAhead16;
    const int w = EXACT ? 16 : w_;
    const int lane = threadIdx.x, i = lane & 15, g = lane >> 4;
    const int c = blockIdx.x % C, b = blockIdx.x / C;
    const int m0 = c * Lc, m1 = min(L, m0 + Lc);
    const float* rb = r.base + b * r.bstride;
    float* ob = out.base + b * out.bstride;
    unsigned mx = 0u, mz = 0u;
    auto emit = [&](int row, f4 x, f4 z) {
        if constexpr (UPD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                z[e] += x[e];
                mx = max(mx, __float_as_uint(fabsf(x[e])));
                mz = max(mz, __float_as_uint(fabsf(z[e])));
            }
        } else {
            z = x;
        }
        if (i == 0) put16<EXACT>(ob + (long long)row * out.rstride, w, g, z);
    };
    f4 x, a[NB], rr[NB], zz[NB] = {};
    int m = m0;
    if (c == 0) {
        x = vec16<EXACT>(rb + (long long)m * r.rstride, w, g);
        f4 z = {};
        if constexpr (UPD) z = vec16<EXACT>(ob + (long long)m * out.rstride, w, g);
        emit(m, x, z);
        ++m;
    } else if (!P) {
        x = vec16<EXACT>(xe + ((long long)b * (C - 1) + c - 1) * w, w, g);
    } else {
        // x_in from the chunk ends before this chunk: x_e = P_e x_{e-1} + q_e
        const BlockSrc ends{P, (long long)(C - 1) * w * w, (long long)w * w, 0};
        const float* qb = xe + (long long)b * (C - 1) * w;
        auto ask = [&](int e, int s) {
            const int ee = min(e, c - 1);
            a[s] = block16<false, EXACT, false>(ends, y, b, ee, w, i, g);
            rr[s] = vec16<EXACT>(qb + ee * w, w, g);
        };
        x = vec16<EXACT>(qb, w, g);
        if (c > 1)
#pragma unroll
            for (int s = 0; s < NB; ++s) ask(1 + s, s);
        for (int e = 1; e < c; e += NB) {
#pragma unroll
            for (int s = 0; s < NB; ++s) {
                if (e + s >= c) break;
                x = rr[s] + product16(a[s], x);
                ask(e + s + NB, s);
            }
        }
    }
    auto request = [&](int row, int s) {
        const int mm = min(row, m1 - 1);
        a[s] = block16<TRANS, EXACT, LAYER>(A, y, b, mm, w, i, g);
        if constexpr (LAYER && TRANS)
            rr[s] = f4{0.f, 0.f, 0.f, 0.f};
        else
            rr[s] = vec16<EXACT>(rb + (long long)mm * r.rstride, w, g);
        if constexpr (UPD) zz[s] = vec16<EXACT>(ob + (long long)mm * out.rstride, w, g);
    };
    if (m < m1)
#pragma unroll
        for (int s = 0; s < NB; ++s) request(m + s, s);
    for (; m < m1; m += NB) {
#pragma unroll
        for (int s = 0; s < NB; ++s) {
            if (m + s >= m1) break;
            x = rr[s] + product16(a[s], x);
            emit(m + s, x, zz[s]);
            request(m + s + NB, s);
        }
    }
    if constexpr (UPD) reduce_maxima(red, mx, mz);
}

// ----------------------------------------------------------- w = 17 .. 128
// One wave per 32 columns of P; wave v also forms rows 32 v .. of q (vector
// FMAs beside the products, from the left operands as they pass).  The left
// operand comes from memory in pieces of 32 rows, requested NS - 1 pieces
// ahead (every wave reads them, the others' requests hit the cache).
template <int WP>
struct UpShape {
    static constexpr int MT = WP / 32;               // 32-row pieces, waves
    static constexpr int NQ = WP / 8;                // 16-byte loads per piece
    static constexpr int NS = WP == 32 ? 4 : 2;      // pieces in registers
    static constexpr int UNR = MT > NS ? MT : NS;    // pieces per loop step
    static constexpr int ITEMS = 4 / MT;             // chunks per workgroup
};

// Workgroups of four waves, one per SIMD (two waves of a two-wave workgroup
// met those of the next one on the same SIMDs: w = 64, 496 chunks, 4.4 us per
// row against 2.35 for a lone chunk).
template <int WP, bool TRANS, bool EXACT>
__global__ __launch_bounds__(256, WP == 128 ? 1 : WP == 64 ? 2 : 4) void block_up(
    BlockSrc A, VecSrc r, float* __restrict__ P, float* __restrict__ q, int items, int w_, int Lc,
    int C) {
    using S = UpShape<WP>;
    constexpr int MT = S::MT;
    __shared__ __attribute__((aligned(16))) float xs_[S::ITEMS][2][WP];
    const int w = EXACT ? WP : w_;
    const int t = threadIdx.x, v = (t >> 6) % MT, lane = t & 63, i = lane & 31, h = lane >> 5;
    const int sub = __builtin_amdgcn_readfirstlane(t / (64 * MT));
    float (&xs)[2][WP] = xs_[sub];
    const int want = blockIdx.x * S::ITEMS + sub;
    const int item = min(want, items - 1);
    const int c = item % (C - 1), b = item / (C - 1);
    const int m0 = c * Lc;  // every chunk here has Lc rows
    const float* rb = r.base + b * r.bstride;
    const int own = 32 * v + i;  // the row of q, and the column of P, of this lane
    const bool in = EXACT || own < w;

    f16v p[MT], pn[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            p[mt][e] = 32 * mt + 8 * (e / 4) + 4 * h + e % 4 == own ? 1.f : 0.f;
    if (h == 0) xs[0][own] = 0.f;
    __syncthreads();
    f4 a[S::NS][S::NQ];
    const int total = Lc * MT;
    auto request = [&](int u, auto slot) {
        const int uu = min(u, total - 1);
        const int mt = uu % MT, row = m0 + uu / MT;
        // (row 0 has no block: x = r there, and no P is formed)
        const Src<EXACT> s = block_at<EXACT>(A, b, max(row, 1), w);
#pragma unroll
        for (int k = 0; k < S::NQ; ++k) {
            f4 x;
            if constexpr (!TRANS) {
                x = s.at((32 * mt + i) * w + 8 * k + 4 * h);
                if constexpr (!EXACT)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = 8 * k + 4 * h + e < w ? x[e] : 0.f;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = s.one((8 * k + 4 * h + e) * w + 32 * mt + i);
                    if constexpr (!EXACT) x[e] = 32 * mt + i < w ? x[e] : 0.f;
                }
            }
            a[slot][k] = x;
        }
    };
    unrolled<0, S::NS - 1>([&](auto s) { request(decltype(s)::value, s); });
    float rr = in ? rb[(long long)m0 * r.rstride + own] : 0.f;
    int buf = 0;
    for (int u0 = 0; u0 < total; u0 += S::UNR) {
        unrolled<0, S::UNR>([&](auto sc) {
            constexpr int s = decltype(sc)::value, slot = s % S::NS, mt = s % MT;
            const int u = u0 + s;
            if (u >= total) return;  // uniform: total is a multiple of MT
            request(u + S::NS - 1, std::integral_constant<int, (s + S::NS - 1) % S::NS>{});
            if (c > 0) {
                f16v acc = {};
#pragma unroll
                for (int k = 0; k < S::NQ; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc = mfma2(a[slot][k][e], p[k / 4][4 * (k % 4) + e], acc);
                pn[mt] = acc;
            }
            if (mt == v || MT == 1) {
                float y = 0.f;
                if (m0 + u / MT > 0) {
                    const float* x = xs[buf] + 4 * h;
                    float y0 = 0.f, y1 = 0.f;
#pragma unroll
                    for (int k = 0; k < S::NQ; ++k) {
                        const f4 xv = *reinterpret_cast<const f4*>(x + 8 * k);
                        y0 = fmaf(a[slot][k][0], xv[0], y0);
                        y1 = fmaf(a[slot][k][1], xv[1], y1);
                        y0 = fmaf(a[slot][k][2], xv[2], y0);
                        y1 = fmaf(a[slot][k][3], xv[3], y1);
                    }
                    y = y0 + y1;
                    y += __shfl_xor(y, 32, 64);
                }
                if (h == 0) xs[buf ^ 1][own] = in ? y + rr : 0.f;
            }
            if constexpr (mt == MT - 1) {
                const int row = min(u / MT + 1, Lc - 1) + m0;
                rr = in ? rb[(long long)row * r.rstride + own] : 0.f;
                if (c > 0)
#pragma unroll
                    for (int k = 0; k < MT; ++k) p[k] = pn[k];
                buf ^= 1;
                if constexpr (MT > 1)
                    __syncthreads();
                else
                    wave_sync();
            }
        });
    }
    if (want >= items) return;
    const long long o = item;
    if (h == 0 && in) q[o * w + own] = xs[buf][own];
    if (c > 0 && in) {
        float* out = P + o * w * w + own;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = 32 * mt + 8 * (e / 4) + 4 * h + e % 4;
                if (EXACT || row < w) out[(long long)row * w] = p[mt][e];
            }
    }
}

// One workgroup per chunk.  Thread (row i, part p) multiplies 1/TPR of a row;
// the parts meet through lane permutations, transposed blocks (whose rows are
// the lanes' consecutive addresses) through LDS; the next D rows are
// requested ahead.  Measured for the chain of all rows of a system (one
// MI355X): at w = 128, 1024 threads and one row ahead 206 us for 64 rows of
// 256 chains against 217 with 512 threads and 246 with two rows ahead; w = 32:
// 4 rows ahead 49 us, 8 rows 59; w = 64: 1-3 rows ahead 224-227, 4 rows 235.
template <int WP>
struct DownShape {
    static constexpr int NT = WP == 128 ? 1024 : 256;
    static constexpr int TPR = NT / WP;   // threads per block row
    static constexpr int CPT = WP / TPR;  // columns per thread
    static constexpr int NV = CPT / 4;
    static constexpr int D = WP == 32 ? 4 : WP == 64 ? 2 : 1;
    static constexpr int NB = D + 1;
};

// Rows m .. m1 - 1 of one chain, x of row m - 1 in xs[buf]; returns the buffer
// that holds the last row's x.  emit(row, i, x, z) gets every row's elements
// once, z the element of zb's row (ITER).
template <int WP, bool TRANS, bool EXACT, bool ITER, class Emit>
__device__ __forceinline__ int chain_rows(const BlockSrc& A, int b, const float* rb,
                                          long long rstride, const float* zb, long long zstride,
                                          int m, int m1, int w, float (&xs)[2][WP], float* part,
                                          int buf, Emit&& emit) {
    using S = DownShape<WP>;
    const int t = threadIdx.x;
    const int i = TRANS ? t % WP : t / S::TPR, p = TRANS ? t / WP : t % S::TPR;
    const int col0 = p * S::CPT;
    const bool in = EXACT || i < w;
    f4 blk[S::NB][S::NV];
    float rr[S::NB], zz[S::NB];
    auto request = [&](int row, auto slot) {
        const int mm = min(row, m1 - 1);
        const Src<EXACT> s = block_at<EXACT>(A, b, mm, w);
#pragma unroll
        for (int k = 0; k < S::NV; ++k) {
            f4 x;
            if constexpr (!TRANS) {
                x = s.at(i * w + col0 + 4 * k);
                if constexpr (!EXACT)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = col0 + 4 * k + e < w ? x[e] : 0.f;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = s.one((col0 + 4 * k + e) * w + i);
                    if constexpr (!EXACT) x[e] = in ? x[e] : 0.f;
                }
            }
            blk[slot][k] = x;
        }
        rr[slot] = in ? rb[mm * rstride + i] : 0.f;
        if constexpr (ITER) zz[slot] = in ? zb[mm * zstride + i] : 0.f;
    };
    if (m < m1) unrolled<0, S::D>([&](auto s) { request(m + decltype(s)::value, s); });
    __syncthreads();
    for (int mb = m; mb < m1; mb += S::NB) {
        unrolled<0, S::NB>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            const int row = mb + s;
            if (row >= m1) return;  // uniform over the workgroup
            request(row + S::D, std::integral_constant<int, (s + S::D) % S::NB>{});
            const float* xp = xs[buf] + col0;
            float acc = 0.f;
#pragma unroll
            for (int k = 0; k < S::NV; ++k) {
                const f4 xv = *reinterpret_cast<const f4*>(xp + 4 * k);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = fmaf(blk[s][k][e], xv[e], acc);
            }
            if constexpr (!TRANS) {
                acc = row_sum<S::TPR>(acc);
            } else {
                part[p * WP + i] = acc;
                __syncthreads();
                if (p == 0)
#pragma unroll
                    for (int k = 1; k < S::TPR; ++k) acc += part[k * WP + i];
            }
            buf ^= 1;
            if (p == 0) {
                const float x = in ? rr[s] + acc : 0.f;
                if (in) emit(row, i, x, ITER ? zz[s] : 0.f);
                xs[buf][i] = x;
            }
            __syncthreads();
        });
    }
    return buf;
}

template <int WP, bool TRANS, bool EXACT, bool UPD>
__global__ __launch_bounds__(DownShape<WP>::NT) void block_down(BlockSrc A, VecSrc r, VecDst out,
                                                               const float* __restrict__ xe,
                                                               const float* __restrict__ P,
                                                               unsigned* red, int L, int w_,
                                                               int Lc, int C) {
    using S = DownShape<WP>;
    __shared__ __attribute__((aligned(16))) float xs[2][WP];
    __shared__ float part[TRANS ? S::TPR * WP : 1];
    const int w = EXACT ? WP : w_;
    const int t = threadIdx.x;
    const int c = blockIdx.x % C, b = blockIdx.x / C;
    const int m0 = c * Lc, m1 = min(L, m0 + Lc);
    const float* rb = r.base + b * r.bstride;
    float* ob = out.base + b * out.bstride;
    unsigned mx = 0u, mz = 0u;
    auto emit = [&](int row, int i, float x, float z) {
        if constexpr (UPD) {
            z += x;
            mx = max(mx, __float_as_uint(fabsf(x)));
            mz = max(mz, __float_as_uint(fabsf(z)));
        } else {
            z = x;
        }
        ob[(long long)row * out.rstride + i] = z;
    };
    int m = m0, buf = 0;
    const float* qb = xe + (long long)b * (C - 1) * w;
    if (t < WP) {
        float x = 0.f;
        if (t < w) {
            if (c == 0) {
                x = rb[(long long)m * r.rstride + t];
                emit(m, t, x, UPD ? ob[(long long)m * out.rstride + t] : 0.f);
            } else {
                x = qb[(P ? 0 : c - 1) * w + t];
            }
        }
        xs[0][t] = x;
    }
    if (c == 0) ++m;
    if (P && c > 1) {
        // x_in from the chunk ends before this chunk: x_e = P_e x_{e-1} + q_e
        const BlockSrc ends{P, (long long)(C - 1) * w * w, (long long)w * w, 0};
        buf = chain_rows<WP, false, EXACT, false>(ends, b, qb, w, nullptr, 0, 1, c, w, xs, part, buf,
                                                  [](int, int, float, float) {});
    }
    chain_rows<WP, TRANS, EXACT, UPD>(A, b, rb, r.rstride, ob, out.rstride, m, m1, w, xs, part, buf,
                                      emit);
    if constexpr (UPD) reduce_maxima(red, mx, mz);
}

int block_pad(int w) { return w <= 16 ? 16 : w <= 32 ? 32 : w <= 64 ? 64 : 128; }

// Estimated time (us) of a solve, from costs measured on one MI355X: a row of
// block_up and of block_down where a chunk is alone, the rows per us of the
// whole chip (block_up at w = 128: one workgroup per CU), and a launch.  The
// chunk ends are solved on their own, or (walk) every chunk substitutes
// through the ends before it first, which saves launches where they are few.
double plan_cost(int B, int L, int WP, bool top, BlockPlan* plan) {
    const int k = WP == 16 ? 0 : WP == 32 ? 1 : WP == 64 ? 2 : 3;
    static const double up[] = {0.2, 0.8, 2.45, 9.5}, down[] = {0.14, 0.17, 0.29, 0.85};
    static const double up_rate[] = {4200, 1090, 172, 27}, down_rate[] = {4700, 1524, 400, 103};
    const double launch = 4.0, rows = (double)B * L;
    auto atleast = [](double a, double b) { return a > b ? a : b; };
    BlockPlan best{0, false};
    double t_best = launch + atleast(L * down[k], rows / down_rate[k]);
    static const int all[] = {4, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64, 96, 128},
                     few[] = {8, 16, 32};
    const int* ms = top ? all : few;
    const int n = top ? 14 : 3;
    for (int j = 0; j < n && ms[j] < L; ++j) {
        const int m = ms[j], C = (L + m - 1) / m;
        const int rounds = WP == 128 ? (B * (C - 1) + 255) / 256 : 1;
        const double t = 2 * launch + atleast(m * up[k] * rounds, rows / up_rate[k]);
        const double walked = (double)B * C * (C - 1) / 2;
        const double t_walk = t + atleast((m + C - 2) * down[k], (rows + 0.5 * walked) / down_rate[k]);
        const double t_ends = t + atleast(m * down[k], rows / down_rate[k]) +
                              (C > 2 ? plan_cost(B, C - 1, WP, false, nullptr) : 0.0);
        if (t_walk < t_best) {
            t_best = t_walk;
            best = BlockPlan{m, true};
        }
        if (t_ends < t_best) {
            t_best = t_ends;
            best = BlockPlan{m, false};
        }
    }
    if (plan) *plan = best;
    return t_best;
}

}  // namespace

double block_plan(int B, int L, int w, BlockPlan* plan) {
    return plan_cost(B, L, block_pad(w), plan != nullptr, plan);
}

#define DEEPPCR_BLOCK_WIDTHS(CALL, CALL16)        \
    do {                                          \
        switch (w) {                              \
            case 16: CALL16(true); break;         \
            case 32: CALL(32, true); break;       \
            case 64: CALL(64, true); break;       \
            case 128: CALL(128, true); break;     \
            default:                              \
                if (w < 16) CALL16(false);        \
                else if (w < 32) CALL(32, false); \
                else if (w < 64) CALL(64, false); \
                else CALL(128, false);            \
        }                                         \
    } while (0)

// A launch has at most 2^32 - 1 threads: more systems than that takes go in
// several, launch(first system, systems).
template <class F>
static hipError_t by_systems(int B, long long threads_per_system, F&& launch) {
    const long long most = 0xffffffffLL / threads_per_system;
    if (most < 1) return hipErrorInvalidValue;
    for (long long b = 0; b < B; b += most) {
        const hipError_t e = launch(b, (int)(B - b < most ? B - b : most));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
static BlockSrc from(const BlockSrc& A, long long b) {
    return {A.base + b * A.bstride, A.bstride, A.rstride, A.trans};
}
static VecSrc from(const VecSrc& v, long long b) {
    return {v.base + b * v.bstride, v.bstride, v.rstride};
}
static VecDst from(const VecDst& v, long long b) {
    return {v.base + b * v.bstride, v.bstride, v.rstride};
}
static LayerScale from(const LayerScale* y, long long b) {
    return y ? LayerScale{y->d + b * y->bstride, y->bstride, y->rstride, y->residual}
             : LayerScale{};
}

static hipError_t block_up_some(const BlockSrc& A, const LayerScale* y, const LayerScale& ly,
                                const VecSrc& r, float* P, float* q, int B, int L, int w, int Lc,
                                int C, hipStream_t st) {
    const int items = B * (C - 1);
    const int WP = block_pad(w), per = WP == 16 ? 1 : 128 / WP;
    const dim3 grid((unsigned)((items + per - 1) / per));
#define UP16_AS(T, EX, LY) \
    hipLaunchKernelGGL((block_up16<T, EX, LY>), grid, dim3(64), 0, st, A, ly, r, P, q, L, w, Lc, C)
#define UP16(EX)                                  \
    do {                                          \
        if (A.trans && y) UP16_AS(true, EX, true);        \
        else if (A.trans) UP16_AS(true, EX, false);       \
        else if (y) UP16_AS(false, EX, true);             \
        else UP16_AS(false, EX, false);           \
    } while (0)
#define UP(WP_, EX)                                                                             \
    do {                                                                                       \
        if (A.trans) hipLaunchKernelGGL((block_up<WP_, true, EX>), grid, dim3(256), 0, st, A, r, P, q, items, w, Lc, C); \
        else hipLaunchKernelGGL((block_up<WP_, false, EX>), grid, dim3(256), 0, st, A, r, P, q, items, w, Lc, C); \
    } while (0)
    DEEPPCR_BLOCK_WIDTHS(UP, UP16);
#undef UP
#undef UP16
#undef UP16_AS
    return hipGetLastError();
}

hipError_t launch_block_up(const BlockSrc& A, const LayerScale* y, const VecSrc& r, float* P,
                           float* q, int B, int L, int w, int Lc, int C, hipStream_t st) {
    if (y && w > 16) return hipErrorInvalidValue;
    const long long ends = C - 1;
    return by_systems(B, ends * (w <= 16 ? 64 : 256), [&](long long b, int n) {
        return block_up_some(from(A, b), y, from(y, b), from(r, b), P + b * ends * w * w,
                             q + b * ends * w, n, L, w, Lc, C, st);
    });
}

static hipError_t block_down_some(const BlockSrc& A, const LayerScale* y, const LayerScale& ly,
                                  const VecSrc& r, const VecDst& x, const float* xe,
                                  const float* P, unsigned* red, int B, int L, int w, int Lc,
                                  int C, hipStream_t st) {
    const dim3 grid((unsigned)((long long)B * C));
#define DOWN_AS(K, NT)                                                                         \
    hipLaunchKernelGGL(K, grid, dim3(NT), 0, st, A, r, x, xe, P, red, L, w, Lc, C)
#define DOWN16_AS(T, EX, U, LY)                                                             \
    hipLaunchKernelGGL((block_down16<T, EX, U, LY>), grid, dim3(64), 0, st, A, ly, r, x, xe, P, red, \
                       L, w, Lc, C)
#define DOWN16(EX)                                                   \
    do {                                                             \
        if (A.trans && red) return hipErrorInvalidValue;             \
        if (A.trans && y) DOWN16_AS(true, EX, false, true);          \
        else if (A.trans) DOWN16_AS(true, EX, false, false);         \
        else if (red && y) DOWN16_AS(false, EX, true, true);         \
        else if (red) DOWN16_AS(false, EX, true, false);             \
        else if (y) return hipErrorInvalidValue;                     \
        else DOWN16_AS(false, EX, false, false);                     \
    } while (0)
#define DOWN(WP, EX)                                                                           \
    do {                                                                                       \
        if (A.trans && red) return hipErrorInvalidValue;                                       \
        if (A.trans) DOWN_AS((block_down<WP, true, EX, false>), DownShape<WP>::NT);            \
        else if (red) DOWN_AS((block_down<WP, false, EX, true>), DownShape<WP>::NT);           \
        else DOWN_AS((block_down<WP, false, EX, false>), DownShape<WP>::NT);                   \
    } while (0)
    DEEPPCR_BLOCK_WIDTHS(DOWN, DOWN16);
#undef DOWN
#undef DOWN16
#undef DOWN16_AS
#undef DOWN_AS
    return hipGetLastError();
}

hipError_t launch_block_down(const BlockSrc& A, const LayerScale* y, const VecSrc& r,
                             const VecDst& x, const float* xe, const float* P, unsigned* red,
                             int B, int L, int w, int Lc, int C, hipStream_t st) {
    if (y && w > 16) return hipErrorInvalidValue;
    const long long ends = C - 1;
    return by_systems(B, (long long)C * (w <= 16 ? 64 : w <= 64 ? 256 : 1024),
                      [&](long long b, int n) {
        return block_down_some(from(A, b), y, from(y, b), from(r, b), from(x, b),
                               xe ? xe + b * ends * w : nullptr,
                               P ? P + b * ends * w * w : nullptr, red, n, L, w, Lc, C, st);
    });
}

}  // namespace deeppcr
