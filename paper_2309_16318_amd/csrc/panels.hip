// The Newton solve and the backward solve of MLP layers by row chunks, for
// widths 17 to 128: the operators J_l = diag(d_l) W_l (+ I) (App. A.1) are
// never stored.
//
// The rows of every system are cut into C consecutive chunks.  Inside a chunk
// x_l = P_l x_in + q_l with x_in the row before it, so that
//   1. chunk_pass forms, for every chunk but the first and the last, the
//      product P of its operators, one block product per row (Alg. 1 forms
//      one per row and level), and, beside it, every chunk's q;
//   2. the chunk ends are a block-bidiagonal system of C - 1 rows with the
//      operators P, solved as stored blocks (blocks.hip);
//   3. apply_pass substitutes inside every chunk from its x_in, which also
//      applies the Newton update, or writes the adjoints.
// In exact arithmetic this is the solution of Eq. 3 (Eq. 12 for the
// transposed system).  Per row it reads one weight block, shared by all
// systems through the caches, and writes vectors only.
//
// All products run on the bf16 matrix cores at float32 precision: a float32
// value, scaled where it is near the ends of the range, is split into three
// bf16 parts (round to nearest, exact: 8 + 8 + 8 significant bits), and of the nine products of two split values the six
// above 2^-24 are accumulated in float32, the five small ones in an
// accumulator of their own.  Infinities have no parts: a row of a vector that
// meets one is summed again in plain float32.  Measured on one MI355X, the six cost 32 cycles
// each per 32 x 32 x 16 tile against 8 x 64 cycles of float32 instructions:
// 2.7 times the rate, with fewer roundings (one per 16 terms and part).
#include "internal.h"
#include "rows.h"

#include <type_traits>

namespace deeppcr {
namespace {

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

constexpr int kThr = 256;

template <int I, int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<I + 1, N>(f);
    }
}

// The three bf16 parts of two values, packed.
struct Parts2 {
    unsigned h, m, l;
};
__device__ __forceinline__ unsigned pack2(float x, float y) {
    const b2 p = __builtin_convertvector(f2{x, y}, b2);
    return __builtin_bit_cast(unsigned, p);
}
__device__ __forceinline__ float lo_f(unsigned p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi_f(unsigned p) { return __uint_as_float(p & 0xffff0000u); }
__device__ __forceinline__ Parts2 split2(float x, float y) {
    Parts2 p;
    p.h = pack2(x, y);
    const float x1 = x - lo_f(p.h), y1 = y - hi_f(p.h);
    p.m = pack2(x1, y1);
    p.l = pack2(x1 - lo_f(p.m), y1 - hi_f(p.m));
    return p;
}
// bf16 has float32's exponents and 16 bits less, so the parts of x add up to
// it only if its last bit is at least 2^-133, bf16's smallest value (which the
// matrix cores keep).  Vectors are therefore split as 2^16 x, which is exact
// for every x below 2^111; values from 2^110 on count as having no parts.
constexpr float kShift = 0x1p16f, kUnshift = 0x1p-16f, kNoParts = 0x1p110f;

// Eight values as three operand registers.
struct Parts8 {
    b8 h, m, l;
};
__device__ __forceinline__ Parts8 split8(const float (&v)[8], float shift = 1.f) {
    u4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const Parts2 p = split2(shift * v[2 * j], shift * v[2 * j + 1]);
        h[j] = p.h;
        m[j] = p.m;
        l[j] = p.l;
    }
    return {__builtin_bit_cast(b8, h), __builtin_bit_cast(b8, m), __builtin_bit_cast(b8, l)};
}

__device__ __forceinline__ f16v mfma32(b8 a, b8 b, f16v c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16(b8 a, b8 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// c += A B at float32 precision: the leading products into c.x, the others into c.s.
template <class V>
struct Acc {
    V x, s;
};
__device__ __forceinline__ void mac(Acc<f16v>& c, const Parts8& a, const Parts8& b) {
    c.s = mfma32(a.l, b.h, c.s);
    c.x = mfma32(a.h, b.h, c.x);
    c.s = mfma32(a.m, b.m, c.s);
    c.s = mfma32(a.h, b.l, c.s);
    c.s = mfma32(a.m, b.h, c.s);
    c.s = mfma32(a.h, b.m, c.s);
}
__device__ __forceinline__ void mac(Acc<f4>& c, const Parts8& a, const Parts8& b) {
    c.s = mfma16(a.l, b.h, c.s);
    c.x = mfma16(a.h, b.h, c.x);
    c.s = mfma16(a.m, b.m, c.s);
    c.s = mfma16(a.h, b.l, c.s);
    c.s = mfma16(a.m, b.h, c.s);
    c.s = mfma16(a.h, b.m, c.s);
}

// ------------------------------------------------------------ shapes
// Vector panels: 16 systems per group, a 16 x 16 x 32 tile per 16 rows.
// Wave v of a group owns rows 16 MTW v ..; tile t's row index i stands for
// row MTW i + t of them, so that a lane's results are 4 MTW consecutive rows.
template <int WP>
struct VecShape {
    static constexpr int MTW = WP == 128 ? 2 : 1;
    static constexpr int NR = 4 * MTW;             // consecutive rows per lane
    static constexpr int KT = WP / 32;             // k tiles
    static constexpr int WPG = WP / (16 * MTW);    // waves per group
    static constexpr int GPW = 4 / WPG;            // groups per workgroup
    static constexpr int RAW = KT * 3 * 1024;      // a vector panel's parts in LDS, bytes
    static constexpr int BUF = RAW + 16 * WP * 4;  // and its float32 values
    static constexpr int LDS = GPW * 2 * BUF;
};
// Product panels: 32 columns of one system's P per wave, all rows.
template <int WP>
struct ProdShape {
    static constexpr int MT = WP / 32, KT = WP / 16;
    static constexpr int SYS = 4 / MT;             // systems per workgroup
    static constexpr int LPS = WP == 32 ? 4 : 1;   // layers a stage starts
    static constexpr int WB = 4096 * 6;            // 4096 split weights, bytes
    static constexpr int STAGE = WB + LPS * 512;   // and the layers' d, 128 floats each
    static constexpr int LDS = 2 * STAGE;
};

// Weights split once for all passes of a call: per layer and part (h, m, l)
// the 1 KiB operand tiles of the product panels, 32 rows x 16 columns each,
// rows padded with zeros; at WP = 128 per 32 rows [part][tile], below
// [part][all tiles].
template <int WP>
struct SplitShape {
    static constexpr int LAYER = WP * WP * 6;                       // bytes of a layer
    static constexpr int PART = WP == 32 ? 2048 : 8192;             // bytes of a part
    static constexpr int SLICE = WP == 128 ? 3 * PART : LAYER;      // bytes of 32 rows (128)
};

// The rows of W_l (TRANS: of W_l^T) a lane multiplies with, for the vector
// panels, in put_panel's k order.  Where w is not the padded width, elements beyond a row's end hold
// the next row's weights: they meet zeros of the panel, or (TRANS) give rows
// that the caller drops.
template <int WP, bool TRANS, bool EXACT>
__device__ __forceinline__ void load_strip(const Src<EXACT>& Wl, int w, int base, int idx, int g,
                                           float (&raw)[VecShape<WP>::MTW][VecShape<WP>::KT][8]) {
    using S = VecShape<WP>;
    const int k0 = 16 * (g / 2) + 4 * (g % 2);  // and k0 + 8
    if constexpr (!TRANS) {
#pragma unroll
        for (int t = 0; t < S::MTW; ++t) {
            const unsigned row = (base + S::MTW * idx + t) * w + k0;
#pragma unroll
            for (int k = 0; k < S::KT; ++k)
#pragma unroll
                for (int q = 0; q < 8; q += 4) {
                    const f4 x = Wl.at(row + 32 * k + 2 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) raw[t][k][q + e] = x[e];
                }
        }
    } else {
        const unsigned col = base + S::MTW * idx + k0 * w;
#pragma unroll
        for (int k = 0; k < S::KT; ++k)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int kk = 32 * k + j + (j & 4);
                if constexpr (EXACT && S::MTW == 2) {
                    const f2 x = *reinterpret_cast<const f2*>(Wl.p + col + kk * w);
                    raw[0][k][j] = x[0];
                    raw[1][k][j] = x[1];
                } else {
#pragma unroll
                    for (int t = 0; t < S::MTW; ++t) raw[t][k][j] = Wl.one(col + kk * w + t);
                }
            }
    }
}

// Elements i .. i + 3 and i + 8 .. i + 11 of a row.
template <bool EXACT>
__device__ __forceinline__ void load_operand(const Src<EXACT>& src, unsigned row, int i, int w,
                                             float (&v)[8]) {
    float a[4], b[4];
    load_row<4>(src, row, i, w, a);
    load_row<4>(src, row, i + 8, w, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = a[e];
        v[4 + e] = b[e];
    }
}

// A lane's NR rows of a vector panel as operand parts in LDS, for the k order
// of the split weights: a lane (n, g) of k tile K multiplies rows 16 T + 4 h ..
// + 3 and 16 T + 8 + 4 h .. + 3, T = 2 K + g / 2, h = g % 2.
template <int WP>
__device__ __forceinline__ void put_panel(char* buf, int r0, int n,
                                          const float (&x)[VecShape<WP>::NR]) {
    using S = VecShape<WP>;
#pragma unroll
    for (int j = 0; j < S::NR; j += 4) {
        const int u = (r0 % 16 + j) / 4;  // the quarter of its 16 rows
        char* p = buf + r0 / 32 * 1024 + (n + 16 * (2 * (r0 / 16 % 2) + u % 2)) * 16 + 8 * (u / 2);
        const Parts2 a = split2(kShift * x[j], kShift * x[j + 1]),
                     b = split2(kShift * x[j + 2], kShift * x[j + 3]);
        *reinterpret_cast<u2*>(p) = u2{a.h, b.h};
        *reinterpret_cast<u2*>(p + S::KT * 1024) = u2{a.m, b.m};
        *reinterpret_cast<u2*>(p + 2 * S::KT * 1024) = u2{a.l, b.l};
    }
}

// Element k of system n of a vector panel: the sum of its parts or, where it
// has none (infinities, NaN and the largest values), its float32 value, which
// vector_panel stores beside them then.
template <int WP>
__device__ __forceinline__ float panel_value(const char* buf, int n, int k) {
    using S = VecShape<WP>;
    const int u = k % 16 / 4;
    const char* p =
        buf + k / 32 * 1024 + (n + 16 * (2 * (k / 16 % 2) + u % 2)) * 16 + 8 * (u / 2) + 2 * (k % 4);
    auto part = [&](int i) {
        return __uint_as_float(
            (unsigned)*reinterpret_cast<const unsigned short*>(p + i * S::KT * 1024) << 16);
    };
    const float x = part(0) + part(1) + part(2);
    return fabsf(x) < __builtin_inff() ? kUnshift * x
                                       : reinterpret_cast<const float*>(buf + S::RAW)[n * WP + k];
}

// ------------------------------------------------------------ vector panels
// One chunk of the recurrence for 16 systems per group.  APPLY: from x_in to
// every row; otherwise from zero to the chunk's last row, q.
template <int WP, bool BWD, bool EXACT, bool APPLY, bool PRE>
__device__ __forceinline__ void vector_panel(const PanelArgs& a, char* lds, int c, int wg) {
    using S = VecShape<WP>;
    // rows requested ahead (beside the products, their registers allow fewer)
    constexpr int D = WP == 128 ? (APPLY ? 2 : 1) : WP == 64 ? 3 : 5;
    constexpr int NB = D + 1, NR = S::NR;
    const int t = threadIdx.x, v = t >> 6, lane = t & 63;
    const int sub = v / S::WPG, wv = v % S::WPG;
    const int n = lane & 15, g = lane >> 4;
    const int w = EXACT ? WP : a.w, L = a.L;
    const int base = wv * 16 * S::MTW, r0 = base + NR * g;
    const int bb = (wg * S::GPW + sub) * 16 + n;
    const bool live = bb < a.B;
    const int b = live ? bb : a.B - 1;
    const int m0 = c * a.Lc, m1 = min(a.rows, m0 + a.Lc);
    char* const panel = lds + sub * 2 * S::BUF;
    const unsigned bL = (unsigned)b * L, nv = (unsigned)a.B * L * w;
    const Src<EXACT> sd(a.d, nv), sr(a.r, BWD ? (unsigned)a.B * w : nv), sz(a.Z, nv);

    if constexpr (BWD && !APPLY) {
        // only row 0 has a right-hand side
        if (c > 0) {
            if (live) {
                const float zero[NR] = {};
                store_row<NR, true>(a.q + ((long long)b * (a.C - 1) + c) * WP, r0, WP, zero);
            }
            return;
        }
    }
    unsigned mx = 0u, mz = 0u;
    float raw[PRE ? 1 : NB][S::MTW][S::KT][8];
    Parts8 pre[PRE ? NB : 1][S::MTW][S::KT];
    float ad[NB][NR], ar[NB][NR], az[NB][NR];
    // row m's weights, and the vectors its result meets: d and r (forward),
    // d of the next row's layer (backward), the iterate
    auto aux = [&](int m, float (&d)[NR], float (&r)[NR], float (&z)[NR]) {
        if constexpr (!BWD) {
            load_row<NR>(sd, (bL + m) * w, r0, w, d);
            load_row<NR>(sr, (bL + m) * w, r0, w, r);
            if constexpr (APPLY) load_row<NR>(sz, (bL + m) * w, r0, w, z);
        } else {
            load_row<NR>(sd, (bL + max(L - m - 1, 0)) * w, r0, w, d);
        }
    };
    auto emit = [&](int m, const float (&x)[NR], const float (&z)[NR]) {
        if constexpr (!APPLY) {
            if (m == m1 - 1 && live)
                store_row<NR, true>(a.q + ((long long)b * (a.C - 1) + c) * WP, r0, WP, x);
        } else if constexpr (!BWD) {
            float y[NR];
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                y[j] = z[j] + x[j];
                mx = max(mx, __float_as_uint(fabsf(x[j])));
                mz = max(mz, __float_as_uint(fabsf(y[j])));
            }
            if (live) store_row<NR, EXACT>(a.Z + (long long)(bL + m) * w, r0, w, y);
        } else if (live) {
            store_row<NR, EXACT>(m < L ? a.Lambda + (long long)(bL + L - 1 - m) * w : a.dz0 + (long long)b * w,
                                 r0, w, x);
        }
    };
    // split weights of this lane's rows: tile row within 32 rows, and tile
    const int trow = (base + S::MTW * n) % 32;
    const unsigned off = base / 32 * (WP == 128 ? SplitShape<WP>::SLICE : WP / 16 * 1024) +
                         g / 2 * 1024 + (trow + 32 * (g % 2)) * 16;
    auto request = [&](int m, auto slot) {
        constexpr int s = decltype(slot)::value;
        const int mm = min(m, m1 - 1);
        const int op = BWD ? min(L - mm, L - 1) : mm;
        if constexpr (PRE) {
            const char* p = a.S + (long long)op * SplitShape<WP>::LAYER + off;
#pragma unroll
            for (int q = 0; q < S::MTW; ++q)
#pragma unroll
                for (int k = 0; k < S::KT; ++k) {
                    const char* o = p + k * 2048 + q * 16;
                    pre[s][q][k].h = *reinterpret_cast<const b8*>(o);
                    pre[s][q][k].m = *reinterpret_cast<const b8*>(o + SplitShape<WP>::PART);
                    pre[s][q][k].l = *reinterpret_cast<const b8*>(o + 2 * SplitShape<WP>::PART);
                }
        } else {
            load_strip<WP, BWD, EXACT>(Src<EXACT>(a.W + (long long)op * w * w, w * w), w, base, n,
                                       g, raw[s]);
        }
        aux(mm, ad[s], ar[s], az[s]);
    };
    float x[NR];
    int m = m0;
    // the B operand of row m: x, scaled by row m's own d when transposed;
    // whether all of it has parts
    auto put = [&](int buf, const float (&d)[NR]) {
        float y[NR], size = 0.f;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            y[j] = BWD ? d[j] * x[j] : x[j];
            size += fabsf(y[j]);
        }
        put_panel<WP>(panel + buf * S::BUF, r0, n, y);
        return size < kNoParts;
    };
    auto put_values = [&](int buf, const float (&d)[NR]) {
        float y[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) y[j] = BWD ? d[j] * x[j] : x[j];
        store_row<NR, true>(reinterpret_cast<float*>(panel + buf * S::BUF + S::RAW) + n * WP, r0,
                            WP, y);
    };
    // Row m's product as plain sums from the panel `buf`, where that of the
    // parts is not finite (a factor has none, or the sum overflows), through
    // the space of the other panel's float32 values.  Rare: the addresses are
    // made anew, so that nothing of it is kept in registers.
    auto plain = [&](int m, int buf, float (&y)[NR]) {
        int nn = n, rr = r0;
        asm volatile("" : "+v"(nn), "+v"(rr));
        const float* Wl = a.W + (long long)(BWD ? L - m : m) * w * w;
        float* out = reinterpret_cast<float*>(panel + (buf ^ 1) * S::BUF + S::RAW) + nn * WP + rr;
#pragma unroll 1
        for (int j = 0; j < NR; ++j) {
            float v = 0.f;
            const int i = rr + j;
            if (i < w)
#pragma unroll 1
                for (int k = 0; k < w; ++k)
                    v = fmaf(Wl[BWD ? k * w + i : i * w + k],
                             panel_value<WP>(panel + buf * S::BUF, nn, k), v);
            out[j] = v;
        }
#pragma unroll
        for (int j = 0; j < NR; ++j) y[j] = out[j];
    };
    {
        float d0[NR] = {}, rr[NR], z0[NR];
        if (APPLY && c > 0) {
            const Src<true> sx(a.xe + ((long long)b * (a.C - 1) + c - 1) * WP, WP);
            load_row<NR>(sx, 0, r0, WP, x);
            if constexpr (BWD) load_row<NR>(sd, (bL + L - m) * w, r0, w, d0);
        } else {
            if constexpr (BWD)
                load_row<NR>(sr, (unsigned)b * w, r0, w, x);  // G
            else
                load_row<NR>(sr, (bL + m) * w, r0, w, x);
            aux(m, d0, rr, z0);
            emit(m, x, z0);
            ++m;
        }
        if (m < m1 && __builtin_expect(!put(0, d0), 0)) put_values(0, d0);
    }
    if (m < m1) {
        unrolled<0, D>([&](auto s) { request(m + decltype(s)::value, s); });
        // (weights out of the ordinary range are multiplied by 1 / scale)
        const float* const scale = a.scale + base / 32;
        const bool scaled = *a.odd == a.stamp;
        int buf = 0;
        for (int mb = m; mb < m1; mb += NB) {
            unrolled<0, NB>([&](auto sc) {
                constexpr int s = decltype(sc)::value;
                const int row = mb + s;
                if (row >= m1) return;  // uniform over the workgroup
                float factor = kUnshift;
                if (__builtin_expect(scaled, 0)) {
                    const float f = scale[(BWD ? L - row : row) * (WP / 32)];
                    factor *= f;
                    if constexpr (!PRE)
#pragma unroll
                        for (int q = 0; q < S::MTW; ++q)
#pragma unroll
                            for (int k = 0; k < 8 * S::KT; ++k) raw[s][q][k / 8][k % 8] *= 1.f / f;
                }
                Parts8 A[S::MTW][S::KT];
#pragma unroll
                for (int q = 0; q < S::MTW; ++q)
#pragma unroll
                    for (int k = 0; k < S::KT; ++k) {
                        if constexpr (PRE)
                            A[q][k] = pre[s][q][k];
                        else
                            A[q][k] = split8(raw[s][q][k]);
                    }
                __syncthreads();  // the panel of row - 1 is complete
                request(row + D, std::integral_constant<int, (s + D) % NB>{});
                const char* in = panel + buf * S::BUF + lane * 16;
                Acc<f4> acc[S::MTW] = {};
#pragma unroll
                for (int k = 0; k < S::KT; ++k) {
                    Parts8 p;
                    p.h = *reinterpret_cast<const b8*>(in + k * 1024);
                    p.m = *reinterpret_cast<const b8*>(in + (S::KT + k) * 1024);
                    p.l = *reinterpret_cast<const b8*>(in + (2 * S::KT + k) * 1024);
#pragma unroll
                    for (int q = 0; q < S::MTW; ++q) mac(acc[q], A[q][k], p);
                }
                float y[NR], xp[NR];
#pragma unroll
                for (int q = 0; q < S::MTW; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        y[S::MTW * e + q] = factor * (acc[q].x[e] + acc[q].s[e]);
#pragma unroll
                for (int j = 0; j < NR; ++j) xp[j] = x[j];
                auto finish = [&] {
#pragma unroll
                    for (int j = 0; j < NR; ++j) {
                        float z = y[j];
                        if constexpr (!BWD) z *= ad[s][j];
                        if (a.residual) z += xp[j];
                        if constexpr (!BWD) z += ar[s][j];
                        x[j] = EXACT || r0 + j < w ? z : 0.f;
                    }
                };
                finish();
                buf ^= 1;
                if (__builtin_expect(!put(buf, ad[s]), 0)) {
                    plain(row, buf ^ 1, y);
                    finish();
                    put(buf, ad[s]);
                    put_values(buf, ad[s]);
                }
                emit(row, x, az[s]);
            });
        }
    }
    if constexpr (APPLY && !BWD) {
        if (!live) mx = mz = 0u;
        for (int off = 32; off > 0; off >>= 1) {
            mx = max(mx, (unsigned)__shfl_xor((int)mx, off, 64));
            mz = max(mz, (unsigned)__shfl_xor((int)mz, off, 64));
        }
        if (lane == 0) {
            const int slot = (blockIdx.x * 4 + v) % kRedShards;
            atomicMax(a.red + kRedDZ + slot, mx);
            atomicMax(a.red + kRedZ + slot, mz);
        }
    }
}

// ----------------------------------------------------------- product panels
// P of chunk c for SYS systems: wave (system, 32 columns) keeps its columns
// of the running product in registers, as the float32 results of a 32 x 32
// tile per 32 rows and as the operand parts of the next product, whose lanes
// hold exactly those rows (the k order of an operand is free, and the
// weights are laid out to match).  So the waves of a workgroup share only
// the weights: 4096 of them per stage are loaded into registers one stage
// ahead, split, and put into one of two LDS buffers in operand order; one
// barrier per stage.
template <int WP, bool BWD, bool EXACT, bool PRE>
__device__ __forceinline__ void product_panel(const PanelArgs& a, char* lds, int c, int wg) {
    using S = ProdShape<WP>;
    const int t = threadIdx.x, v = t >> 6, lane = t & 63;
    const int n = lane & 31, h = lane >> 5;
    const int w = EXACT ? WP : a.w, L = a.L;
    const int panel = v % S::MT;
    const int bb = wg * S::SYS + v / S::MT;
    const bool live = bb < a.B;
    const int b = live ? bb : a.B - 1;
    const int m0 = c * a.Lc, m1 = min(a.rows, m0 + a.Lc);
    const Src<EXACT> sd(a.d, (unsigned)a.B * L * w);
    // (weights out of the ordinary range are multiplied by 1 / scale)
    auto scale_at = [&](int m, int mt) { return a.scale[(long long)(BWD ? L - m : m) * S::MT + mt]; };
    const bool scaled = *a.odd == a.stamp;

    // this thread's 4 x 4 weights of a stage: rows 4 rg .., columns 4 cg .. of
    // the stage's 32-row block blk
    const int rg = t & 7, cg = (t >> 3) % (WP / 4), blk = __builtin_amdgcn_readfirstlane(t / (2 * WP));
    constexpr int LPS = S::LPS;
    constexpr int SPL = WP == 128 ? 4 : 1;  // stages per layer
    f4 raw[PRE ? 1 : 4];
    u4 pre[PRE ? 6 : 1];
    // d of the layers a stage starts: SYS systems x WP rows per layer, thread
    // t's element e is layer (t + 256 e) / 128's t % 128
    constexpr int ND = (LPS + 1) / 2;
    float rd[ND];
    const int dsys = min(a.B - 1, wg * S::SYS + (t & 127) / WP), drow = (t & 127) % WP;
    auto request = [&](int st) {
#pragma unroll
        for (int e = 0; e < ND; ++e) {
            // (transposed: of the operator of the row after, which scales
            // the columns that the product of this row leaves)
            const int j = (t + 256 * e) >> 7;
            const int m = min(m1 - 1, m0 + (WP == 128 ? st / 4 : st * LPS) + (LPS > 1 ? j : 0));
            const int l = BWD ? max(L - m - 1, 0) : m;
            const unsigned o = ((unsigned)dsys * L + l) * w + drow;
            rd[e] = EXACT || drow < w ? sd.one(o) : 0.f;
        }
        if constexpr (PRE) {
            // six 16-byte pieces of the stage per thread
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const int u = t + 256 * j;
                const int m = min(m1 - 1, m0 + (WP == 128 ? st / 4 : WP == 64 ? st : 4 * st + u / 384));
                const char* p = a.S + (long long)(BWD ? L - m : m) * SplitShape<WP>::LAYER +
                                (WP == 128 ? st % 4 * SplitShape<WP>::SLICE : 0);
                pre[j] = *reinterpret_cast<const u4*>(p + (WP == 32 ? u % 384 : u) * 16);
            }
        } else {
            const int m = min(m1 - 1, m0 + (WP == 128 ? st / 4 : WP == 64 ? st : 4 * st + blk));
            const int mt = WP == 128 ? st % 4 : WP == 64 ? blk : 0;
            const int i = 32 * mt + 4 * rg, k = 4 * cg;
            // (as in load_strip, elements beyond a row's end meet zeros, or give
            // rows that meet zeros)
            const Src<EXACT> Wl(a.W + (long long)(BWD ? L - m : m) * w * w, w * w);
#pragma unroll
            for (int e = 0; e < 4; ++e) raw[e] = Wl.at(((BWD ? k : i) + e) * w + (BWD ? i : k));
        }
    };
    char* const dst = lds + (blk * S::KT + cg / 4) * 1024 + (4 * rg + 32 * (cg & 1)) * 16 +
                      8 * ((cg >> 1) & 1);
    auto put = [&](int st) {
        const int buf = st & 1;
        if constexpr (PRE) {
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const int u = t + 256 * j;
                const int o = WP == 32 ? u % 384 / 128 * 8192 + u / 384 * 2048 + u % 128 * 16 : u * 16;
                *reinterpret_cast<u4*>(lds + buf * S::STAGE + o) = pre[j];
            }
        } else {
            if (__builtin_expect(scaled, 0)) {
                const int m = min(m1 - 1, m0 + (WP == 128 ? st / 4 : WP == 64 ? st : 4 * st + blk));
                const float f = 1.f / scale_at(m, WP == 128 ? st % 4 : WP == 64 ? blk : 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[e] *= f;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f4 x = BWD ? f4{raw[0][e], raw[1][e], raw[2][e], raw[3][e]} : raw[e];
                const Parts2 p = split2(x[0], x[1]), q = split2(x[2], x[3]);
                char* o = dst + buf * S::STAGE + e * 16;
                *reinterpret_cast<u2*>(o) = u2{p.h, q.h};
                *reinterpret_cast<u2*>(o + S::WB / 3) = u2{p.m, q.m};
                *reinterpret_cast<u2*>(o + 2 * (S::WB / 3)) = u2{p.l, q.l};
            }
        }
        float* const dd = reinterpret_cast<float*>(lds + buf * S::STAGE + S::WB);
#pragma unroll
        for (int e = 0; e < ND; ++e)
            dd[LPS > 1 ? t + 256 * e : t & 127] = rd[e];
    };

    f16v P[S::MT];
    Parts8 B[S::KT];
    const int col = 32 * panel + n;
#pragma unroll
    for (int mt = 0; mt < S::MT; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            P[mt][e] = 32 * mt + 8 * (e / 4) + 4 * h + e % 4 == col ? 1.f : 0.f;
    // d of rows 32 mt + 8 q + 4 h + 0..3, q = 0..3, from a stage
    auto scale = [&](const float* dd, int mt, float (&d)[16]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f4 x = *reinterpret_cast<const f4*>(dd + 32 * mt + 8 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) d[4 * q + e] = x[e];
        }
    };
    // A column of P, which a wave holds whole (lanes n and n + 32), stays above
    // 2^-60 in its largest element, so that its elements have parts, and P stands
    // for P 2^ex (large columns are scaled down as well, where float32 would
    // overflow).  Six elements of each half show that as a rule (of ReLU units
    // all six are idle once in 64), and only where they do not all are looked at.
    // A forward call without any of the range's checks, with all maxima at every
    // row, and with these, us: 357, 370, 363 at B 256, L 256, w 32; 1279, 1342,
    // 1254 at B 64, L 1024, w 64; 2322, 2350, 2305 at B 16, L 1024, w 128 (an odd
    // number of elements costs 5% at w = 64, in every other respect the same
    // code: where its loop falls).
    int ex = 0;
    auto largest = [&](int tiles, int count) {
        float m = 0.f;
#pragma unroll
        for (int mt = 0; mt < tiles; ++mt)
#pragma unroll
            for (int e = 0; e < count; ++e) m = fmaxf(m, fabsf(P[mt][3 * e % 16]));
        return m;
    };
    auto settle = [&] {
        // (the columns beyond w are zeros)
        const float some = EXACT || col < w ? largest(1, 6) : 1.f;
        const unsigned low = __float_as_uint(0x1p-60f), high = __float_as_uint(0x1p40f);
        if (__builtin_expect(
                __builtin_amdgcn_ballot_w64(__float_as_uint(some) - low > high - low) != 0, 0)) {
            float m = largest(S::MT, 16);
            m = fmaxf(m, __shfl_xor(m, 32, 64));
            const int k = m > 0x1p40f ? 64 : m > 0.f && m < 0x1p-60f ? -64 : 0;
            const float f = k > 0 ? 0x1p-64f : k < 0 ? 0x1p64f : 1.f;
            ex += k;
#pragma unroll
            for (int mt = 0; mt < S::MT; ++mt) P[mt] *= f;
        }
    };
    // Transposed system: a product meets diag(d) P, d of its own row.  Without
    // residuals P is kept as that (so that its columns are settled as they are
    // split), with them it is needed as it is.
    auto first_slopes = [&](int mt, float (&d)[16]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float x[4];
            load_row<4>(sd, ((unsigned)b * L + L - m0) * w, 32 * mt + 8 * q + 4 * h, w, x);
#pragma unroll
            for (int e = 0; e < 4; ++e) d[4 * q + e] = x[e];
        }
    };
    auto operands = [&](const float* dd, bool first) {
        settle();
#pragma unroll
        for (int mt = 0; mt < S::MT; ++mt) {
            float d[16];
            if constexpr (BWD) {
                if (!a.residual) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) d[e] = 1.f;
                } else if (first) {
                    first_slopes(mt, d);
                } else {
                    scale(dd, mt, d);
                }
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                float x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    x[j] = P[mt][8 * half + j];
                    if constexpr (BWD) x[j] *= d[8 * half + j];
                }
                B[2 * mt + half] = split8(x);
            }
        }
    };
    if (BWD && !a.residual)
#pragma unroll
        for (int mt = 0; mt < S::MT; ++mt) {
            float d[16];
            first_slopes(mt, d);
#pragma unroll
            for (int e = 0; e < 16; ++e) P[mt][e] *= d[e];
        }
    const float* const dbase =
        reinterpret_cast<const float*>(lds + S::WB) + v / S::MT * WP + 4 * h;
    request(0);
    put(0);
    request(1);
    operands(nullptr, true);
    for (int m = m0; m < m1; ++m) {
        const int st0 = WP == 128 ? 4 * (m - m0) : (m - m0) / LPS;
#pragma unroll
        for (int mt = 0; mt < S::MT; ++mt) {
            const int st = st0 + (SPL == 4 ? mt : 0);
            if (SPL == 4 || (mt == 0 && (m - m0) % LPS == 0)) {
                __syncthreads();  // stage st is in LDS, stage st - 1 is consumed
            }
            const int tile = WP == 128 ? 0 : WP == 64 ? 4 * mt : 2 * ((m - m0) % LPS);
            const char* in = lds + (st & 1) * S::STAGE + tile * 1024 + lane * 16;
            const float* dd = dbase + (st & 1) * (S::STAGE / 4) + 128 * ((m - m0) % LPS);
            Acc<f16v> acc = {};
            // a part of the weights is read for the next k tile as soon as its
            // last product of this one is issued; the scheduling barriers
            // keep that order and let everything else move
            Parts8 A;
            A.l = *reinterpret_cast<const b8*>(in + 2 * (S::WB / 3));
            A.m = *reinterpret_cast<const b8*>(in + S::WB / 3);
            A.h = *reinterpret_cast<const b8*>(in);
            if (SPL == 4 || (mt == 0 && (m - m0) % LPS == 0)) {
                // (past the last stage: its weights again, never read)
                put(st + 1);
                request(st + 2);
            }
            constexpr int kMove = 0x2 | 0x4 | 0x10 | 0x200;
#pragma unroll
            for (int k = 0; k < S::KT; ++k) {
                const char* const next = in + (k + 1) * 1024;
                const bool more = k + 1 < S::KT;
                acc.s = mfma32(A.l, B[k].h, acc.s);
                if (more) A.l = *reinterpret_cast<const b8*>(next + 2 * (S::WB / 3));
                __builtin_amdgcn_sched_barrier(kMove);
                acc.s = mfma32(A.m, B[k].m, acc.s);
                acc.s = mfma32(A.m, B[k].h, acc.s);
                if (more) A.m = *reinterpret_cast<const b8*>(next + S::WB / 3);
                __builtin_amdgcn_sched_barrier(kMove);
                acc.x = mfma32(A.h, B[k].h, acc.x);
                acc.s = mfma32(A.h, B[k].l, acc.s);
                acc.s = mfma32(A.h, B[k].m, acc.s);
                if (more) A.h = *reinterpret_cast<const b8*>(next);
                __builtin_amdgcn_sched_barrier(kMove);
            }
            if (__builtin_expect(scaled, 0)) {
                const float f = scale_at(m, mt);
                acc.x *= f;
                acc.s *= f;
            }
            float d[16];
            if constexpr (!BWD) scale(dd, mt, d);
            if (a.residual) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    P[mt][e] = BWD ? P[mt][e] + (acc.x[e] + acc.s[e])
                                   : fmaf(d[e], acc.x[e] + acc.s[e], P[mt][e]);
            } else {
                if constexpr (BWD) {
                    if (m + 1 < m1) {
                        scale(dd, mt, d);
                    } else {
#pragma unroll
                        for (int e = 0; e < 16; ++e) d[e] = 1.f;
                    }
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) P[mt][e] = d[e] * (acc.x[e] + acc.s[e]);
            }
        }
        const int last = st0 + SPL - 1;
        if (m + 1 < m1)
            operands(dbase + (last & 1) * (S::STAGE / 4) + 128 * ((m - m0) % LPS), false);
    }
    if (!live) return;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(ex != 0) != 0, 0))
#pragma unroll
        for (int mt = 0; mt < S::MT; ++mt)
#pragma unroll
            for (int e = 0; e < 16; ++e) P[mt][e] = ldexpf(P[mt][e], ex);
    float* out = a.P + ((long long)b * (a.C - 1) + c) * WP * WP + col;
#pragma unroll
    for (int mt = 0; mt < S::MT; ++mt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            out[(long long)(32 * mt + 8 * (e / 4) + 4 * h + e % 4) * WP] = P[mt][e];
}

// The vectors of chunks 0 .. C-2 first (the longer chain per row and few
// workgroups), then the products of chunks 1 .. C-2.
template <int WP, bool BWD, bool EXACT, bool PRE>
__global__ __launch_bounds__(kThr, WP == 128 ? 2 : 3) void chunk_pass(PanelArgs a) {
    __shared__ __attribute__((aligned(16))) char
        lds[ProdShape<WP>::LDS > VecShape<WP>::LDS ? ProdShape<WP>::LDS : VecShape<WP>::LDS];
    const int vg = (a.B + 16 * VecShape<WP>::GPW - 1) / (16 * VecShape<WP>::GPW);
    const int nv = vg * (a.C - 1);
    if ((int)blockIdx.x < nv) {
        vector_panel<WP, BWD, EXACT, false, PRE>(a, lds, blockIdx.x / vg, blockIdx.x % vg);
        return;
    }
    const int pg = (a.B + ProdShape<WP>::SYS - 1) / ProdShape<WP>::SYS;
    const int total = pg * (a.C - 2);
    // workgroups go round-robin to the 8 XCDs: consecutive items, which share
    // a chunk's weights, stay on one XCD and its L2
    const int id = (int)blockIdx.x - nv, per = (total + 7) / 8;
    const int item = (id & 7) * per + (id >> 3);
    if (item >= total || (id >> 3) >= per) return;
    product_panel<WP, BWD, EXACT, PRE>(a, lds, 1 + item / pg, item % pg);
}

template <int WP, bool BWD, bool EXACT, bool PRE>
__global__ __launch_bounds__(kThr) void apply_pass(PanelArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[VecShape<WP>::LDS];
    const int vg = (a.B + 16 * VecShape<WP>::GPW - 1) / (16 * VecShape<WP>::GPW);
    vector_panel<WP, BWD, EXACT, true, PRE>(a, lds, blockIdx.x / vg, blockIdx.x % vg);
}

// ------------------------------------------------------------ split weights
// The tiles of SplitShape from W (BWD: of W^T), 4 x 4 weights per thread, and
// per layer and 32 rows the factor that the results are to be multiplied by:
// 1, unless the largest weight of these rows is below 2^-60 or from 2^60 on;
// then *odd becomes the call's stamp.  (What is in *odd before needs no
// clearing: a stamp left there only makes a call read its factors.)  Without
// `out`, the factors alone.  The work of one workgroup, of those that
// layer_vectors' first launch of a call has beyond its own.
template <int WP, bool BWD, bool EXACT>
__device__ __forceinline__ void split_weights(const float* __restrict__ W, const PanelSplit& job,
                                              int block, int L, int w) {
    constexpr int UNITS = WP * WP / 16, WAVES = WP / 32;  // threads per layer, waves per 32 rows
    const int id = block * kThr + threadIdx.x;
    const int l = __builtin_amdgcn_readfirstlane(id / UNITS), u = id % UNITS;
    if (l >= L) return;
    const int rg = u & 7, cg = (u >> 3) % (WP / 4), mt = u / (2 * WP);
    const int i = 32 * mt + 4 * rg, k = 4 * cg;
    const Src<EXACT> Wl(W + (long long)l * w * w, w * w);
    f4 raw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x[4];
        load_row<4>(Wl, ((BWD ? k : i) + e) * w, BWD ? i : k, w, x);
        raw[e] = f4{x[0], x[1], x[2], x[3]};
    }
    unsigned big = 0u;
#pragma unroll
    for (int e = 0; e < 16; ++e) big = max(big, __float_as_uint(fabsf(raw[e / 4][e % 4])));
    for (int off = 32; off > 0; off >>= 1)
        big = max(big, (unsigned)__shfl_xor((int)big, off, 64));
    if constexpr (WAVES > 1) {  // (all of a workgroup has a layer, or none)
        __shared__ unsigned part[4];
        const int v = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) part[v] = big;
        __syncthreads();
        for (int k = 0; k < WAVES; ++k) big = max(big, part[v / WAVES * WAVES + k]);
    }
    const float m = __uint_as_float(big);
    const float f = m >= 0x1p60f && m < __builtin_inff() ? 0x1p-64f
                    : m > 0.f && m < 0x1p-60f            ? 0x1p64f
                                                         : 1.f;
    if (u % (2 * WP) == 0) {
        job.scale[(long long)l * (WP / 32) + mt] = 1.f / f;
        if (f != 1.f) *job.odd = job.stamp;
    }
    if (!job.out) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) raw[e] *= f;
    char* dst = job.out + (long long)l * SplitShape<WP>::LAYER +
                (WP == 128 ? mt * SplitShape<WP>::SLICE : mt * (WP / 16) * 1024) + cg / 4 * 1024 +
                (4 * rg + 32 * (cg & 1)) * 16 + 8 * ((cg >> 1) & 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const f4 x = BWD ? f4{raw[0][e], raw[1][e], raw[2][e], raw[3][e]} : raw[e];
        const Parts2 p = split2(x[0], x[1]), q = split2(x[2], x[3]);
        *reinterpret_cast<u2*>(dst + e * 16) = u2{p.h, q.h};
        *reinterpret_cast<u2*>(dst + e * 16 + SplitShape<WP>::PART) = u2{p.m, q.m};
        *reinterpret_cast<u2*>(dst + e * 16 + 2 * SplitShape<WP>::PART) = u2{p.l, q.l};
    }
}

// ------------------------------------------------------------ layer vectors
// d = c sigma'(a) and, forward, r = f(Z_{l-1}) - Z_l with its maximum (where
// red is given), for a = W_l Z_{l-1} + b_l.  Items (layer, 16 systems), a
// contiguous range of them per group of waves, which keeps a layer's split
// weights in registers for all its systems.  Bound by one read of W and of the
// states and the write of d and r.  One atomic per workgroup, at most 2048 of
// them (L = 8192, w = 32, B = 1: 42 us with one per wave and a workgroup per
// layer).  Workgroups from `own` on split the weights, which shares the read of W
// and saves a launch per call (2-3 us where B and L are small).
template <int WP, bool BWD, bool EXACT>
__global__ __launch_bounds__(kThr) void layer_vectors(
    const float* __restrict__ W, const float* __restrict__ bias, const float* __restrict__ z0,
    const float* __restrict__ Z, float* __restrict__ d_out, float* __restrict__ r_out,
    unsigned* __restrict__ clear, unsigned* __restrict__ red, int B, int L, int w_, int layer,
    float alpha, int per, int own, PanelSplit job) {
    using S = VecShape<WP>;
    constexpr int NR = S::NR;
    const int t = threadIdx.x, v = t >> 6, lane = t & 63;
    const int sub = v / S::WPG, wv = v % S::WPG;
    const int n = lane & 15, g = lane >> 4;
    const int w = EXACT ? WP : w_;
    const int base = wv * 16 * S::MTW, r0 = base + NR * g;
    if ((int)blockIdx.x >= own) {
        split_weights<WP, BWD, EXACT>(W, job, blockIdx.x - own, L, w);
        return;
    }
    if constexpr (!BWD)
        if (blockIdx.x == 0)
            for (int k = t; k < 2 * kRedShards; k += kThr) clear[k] = 0u;
    const int ng = (B + 15) / 16;
    const unsigned nv = (unsigned)B * L * w;
    const Src<EXACT> sz(Z, nv), s0(z0, (unsigned)B * w);
    const bool res = layer_residual(layer);
    const int k0 = 16 * (g / 2) + 4 * (g % 2);
    const int it0 = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * S::GPW + sub) * per);
    const int it1 = min(it0 + per, L * ng);
    Parts8 A[S::MTW][S::KT];
    float bi[NR];
    int have = -1;
    unsigned mr = 0u;
    for (int it = it0; it < it1; ++it) {
        const int l = it / ng, gr = it - l * ng;
        const float* Wl = W + (long long)l * w * w;
        if (l != have) {
            float raw[S::MTW][S::KT][8];
            load_strip<WP, false, EXACT>(Src<EXACT>(Wl, w * w), w, base, n, g, raw);
            load_row<NR>(Src<EXACT>(bias + (long long)l * w, w), 0, r0, w, bi);
#pragma unroll
            for (int q = 0; q < S::MTW; ++q)
#pragma unroll
                for (int k = 0; k < S::KT; ++k) A[q][k] = split8(raw[q][k], kShift);
            have = l;
        }
        const int bb = gr * 16 + n;
        const bool live = bb < B;
        const int b = live ? bb : B - 1;
        const unsigned op = l == 0 ? b * w : ((unsigned)b * L + l - 1) * w;
        const unsigned o = ((unsigned)b * L + l) * w;
        float zl[NR], zr[NR], x[S::KT][8];
        if (l == 0) {
#pragma unroll
            for (int k = 0; k < S::KT; ++k) load_operand(s0, op, 32 * k + k0, w, x[k]);
            if (!BWD && res) load_row<NR>(s0, op, r0, w, zr);
        } else {
#pragma unroll
            for (int k = 0; k < S::KT; ++k) load_operand(sz, op, 32 * k + k0, w, x[k]);
            if (!BWD && res) load_row<NR>(sz, op, r0, w, zr);
        }
        if constexpr (!BWD) load_row<NR>(sz, o, r0, w, zl);
        Acc<f4> acc[S::MTW] = {};
#pragma unroll
        for (int k = 0; k < S::KT; ++k) {
            const Parts8 p = split8(x[k], kShift);
#pragma unroll
            for (int q = 0; q < S::MTW; ++q) mac(acc[q], A[q][k], p);
        }
        float dv[NR], rv[NR];
#pragma unroll
        for (int q = 0; q < S::MTW; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = S::MTW * e + q;
                float y = fmaf(acc[q].x[e] + acc[q].s[e], kUnshift * kUnshift, bi[j]);
                // where a factor has no parts, or the sum no shift, the row is
                // summed as it stands
                if (__builtin_expect(!(fabsf(y) < __builtin_inff()), 0)) {
                    const float* zp = l == 0 ? z0 : Z;
                    y = bi[j];
                    if (EXACT || r0 + j < w)
                        for (int k = 0; k < w; ++k)
                            y = fmaf(Wl[(long long)(r0 + j) * w + k], zp[(long long)op + k], y);
                }
                float dd;
                const float f = activate(layer, y, &dd);
                dv[j] = res ? alpha * dd : dd;
                if constexpr (!BWD) {
                    rv[j] = (res ? fmaf(alpha, f, zr[j]) : f) - zl[j];
                    if (live && (EXACT || r0 + j < w))
                        mr = max(mr, __float_as_uint(fabsf(rv[j])));
                }
            }
        if (live) {
            store_row<NR, EXACT>(d_out + o, r0, w, dv);
            if constexpr (!BWD) store_row<NR, EXACT>(r_out + o, r0, w, rv);
        }
    }
    if constexpr (!BWD) {
        if (!red) return;
        __shared__ unsigned part[4];
        for (int off = 32; off > 0; off >>= 1) mr = max(mr, (unsigned)__shfl_xor((int)mr, off, 64));
        if (lane == 0) part[v] = mr;
        __syncthreads();
        if (t == 0) {
            for (int i = 1; i < 4; ++i) mr = max(mr, part[i]);
            atomicMax(red + kRedF + (int)(blockIdx.x % kRedShards), mr);
        }
    }
}

int padded(int w) { return w <= 32 ? 32 : w <= 64 ? 64 : 128; }

// K with the padded width, whether w is it, and the template arguments given
#define DEEPPCR_PANEL(KERNEL, GRID, ...)                                                      \
    do {                                                                                      \
        const dim3 grid_((unsigned)(GRID)), thr_(kThr);                                       \
        switch (a_w) {                                                                        \
            case 32: hipLaunchKernelGGL(KERNEL(32, true), grid_, thr_, 0, st, __VA_ARGS__); break;   \
            case 64: hipLaunchKernelGGL(KERNEL(64, true), grid_, thr_, 0, st, __VA_ARGS__); break;   \
            case 128: hipLaunchKernelGGL(KERNEL(128, true), grid_, thr_, 0, st, __VA_ARGS__); break; \
            default:                                                                          \
                if (a_w < 32) hipLaunchKernelGGL(KERNEL(32, false), grid_, thr_, 0, st, __VA_ARGS__); \
                else if (a_w < 64) hipLaunchKernelGGL(KERNEL(64, false), grid_, thr_, 0, st, __VA_ARGS__); \
                else hipLaunchKernelGGL(KERNEL(128, false), grid_, thr_, 0, st, __VA_ARGS__); \
        }                                                                                     \
    } while (0)
#define LAYER_VECTORS_F(WP, EX) (layer_vectors<WP, false, EX>)
#define LAYER_VECTORS_B(WP, EX) (layer_vectors<WP, true, EX>)
#define CHUNK_F(WP, EX) (chunk_pass<WP, false, EX, false>)
#define CHUNK_B(WP, EX) (chunk_pass<WP, true, EX, false>)
#define CHUNK_FP(WP, EX) (chunk_pass<WP, false, EX, true>)
#define CHUNK_BP(WP, EX) (chunk_pass<WP, true, EX, true>)
#define APPLY_F(WP, EX) (apply_pass<WP, false, EX, false>)
#define APPLY_B(WP, EX) (apply_pass<WP, true, EX, false>)
#define APPLY_FP(WP, EX) (apply_pass<WP, false, EX, true>)
#define APPLY_BP(WP, EX) (apply_pass<WP, true, EX, true>)

int vector_groups(int B, int WP) {
    const int per = WP == 32 ? 32 : 16;
    return (B + per - 1) / per;
}
int product_groups(int B, int WP) {
    const int per = 128 / WP;
    return (B + per - 1) / per;
}

}  // namespace

bool panel_width(int w) { return w > 16 && w <= kMaxWidth; }
int panel_pad(int w) { return padded(w); }

// Chunks of a solve, by the estimated time of its parts (us), measured on one
// MI355X over B 1-256 and L 128-8192: a row of the products while there is a
// workgroup per CU at most (beyond, in proportion; at a padded width of 128,
// where two share a CU, twice as much up to 512 workgroups), a row of the
// apply pass, a launch, and the solve over the chunk ends.  B = 16, L = 1024,
// w = 128: 946 us with 8 chunks, 521 with 16, 423 with 32, 447 with 96.
int panel_chunks(int B, int rows, int w) {
    const int WP = padded(w), k = WP == 32 ? 0 : WP == 64 ? 1 : 2;
    static const double prod[] = {0.58, 1.48, 4.75}, apply[] = {0.5, 0.72, 2.6};
    const int pg = product_groups(B, WP), vg = vector_groups(B, WP);
    int best = 1;
    double t_best = 4.0 + rows * apply[k];
    for (int j = 4; j <= 44; ++j) {
        const int C = ((4 + j % 4) << (j / 4)) >> 2;  // 2, 2, 3, 3, 4, 5, 6, 7, 8, 10, ...
        if (C > rows) break;
        const int Lc = (rows + C - 1) / C;
        const double wgs = ((double)pg * (C - 2) + (double)vg * (C - 1)) / 256.0;
        double row = C == 2 ? apply[k] : prod[k];
        if (C > 2 && wgs > 1.0) row *= WP != 128 ? (wgs > 1.2 ? 0.85 * wgs : 1.0) : wgs > 2.0 ? wgs : 2.0;
        double t = 8.0 + Lc * (row + apply[k] * ((double)vg * C > 512 ? vg * C / 512.0 : 1.0));
        if (t < t_best && C > 2) t += block_plan(B, C - 1, WP, nullptr);
        if (t < t_best) {
            t_best = t;
            best = C;
        }
    }
    return best;
}

// The kernels address the vectors of a batch by 32-bit bytes: more systems
// than that takes go in several launches, launch(first system, systems).
template <class F>
static hipError_t by_systems(int B, int L, int w, F&& launch) {
    const long long most = ((1LL << 30) - 1) / ((long long)L * w);
    if (most < 1) return hipErrorInvalidValue;
    for (long long b = 0; b < B; b += most) {
        const hipError_t e = launch(b, (int)(B - b < most ? B - b : most));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
// The arguments of systems b .. b + n - 1.
static PanelArgs systems(PanelArgs a, bool bwd, long long b, int n) {
    const long long v = b * a.L * a.w, WP = padded(a.w), ends = b * (a.C - 1) * WP;
    a.d += v;
    a.r += bwd ? b * a.w : v;
    if (bwd) {
        a.Lambda += v;
        a.dz0 += b * a.w;
    } else {
        a.Z += v;
    }
    if (a.C > 1) {
        a.P += ends * WP;
        a.q += ends;
        if (a.xe) a.xe += ends;
    }
    a.B = n;
    return a;
}

static hipError_t layer_vectors_some(bool bwd, const float* W, const float* bias, const float* z0,
                                     const float* Z, float* d, float* r, unsigned* red,
                                     bool want_max, int B, int L, int w, int layer, float alpha,
                                     const PanelSplit* split, hipStream_t st) {
    // one item per group of waves, or up to 2048 workgroups
    const int WP = padded(w), groups = WP == 32 ? 2 : 1;
    const int items = L * ((B + 15) / 16);
    const int per = (items + 2048 * groups - 1) / (2048 * groups);
    const int own = (items + per * groups - 1) / (per * groups);
    const long long grid =
        own + (split ? ((long long)L * WP * WP / 16 + kThr - 1) / kThr : 0);
    const PanelSplit job = split ? *split : PanelSplit{};
    unsigned* const mx = want_max ? red : nullptr;
    const int a_w = w;
    if (bwd)
        DEEPPCR_PANEL(LAYER_VECTORS_B, grid, W, bias, z0, Z, d, r, red, mx, B, L, w, layer,
                      alpha, per, own, job);
    else
        DEEPPCR_PANEL(LAYER_VECTORS_F, grid, W, bias, z0, Z, d, r, red, mx, B, L, w, layer,
                      alpha, per, own, job);
    return hipGetLastError();
}

hipError_t launch_layer_vectors(bool bwd, const float* W, const float* bias, const float* z0,
                                const float* Z, float* d, float* r, unsigned* red, bool want_max,
                                int B, int L, int w, int layer, float alpha,
                                const PanelSplit* split, hipStream_t st) {
    return by_systems(B, L, w, [&](long long b, int n) {
        const long long v = b * L * w;
        return layer_vectors_some(bwd, W, bias, z0 + b * w, Z + v, d + v, bwd ? r : r + v, red,
                                  want_max, n, L, w, layer, alpha, b == 0 ? split : nullptr, st);
    });
}

size_t split_bytes(int L, int w) { return (size_t)L * padded(w) * padded(w) * 6; }
size_t split_scales(int L, int w) { return (size_t)L * (padded(w) / 32); }

static hipError_t chunk_pass_some(bool bwd, const PanelArgs& a, hipStream_t st) {
    const int WP = padded(a.w), a_w = a.w;
    const long long nv = (long long)vector_groups(a.B, WP) * (a.C - 1);
    const long long np = (long long)product_groups(a.B, WP) * (a.C - 2);
    const long long grid = nv + (np + 7) / 8 * 8;
    if (bwd && a.S) DEEPPCR_PANEL(CHUNK_BP, grid, a);
    else if (bwd) DEEPPCR_PANEL(CHUNK_B, grid, a);
    else if (a.S) DEEPPCR_PANEL(CHUNK_FP, grid, a);
    else DEEPPCR_PANEL(CHUNK_F, grid, a);
    return hipGetLastError();
}

static hipError_t apply_pass_some(bool bwd, const PanelArgs& a, hipStream_t st) {
    const int a_w = a.w;
    const long long grid = (long long)vector_groups(a.B, padded(a.w)) * a.C;
    if (bwd && a.S) DEEPPCR_PANEL(APPLY_BP, grid, a);
    else if (bwd) DEEPPCR_PANEL(APPLY_B, grid, a);
    else if (a.S) DEEPPCR_PANEL(APPLY_FP, grid, a);
    else DEEPPCR_PANEL(APPLY_F, grid, a);
    return hipGetLastError();
}

hipError_t launch_chunk_pass(bool bwd, const PanelArgs& a, hipStream_t st) {
    return by_systems(a.B, a.L, a.w, [&](long long b, int n) {
        return chunk_pass_some(bwd, systems(a, bwd, b, n), st);
    });
}

hipError_t launch_apply_pass(bool bwd, const PanelArgs& a, hipStream_t st) {
    return by_systems(a.B, a.L, a.w, [&](long long b, int n) {
        return apply_pass_some(bwd, systems(a, bwd, b, n), st);
    });
}

}  // namespace deeppcr
