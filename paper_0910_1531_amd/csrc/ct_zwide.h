// Z1 and Z2 of small grids: one wave per transform.  A block holds four columns and eight waves; the
// forward transforms of its columns run side by side, one field a wave, in LDS that only the wave touches
// (wave-level fences); then all threads share the nodes of the block for the spectral products, and the
// inverse transforms run side by side.  The same arithmetic in the same order as k_z1c and k_z2c, which
// run their nine or ten transforms one after the other: at small sizes a pass lasts as long as that chain.
#pragma once

#include "ct_kernels.h"

namespace dft {

constexpr int kZWideCols = 4, kZWideThreads = 512;

template <typename T, int L>
struct ZWideTile {
    using F = ct::Fft<T, typename ct::PlanT<T, L>::type, kZWideCols, 64, false, 1, 0, true>;
    static constexpr int LDS = 8 * F::TILE * (int)sizeof(cx<T>);
};

template <typename T, int L, int MS>
__global__ __launch_bounds__(kZWideThreads) void k_z1w(Geo g_in, Z1Args a) {
    using F = typename ZWideTile<T, L>::F;
    constexpr int P = kZWideCols;
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[8 * F::TILE];
    const Consts &c = *g.cs;
    const int S = g.S;
    const long long NC = g.NC, rs = (long long)g.ny * g.Kx;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    cx<T> *tile = lds + wave * F::TILE;
    const ZTile zt = z_tile<P>(g);   // (every node of a thread lies in one column)
    const cx<T> *tw = twp<T>(g, 2);
    const bool n3 = n3_wanted(a.n3_only);
    const bool es = MS > 0 && c.es && !n3;
    const ZWaveOf<T, L> kw(c, zt.x, zt.y);
    [[maybe_unused]] const Z1Const<T, (MS > 0 ? MS : 1)> kc(c);
    constexpr bool TAB = z_fp64_factors<T, L>();
    const double *tab = TAB ? g.tab64 + zt.off : nullptr;
    [[maybe_unused]] const long long TS = z_tab_row<L>(rs);
    cx<T> v[F::V];
    if (wave < S) {
        const cx<T> *src = reinterpret_cast<const cx<T> *>(a.specA) + (long long)wave * NC + zt.off;
#pragma unroll
        for (int i = 0; i < F::template nin<-1>(); ++i) {
            int p, e;
            const bool ok = F::template in_pos<-1>(i, p, e, lane);
            v[i] = (ok && p < zt.Pact) ? ct::gld(src + e * rs + p) : mk<T>(T(0), T(0));
        }
        typename F::template TwReg<-1> twf;
        F::template load_tw<-1>(twf, tw, lane);
        F::template run<-1>(v, tile, lane, twf);
        F::sync();
#pragma unroll
        for (int i = 0; i < F::template nout<-1>(); ++i) {
            int p, e;
            if (F::template out_pos<-1>(i, p, e, lane)) tile[F::lidx(p, e)] = v[i];
        }
    }
    __syncthreads();
    // products: a thread reads the species values of its nodes and leaves the inputs of the inverse
    // transforms in their place
    [[maybe_unused]] Poisson<T> pd;
    if constexpr (!TAB && MS > 0) pd = Poisson<T>(g, c, zt.x, zt.y);
    const T invN = T(c.invN);
    for (int j = (int)threadIdx.x; j < L * P; j += kZWideThreads) {
        const int e = j / P, p = j % P;
        if (p >= zt.Pact) continue;
        const long long ti = e * rs + p;
        cx<T> *nv = lds + F::lidx(p, e);
        cx<T> acc[5];
        if constexpr (MS == 0) {
#pragma unroll
            for (int m = 0; m < 5; ++m) acc[m] = mk<T>(T(0), T(0));
            for (int s = 0; s < S; ++s) z1_species<T>(c, kw, tab, TS, S, s, e, true, z_tab<L>(e) * rs + p, nv[s * F::TILE], acc);
        } else {
            cx<T> u[MS];
#pragma unroll
            for (int s = 0; s < MS; ++s) u[s] = s < S ? nv[s * F::TILE] : mk<T>(T(0), T(0));
            z1_node<TAB>(kc, a.diff != 0, kw, pd, tab, TS, NC, S, es, e, true, z_tab<L>(e) * rs + p, u, acc,
                           reinterpret_cast<cx<T> *>(a.specA) + zt.off + ti);
        }
        if (n3) {
            nv[0] = mk<T>(acc[3].x * invN, acc[3].y * invN);
            continue;
        }
        const T kz = kw.comp(e, 2);
#pragma unroll
        for (int t = 0; t < 7; ++t) {
            cx<T> sm = acc[t < 5 ? t : (t == 5 ? 4 : 3)];
            if (t >= 5) sm = mk<T>(kz * sm.y, -kz * sm.x);   // -i k_z s
            nv[t * F::TILE] = mk<T>(sm.x * invN, sm.y * invN);
        }
    }
    __syncthreads();
    const int t = wave;
    if (t >= (n3 ? 1 : 7)) return;
    asm volatile("" : "+v"(lane));
    typename F::template TwReg<1> twi;
    F::template load_tw<1>(twi, tw, lane);
    F::template get<F::template rad<1>(0)>(v, tile, lane);
    F::template run<1>(v, tile, lane, twi);
    // store the transform as output o, times -i k_d for d = 0 (x) or 1 (y), plain for d < 0
    auto store = [&](int o, int d) {
        cx<T> *dst = reinterpret_cast<cx<T> *>(a.specB) + (long long)o * NC + zt.off;
#pragma unroll
        for (int i = 0; i < F::template nout<1>(); ++i) {
            int p, e;
            if (!(F::template out_pos<1>(i, p, e, lane) && p < zt.Pact)) continue;
            cx<T> w = v[i];
            if (d >= 0) {
                const T kd = kw.comp(e, d);
                w = mk<T>(kd * w.y, -kd * w.x);
            }
            ct::gst(dst + e * rs + p, w);
        }
    };
    if (n3) {
        store(0, -1);
    } else if (g.compact || t < 3 || t >= 5) {
        store(t < 5 ? t : (t == 5 ? 6 : 9), -1);
    } else if (t == 3) {
        store(3, -1);
        store(7, 0);
        store(8, 1);
    } else {
        store(4, 0);
        store(5, 1);
    }
}

template <typename T, int L>
__global__ __launch_bounds__(kZWideThreads) void k_z2w(Geo g_in, Z2Args a) {
    using F = typename ZWideTile<T, L>::F;
    constexpr int P = kZWideCols;
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[8 * F::TILE];
    const Consts &c = *g.cs;
    const int S = g.S;
    const long long NC = g.NC, rs = (long long)g.ny * g.Kx;
    const int t = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);   // the wave's transform, as in k_z2c
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    cx<T> *tile = lds + t * F::TILE;
    const ZTile zt = z_tile<P>(g);   // (every node of a thread lies in one column)
    const cx<T> *tw = twp<T>(g, 2);
    const ZWaveOf<T, L> kw(c, zt.x, zt.y);
    const cx<T> *specB = reinterpret_cast<const cx<T> *>(a.specB) + zt.off;
    cx<T> v[F::V];
    if (g.compact || t < 4 || t == 5 || t == 7) {
        const cx<T> *src = specB + (long long)(t < 5 ? t : (t == 5 ? 6 : (t == 6 ? 7 : 9))) * NC;
#pragma unroll
        for (int i = 0; i < F::template nin<-1>(); ++i) {
            int p, e;
            const bool ok = F::template in_pos<-1>(i, p, e, lane);
            v[i] = (ok && p < zt.Pact) ? ct::gld(src + e * rs + p) : mk<T>(T(0), T(0));
        }
    } else {
        // the x and y components of a vector derivative combined before one transform
        const cx<T> *sx = specB + (long long)(t == 4 ? 4 : 7) * NC, *sy = sx + NC;
#pragma unroll
        for (int i = 0; i < F::template nin<-1>(); ++i) {
            int p, e;
            const bool ok = F::template in_pos<-1>(i, p, e, lane) && p < zt.Pact;
            cx<T> w = mk<T>(T(0), T(0));
            if (ok) {
                const cx<T> fx = ct::gld(sx + e * rs + p), fy = ct::gld(sy + e * rs + p);
                const T kx = kw.comp(e, 0), ky = kw.comp(e, 1);
                w = mk<T>(-(kx * fx.y + ky * fy.y), kx * fx.x + ky * fy.x);   // i k_x fx + i k_y fy
            }
            v[i] = w;
        }
    }
    {
        typename F::template TwReg<-1> twf;
        F::template load_tw<-1>(twf, tw, lane);
        F::template run<-1>(v, tile, lane, twf);
        F::sync();
    }
#pragma unroll
    for (int i = 0; i < F::template nout<-1>(); ++i) {
        int p, e;
        if (!F::template out_pos<-1>(i, p, e, lane)) continue;
        cx<T> w = v[i];
        if (t == 5 || t == 7) {
            const T kd = kw.comp(e, 2);
            w = mk<T>(-kd * w.y, kd * w.x);   // + i k_z w
        }
        tile[F::lidx(p, e)] = w;
    }
    __syncthreads();
    const T invN = T(c.invN);
    for (int j = (int)threadIdx.x; j < L * P; j += kZWideThreads) {
        const int e = j / P, p = j % P;
        if (p >= zt.Pact) continue;
        const long long ti = e * rs + p;
        cx<T> *nv = lds + F::lidx(p, e);
        cx<T> u[6];
#pragma unroll
        for (int m = 0; m < 4; ++m) u[m] = nv[m * F::TILE];
        u[4] = add(nv[4 * F::TILE], nv[5 * F::TILE]);
        u[5] = add(nv[6 * F::TILE], nv[7 * F::TILE]);
        const T kmag = kw.kmag(e);
        for (int is = 0; is < S; ++is) {
            const T Ri = T(c.R[is]), a0 = T(c.i4piR2[is]), a1 = T(c.i4piR[is]);
            T w2, w3;
            if constexpr (std::is_same<T, double>::value) {
                const double *tab = g.tab64 + zt.off + z_tab<L>(e) * rs + p;
                w2 = ct::cld(tab + (long long)is * z_tab_row<L>(rs));
                w3 = ct::cld(tab + (long long)(S + is) * z_tab_row<L>(rs));
            } else {
                weight_w2_w3<T>(kmag, Ri, w2, w3);
            }
            const cx<T> ev = c.es ? ct::gld(reinterpret_cast<const cx<T> *>(a.specA) + (long long)is * NC + zt.off + ti)
                                  : mk<T>(T(0), T(0));
            const T s2x = u[0].x * a0 + u[1].x * a1 + u[2].x;
            const T s2y = u[0].y * a0 + u[1].y * a1 + u[2].y;
            const T s3x = u[3].x + u[4].x * a1 + u[5].x;
            const T s3y = u[3].y + u[4].y * a1 + u[5].y;
            T ex = -(s2x * w2 + s3x * w3);
            T ey = -(s2y * w2 + s3y * w3);
            ex += ev.x;
            ey += ev.y;
            nv[is * F::TILE] = mk<T>(ex * invN, ey * invN);
        }
    }
    __syncthreads();
    if (t >= S) return;
    asm volatile("" : "+v"(lane));
    typename F::template TwReg<1> twi;
    F::template load_tw<1>(twi, tw, lane);
    F::template get<F::template rad<1>(0)>(v, tile, lane);
    F::template run<1>(v, tile, lane, twi);
    cx<T> *dst = reinterpret_cast<cx<T> *>(a.specA) + (long long)t * NC + zt.off;
#pragma unroll
    for (int i = 0; i < F::template nout<1>(); ++i) {
        int p, e;
        if (F::template out_pos<1>(i, p, e, lane) && p < zt.Pact) ct::gst(dst + e * rs + p, v[i]);
    }
}

#define DFT_ZWIDE_LENGTHS(X) \
    X(8) X(9) X(12) X(16) X(18) X(24) X(27) X(32) X(36) X(48) X(54) X(64) X(72) X(81) X(96) X(108) X(128) X(144) X(162) \
    X(192) X(216) X(243) X(256)

// The rule: few blocks of four columns, so that all are in flight at once (the longer the pencils, the
// fewer fit a CU).  Measured FP64, us, one block per tile / one wave per transform, Z1 and Z2: 24^3 (78
// blocks) 14.0 / 9.0 and 15.9 / 8.4; 32^3 (136) 12.4 / 9.6 and 15.8 / 8.1; 48^3 (300) 18.1 / 13.1 and
// 20.6 / 13.2; 64^3 (528) 20.7 / 18.7 and 20.3 / 13.3; 32 x 32 x 192 33 / 20 and 39 / 20; against
// 48 x 48 x 128 (300) 24.9 / 29.2, 32 x 32 x 243 30.7 / 33.1 (spills), FP32 72^3 (666) 22.7 / 27.1.
// Z2 stays ahead for longer: 384 x 16 x 16 (772) 14.3 / 10.4 but Z1 11.9 / 12.7, FP32 128 x 64 x 48
// (1040) 17.9 / 16.7 but Z1 21.6 / 27.0.
template <typename T, int L, bool Z2>
bool z_wide(const Geo &g) {
    constexpr long long most = sizeof(T) == 8 && L > 192 ? 0 : Z2 && L <= 48 ? 1100 : L <= 64 ? 640 : L <= 96 ? 384 : 256;
    return ct_cdiv((long long)g.ny * g.Kx, kZWideCols) * g.nprob <= most;
}

template <typename T, int L>
bool launch_z1w_len(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    if constexpr (sizeof(T) == 8 && L > 192) {
        return false;
    } else {
        if (!z_wide<T, L, false>(g)) return false;
        const dim3 grid((unsigned)ct_cdiv((long long)g.ny * g.Kx, kZWideCols), 1, (unsigned)g.nprob), block(kZWideThreads);
        if (!es) hipLaunchKernelGGL((k_z1w<T, L, 0>), grid, block, 0, s, g, a);
        else if (g.S <= 2) hipLaunchKernelGGL((k_z1w<T, L, 2>), grid, block, 0, s, g, a);
        else if (g.S == 3) hipLaunchKernelGGL((k_z1w<T, L, 3>), grid, block, 0, s, g, a);
        else hipLaunchKernelGGL((k_z1w<T, L, 4>), grid, block, 0, s, g, a);
        ct_check("z1 (one wave per transform)");
        return true;
    }
}

template <typename T, int L>
bool launch_z2w_len(const Geo &g, const Z2Args &a, hipStream_t s) {
    if constexpr (sizeof(T) == 8 && L > 192) {
        return false;
    } else {
        if (!z_wide<T, L, true>(g)) return false;
        const dim3 grid((unsigned)ct_cdiv((long long)g.ny * g.Kx, kZWideCols), 1, (unsigned)g.nprob);
        hipLaunchKernelGGL((k_z2w<T, L>), grid, dim3(kZWideThreads), 0, s, g, a);
        ct_check("z2 (one wave per transform)");
        return true;
    }
}

// Whether Z1 (Z2) of the grid takes the kernels here, whatever the tuned shape.
template <typename T>
bool z1_is_wide(const Geo &g) {
    switch (g.nz) {
#define DFT_CASE(n) case n: return z_wide<T, n, false>(g);
        DFT_ZWIDE_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}
template <typename T>
bool z2_is_wide(const Geo &g) {
    switch (g.nz) {
#define DFT_CASE(n) case n: return z_wide<T, n, true>(g);
        DFT_ZWIDE_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

// False where the rule takes the kernels with one block per tile, or the length has no kernel here.
template <typename T>
bool launch_z1_wide(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    switch (g.nz) {
#define DFT_CASE(n) case n: return launch_z1w_len<T, n>(g, a, es, s);
        DFT_ZWIDE_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

template <typename T>
bool launch_z2_wide(const Geo &g, const Z2Args &a, hipStream_t s) {
    if (a.mode != Z2_EL) return false;
    switch (g.nz) {
#define DFT_CASE(n) case n: return launch_z2w_len<T, n>(g, a, s);
        DFT_ZWIDE_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

}  // namespace dft
