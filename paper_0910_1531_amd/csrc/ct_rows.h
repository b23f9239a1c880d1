// Rows of the x passes.  Two real rows (r0, r0 + 1) travel as the real and imaginary parts of one
// complex row: the forward transform C of c = a + i b gives A_k = (C_k + conj C_{L-k}) / 2 and
// B_k = (C_k - conj C_{L-k}) / (2i); the inverse rebuilds C from the half spectra.  A tile of row
// pairs belongs to one wave, so its exchanges through LDS need wave-level fences only.
#pragma once

#include "ct_kernels.h"

namespace dft {

// Row lengths, in groups: the X2 kernels of a group are a code object of their own (ct_launch_x2.hip), since the
// runtime loads a whole code object at the first launch from it (about 1.3 ms per MB).
#define DFT_X_GROUP_0(X) X(8) X(9) X(12) X(16) X(18)
#define DFT_X_GROUP_1(X) X(24) X(27) X(32) X(36) X(48)
#define DFT_X_GROUP_2(X) X(54) X(64) X(72) X(81) X(96)
#define DFT_X_GROUP_3(X) X(108) X(128) X(144) X(162) X(192)
#define DFT_X_GROUP_4(X) X(216) X(243) X(256) X(288) X(324)
#define DFT_X_GROUP_5(X) X(384) X(432) X(486) X(512)
constexpr int kXGroups = 6;
#define DFT_X_LENGTHS(X) \
    DFT_X_GROUP_0(X) DFT_X_GROUP_1(X) DFT_X_GROUP_2(X) DFT_X_GROUP_3(X) DFT_X_GROUP_4(X) DFT_X_GROUP_5(X)

// Element at a 32-bit byte offset of a base that all lanes share: the base stays in scalar registers
// and a lane holds one register of address.
template <typename V>
__device__ __forceinline__ V *at(V *base, unsigned off) {
    return reinterpret_cast<V *>(reinterpret_cast<char *>(const_cast<typename std::remove_const<V>::type *>(base)) + off);
}

template <int L>
struct XRow {
    static constexpr int PW = 256 / L > 0 ? 256 / L : 1;   // row pairs of a wave: about one radix-4 butterfly a lane
    static constexpr int KX = L / 2 + 1;
    static constexpr bool EVEN = L % 2 == 0;
    static constexpr int KH = (L + 1) / 2;                 // elements that are not their own mirror image, and k = 0
    static constexpr int NIT = (PW * KH + 63) / 64;
    static_assert(2 * PW <= 64, "one lane per row for the Nyquist elements");
    template <typename T>
    using F = ct::Fft<T, typename ct::XPlan<L>::type, PW, 64, true, 1, 0, true>;
};

// Half spectra of the rows of a wave's pairs in registers: elements below L/2 of both rows of every
// pair (lanes along k), and the Nyquist elements, one row a lane.
template <typename T, int L>
struct HalfRows {
    using X = XRow<L>;
    cx<T> A[X::NIT], B[X::NIT], Q;

    // in: first row's half spectrum (the same for all lanes); rows past rows_here read as zero
    __device__ __forceinline__ void load(const cx<T> *in, int rows_here, int lane) {
        constexpr unsigned CB = sizeof(cx<T>);
        const cx<T> z = mk<T>(T(0), T(0));
#pragma unroll
        for (int it = 0; it < X::NIT; ++it) {
            const int i = lane + it * 64;
            const int p = i / X::KH, k = i - p * X::KH;
            const unsigned o = (unsigned)(2 * p * X::KX + k) * CB;
            A[it] = B[it] = z;
            if (2 * p < rows_here) A[it] = ct::gld(at(in, o));
            if (2 * p + 1 < rows_here) B[it] = ct::gld(at(in, o + X::KX * CB));
        }
        Q = z;
        if (X::EVEN && lane < rows_here) Q = ct::gld(at(in, (unsigned)(lane * X::KX + L / 2) * CB));
    }

    // C = A + i B on the full length, in the tile: element L - k holds conj(A_k) + i conj(B_k)
    __device__ __forceinline__ void put(cx<T> *tile, int lane) {
        using F = typename X::template F<T>;
#pragma unroll
        for (int it = 0; it < X::NIT; ++it) {
            const int i = lane + it * 64;
            const int p = i / X::KH, k = i - p * X::KH;
            if (p >= X::PW) continue;
            cx<T> a = A[it], b = B[it];
            if (k == 0) a.y = b.y = T(0);
            tile[F::lidx(p, k)] = mk<T>(a.x - b.y, a.y + b.x);
            if (k > 0) tile[F::lidx(p, L - k)] = mk<T>(a.x + b.y, -a.y + b.x);
        }
        if constexpr (X::EVEN) {
            // Nyquist: real parts of the even (real) and odd (imaginary) row
            if (lane < 2 * X::PW) reinterpret_cast<T *>(&tile[F::lidx(lane >> 1, L / 2)])[lane & 1] = Q.x;
        }
    }
};

// Half spectra of the two real rows of every pair from the forward transforms C in the tile; out:
// first row's half spectrum (the same for all lanes).  times_ikx: both multiplied by i k_x
// (k_x = k dkx, rounded once; zero on the Nyquist column).
template <typename T, int L>
__device__ __forceinline__ void store_half_rows(const cx<T> *tile, cx<T> *out, int rows_here, int lane, bool times_ikx,
                                                double dkx) {
    using X = XRow<L>;
    using F = typename X::template F<T>;
    constexpr unsigned CB = sizeof(cx<T>);
#pragma unroll
    for (int it = 0; it < X::NIT; ++it) {
        const int i = lane + it * 64;
        const int p = i / X::KH, k = i - p * X::KH;
        if (2 * p >= rows_here) continue;
        const cx<T> ck = tile[F::lidx(p, k)];
        const cx<T> cm = tile[F::lidx(p, k == 0 ? 0 : L - k)];
        cx<T> a = mk<T>(T(0.5) * (ck.x + cm.x), T(0.5) * (ck.y - cm.y));
        cx<T> b = mk<T>(T(0.5) * (ck.y + cm.y), T(-0.5) * (ck.x - cm.x));
        if (times_ikx) {
            const T kx = T(k * dkx);
            a = mk<T>(-kx * a.y, kx * a.x);
            b = mk<T>(-kx * b.y, kx * b.x);
        }
        const unsigned o = (unsigned)(2 * p * X::KX + k) * CB;
        ct::gst(at(out, o), a);
        if (2 * p + 1 < rows_here) ct::gst(at(out, o + X::KX * CB), b);
    }
    if constexpr (X::EVEN) {
        // an element that is its own mirror image: (C_k + conj C_k) / 2 and (C_k - conj C_k) / (2i)
        if (lane < rows_here) {
            const cx<T> c = tile[F::lidx(lane >> 1, L / 2)];
            const T re = (lane & 1) ? c.y : c.x;
            ct::gst(at(out, (unsigned)(lane * X::KX + L / 2) * CB), mk<T>(times_ikx ? T(0) : T(0.5) * (re + re), T(0)));
        }
    }
}

// X1: real rows of field blockIdx.y (plain, or the line-search trial point
// rho0 + alpha (g0 - rho0), written out; FP32-mixed: minus the reference) -> forward x ->
// half spectra.  Up to four waves a block, each with its own row pairs.
template <typename T, int L>
__global__ __launch_bounds__(256) void k_x1c(Geo g_in, XFwdArgs a) {
    using X = XRow<L>;
    using F = typename X::template F<T>;
    constexpr int PW = X::PW;
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    resolve_roles(a);
    __shared__ cx<T> lds[4 * F::TILE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = (int)threadIdx.x & 63;
    cx<T> *tile = lds + w * F::TILE;
    const int f = blockIdx.y;
    const long long rows = (long long)g.ny * g.nz;
    const long long pair0 = ((long long)blockIdx.x * (blockDim.x / 64) + w) * PW;
    const int rows_here = (int)max(0LL, min((long long)(2 * PW), rows - 2 * pair0));
    const long long first = (long long)f * g.N + 2 * pair0 * L;
    const bool trial = a.mode == XF_TRIAL;
    const double alpha = trial ? *a.alpha : 0.0;
    typename F::template TwReg<-1> tw;
    F::template load_tw<-1>(tw, twp<T>(g, 0), lane);
    cx<T> v[F::V];
#pragma unroll
    for (int i = 0; i < F::template nin<-1>(); ++i) {
        int p, e;
        const bool in = F::template in_pos<-1>(i, p, e, lane);
        double x[2] = {0.0, 0.0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!(in && 2 * p + h < rows_here)) continue;
            const unsigned o = (unsigned)((2 * p + h) * L + e) * 8u;
            double xv = ct::cld(at(a.src + first, o));
            if (trial) {
                xv = fma(alpha, ct::cld(at(a.g0 + first, o)) - xv, xv);
                if (a.rho_t) ct::gst(at(a.rho_t + first, o), xv);
            }
            if (a.ref) xv -= ct::cld(at(a.ref + first, o));
            x[h] = xv;
        }
        v[i] = mk<T>(T(x[0]), T(x[1]));
    }
    int ph = lane;
    F::template run<-1>(v, tile, ph, tw);
    F::sync();
#pragma unroll
    for (int i = 0; i < F::template nout<-1>(); ++i) {
        int p, e;
        if (F::template out_pos<-1>(i, p, e, lane)) tile[F::lidx(p, e)] = v[i];
    }
    F::sync();
    store_half_rows<T, L>(tile, reinterpret_cast<cx<T> *>(a.spec) + (long long)f * g.NC + 2 * pair0 * X::KX, rows_here,
                          lane, false, 0.0);
}

// X3: half spectra of E_k (species blockIdx.y) -> inverse x -> Euler-Lagrange update
// G = rho_b exp(base + E) (eq. rhoEquation) and the weighted residual sums; raw mode
// writes E (+ addend) only.
template <typename T, int L>
__global__ __launch_bounds__(256) void k_x3c(Geo g_in, X3Args a) {
    using X = XRow<L>;
    using F = typename X::template F<T>;
    constexpr int PW = X::PW;
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    resolve_roles(a);
    __shared__ cx<T> lds[4 * F::TILE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = (int)threadIdx.x & 63;
    cx<T> *tile = lds + w * F::TILE;
    const Consts &c = *g.cs;
    const int sp = blockIdx.y;
    const long long N = g.N;
    const long long rows = (long long)g.ny * g.nz;
    const long long pair0 = ((long long)blockIdx.x * (blockDim.x / 64) + w) * PW;
    const int rows_here = (int)max(0LL, min((long long)(2 * PW), rows - 2 * pair0));
    HalfRows<T, L> half;
    half.load(reinterpret_cast<const cx<T> *>(a.specA) + (long long)sp * g.NC + 2 * pair0 * X::KX, rows_here, lane);
    typename F::template TwReg<1> tw;
    F::template load_tw<1>(tw, twp<T>(g, 0), lane);
    half.put(tile, lane);
    F::sync();
    cx<T> v[F::V];
    F::template get<F::template rad<1>(0)>(v, tile, lane);
    int ph = lane;
    F::template run<1>(v, tile, ph, tw);
    double acc = 0.0;
    int flag = 0;
    const double rb = c.rho_b[sp], irb = c.inv_rho_b[sp], zs = c.z[sp];
    const long long node0 = 2 * pair0 * L, first = (long long)sp * N + node0;
#pragma unroll
    for (int i = 0; i < F::template nout<1>(); ++i) {
        int p, e;
        if (!F::template out_pos<1>(i, p, e, lane)) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (2 * p + h >= rows_here) break;
            const double E = h == 0 ? (double)v[i].x : (double)v[i].y;
            const unsigned o = (unsigned)((2 * p + h) * L + e) * 8u;
            if (a.raw) {
                double r = E;
                if (a.addend) r += ct::gld(at(a.addend + node0, o));
                ct::gst(at(a.raw_out + first, o), r);
                continue;
            }
            const double b = ct::cld(at(a.base + first, o));
            const bool fluid = b > -INFINITY;
            const double G = fluid ? rb * exp(b + E) : 0.0;
            if (a.g_out) ct::gst(at(a.g_out + first, o), G);
            if (a.e_out) ct::gst(at(a.e_out + first, o), a.e_phi ? E - zs * ct::gld(at(a.e_phi + node0, o)) : E);
            if (a.lp_out) ct::gst(at(a.lp_out + first, o), fluid ? b + E : -INFINITY);
            if (fluid) {
                const double dlt = (ct::cld(at(a.rho_t + first, o)) - G) * irb;
                acc += dlt * dlt;
                if (!isfinite(G)) flag |= 1;
            }
        }
    }
    if (a.raw) return;
    const long long slot = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    if (blockDim.x == 64) block_reduce_nt<false, 64>(acc, flag, a.red.fpart + slot, a.red.fflag + slot);
    else block_reduce_nt<false, 256>(acc, flag, a.red.fpart + slot, a.red.fflag + slot);
}

}  // namespace dft
