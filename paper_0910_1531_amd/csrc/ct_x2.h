// X2 of the compiled lengths: the ten weighted-density spectra after the y inverse -> inverse x ->
// pointwise dPhi/dn (eq. Phi) -> forward x -> half spectra, in place in specB.
#pragma once

#include "ct_rows.h"

namespace dft {

// Nodewise variants of X2: FP64 eq. (Phi) (with FP32 transforms, the difference of its values at the density
// and at the reference, both in FP64); FP32 differences from the reference (eq. (Phi), x2_node_diff); FP64 with
// an alternative functional chosen by X2Args::hs; the product of the FMT Hessian at nstar (X2_HESS) of eq. (Phi)
// and of an alternative functional.
enum X2Node { X2N_FP64 = 0, X2N_D32 = 1, X2N_ALT = 2, X2N_HESS = 3, X2N_HESS_ALT = 4 };

// Rows whose FP32-mixed evaluations form the differences in FP32: the lengths of the tuned kernels (us, FP32
// differences / FP64: 48^3 13.3 / 14.3, 96^3 39 / 46, 128^3 60 / 86, 256^3 431 / 567).  All other rows take
// dPhi/dn in FP64, the more precise of the two (the cost there: 27^3 none, 81^3 34 / 50, 108^3 51 / 70, 144^3
// 113 / 150, 216 x 108 x 108 108 / 140, 512 x 48 x 48 58 / 61).
constexpr bool x2_fp32_nodes(int L) {
    switch (L) {
#define DFT_CASE(n) case n: return true;
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

// Small grids.  A block holds PW row pairs and ten waves, one per field: wave f transforms field f of
// every pair in LDS that only it touches (wave-level fences, no block barrier), then all threads
// share the nodes of the block, one real node each, and the waves transform their fields back.  Bound
// by the latency of one block's chain, which has two transforms one after the other (a block that
// held all ten fields in registers ran twenty: 24^3 56 us, 48^3 62 us; now 13 and 15).
constexpr int kX2WideThreads = 64 * DFT_NALPHA;

template <typename T, int L, int NODE>
__global__ __launch_bounds__(kX2WideThreads) __attribute__((amdgpu_waves_per_eu(3))) void
k_x2w(Geo g_in, X2Args a) {
    using X = XRow<L>;
    using F = typename X::template F<T>;
    constexpr int PW = X::PW, NTB = kX2WideThreads, KX = X::KX;
    constexpr bool D32 = NODE == X2N_D32, ALT = NODE == X2N_ALT || NODE == X2N_HESS_ALT;
    constexpr bool HESS = NODE == X2N_HESS || NODE == X2N_HESS_ALT;
    static_assert(!D32 || std::is_same<T, float>::value, "FP32 difference path");
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[DFT_NALPHA * F::TILE];
    const int f = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);   // the wave's field
    // the lane, opaque to the compiler: index arithmetic is redone after the nodewise work instead of
    // held in registers through it
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    cx<T> *tile = lds + f * F::TILE;
    const long long N = g.N, NC = g.NC;
    const long long rows = (long long)g.ny * g.nz;
    const long long npairs = (rows + 1) / 2;
    const long long pair0 = (long long)blockIdx.x * PW;
    const int Pact = (int)min((long long)PW, npairs - pair0);
    const cx<T> *tw = twp<T>(g, 0);
    const double dk0 = k_step<T>(g, 0);   // k_x step, read before any store
    // compact layout: n_V2,x = -i k_x n3 is formed here from the n3 spectrum
    const bool from_n3 = g.compact && f == 7;
    // half spectra of the row pairs, every load in flight together
    const cx<T> *in = reinterpret_cast<const cx<T> *>(a.specB) + (long long)(from_n3 ? 3 : f) * NC + 2 * pair0 * KX;
    const int rows_here = (int)min((long long)(2 * PW), rows - 2 * pair0);   // real rows of the block
    HalfRows<T, L> half;
    half.load(in, rows_here, lane);
    typename F::template TwReg<1> tri;
    F::template load_tw<1>(tri, tw, lane);
    // real node of thread m: row h = m % 2 of its pair, element e
    auto node_of = [&](int m, int &p, int &e, int &h) {
        h = m & 1;
        p = (m >> 1) / L;
        e = (m >> 1) - p * L;
    };
    // the reference weighted densities of the thread's first node, fetched ahead of the transforms
    const long long idx0 = 2 * pair0 * L;   // first node of the block
    float nr[DFT_NALPHA];
    auto fetch_nref = [&](int m) {
        int p, e, h;
        node_of(m, p, e, h);
        const unsigned o = (unsigned)((2 * p + h) * L + e) * 4u;
#pragma unroll
        for (int q = 0; q < DFT_NALPHA; ++q)
            nr[q] = 2 * p + h < rows_here ? ct::cld(at(a.nref + q * N + idx0, o)) : 0.0f;
    };
    if constexpr (D32) fetch_nref((int)threadIdx.x);
    half.put(tile, lane);
    F::sync();
    cx<T> v[F::V];
    F::template get<F::template rad<1>(0)>(v, tile, lane);
    if (from_n3) {
#pragma unroll
        for (int i = 0; i < F::template nin<1>(); ++i) {
            int p, e;
            F::template in_pos<1>(i, p, e, lane);
            const T kx = (L % 2 == 0 && 2 * e == L) ? T(0) : T((e <= L / 2 ? e : e - L) * dk0);
            v[i] = mk<T>(kx * v[i].y, -kx * v[i].x);
        }
    }
    F::template run<1>(v, tile, lane, tri);
    F::sync();
#pragma unroll
    for (int i = 0; i < F::template nout<1>(); ++i) {
        int p, e;
        if (F::template out_pos<1>(i, p, e, lane)) tile[F::lidx(p, e)] = v[i];
    }
    __syncthreads();
    // nodewise work: the pair of real rows sits as (real, imaginary), so consecutive threads read
    // consecutive reals
    double mloc = -INFINITY;
    int flag = 0;
    T *real = reinterpret_cast<T *>(lds);
    for (int m = (int)threadIdx.x; m < 2 * Pact * L; m += NTB) {
        int p, e, h;
        node_of(m, p, e, h);
        T *nv = real + 2 * F::lidx(p, e) + h;
        if (2 * p + h >= rows_here) {
            // the missing partner row transforms as zero
#pragma unroll
            for (int q = 0; q < DFT_NALPHA; ++q) nv[2 * q * F::TILE] = T(0);
            continue;
        }
        if constexpr (D32) {
            if (m >= NTB) fetch_nref(m);
            float dn[DFT_NALPHA], dd[DFT_NALPHA];
#pragma unroll
            for (int q = 0; q < DFT_NALPHA; ++q) dn[q] = nv[2 * q * F::TILE];
            x2_node_diff(nr, dn, dd, mloc, flag);
#pragma unroll
            for (int q = 0; q < DFT_NALPHA; ++q) nv[2 * q * F::TILE] = dd[q];
        } else {
            double n[DFT_NALPHA], d[DFT_NALPHA];
#pragma unroll
            for (int q = 0; q < DFT_NALPHA; ++q) n[q] = (double)nv[2 * q * F::TILE];
            x2_node<ALT, HESS, std::is_same<T, float>::value>(a, N, idx0, (unsigned)((2 * p + h) * L + e), n, d, mloc, flag);
#pragma unroll
            for (int q = 0; q < DFT_NALPHA; ++q) nv[2 * q * F::TILE] = T(d[q]);
        }
    }
    asm volatile("" : "+v"(lane));
    typename F::template TwReg<-1> trf;   // after the nodewise work, whose registers they would take
    F::template load_tw<-1>(trf, tw, lane);
    if (flag & 4) mloc = INFINITY;   // the n3 bound needs finite n3 only
    // (its barrier also ends the nodewise work before the transforms below)
    block_reduce_nt<true, NTB>(mloc, flag, a.red.mpart + blockIdx.x, a.red.mflag + blockIdx.x);
    F::template get<F::template rad<-1>(0)>(v, tile, lane);
    F::template run<-1>(v, tile, lane, trf);
    F::sync();
#pragma unroll
    for (int i = 0; i < F::template nout<-1>(); ++i) {
        int p, e;
        if (F::template out_pos<-1>(i, p, e, lane)) tile[F::lidx(p, e)] = v[i];
    }
    F::sync();
    // compact layout: the x components of the vector derivatives leave multiplied by i k_x
    store_half_rows<T, L>(tile, reinterpret_cast<cx<T> *>(a.specB) + (long long)f * NC + 2 * pair0 * KX, rows_here, lane,
                          g.compact && (f == 4 || f == 7), dk0);
}

// Large grids.  The ten fields of a row pair shared by two waves of the block.  Wave h of a pair transforms the
// five fields x2_half_field(h, 0..4) of its PW row pairs one after the other in its own LDS region
// and does the nodewise work at half of the nodes of its registers; the other five values of those
// nodes come from the partner wave through LDS, and their derivatives go back the same way.  The
// half spectra pass through LDS on their way in (C_k and its mirror image C_{L-k} written together),
// so the tile works for every length, each element is loaded once, and a wave needs no block barrier
// except around the swap.  Bound by HBM once enough waves are in flight: FP32 four waves per SIMD
// (126 registers).  Measured at 128^3 FP32 123 us before (two waves per SIMD, ten fields a thread) and
// 62 now; 192^3 578 / 211 us; 256^3 502 / 433 us FP32 (4.5 TB/s of algorithmic traffic) and
// 856 / 699 us FP64.
__host__ __device__ constexpr int x2_half_field(int h, int j) {
    return h == 0 ? (j < 4 ? j : 7) : (j < 3 ? 4 + j : 5 + j);
}

// Nodewise work of one paired wave (H: its half of the registers) with the swap through LDS: the
// own fields at the partner's registers go out to the own region; after a barrier the wave takes
// the partner's fields at its own registers from the partner's region, one register at a time, and
// leaves the partner's derivatives in the same place; after a second barrier it reads its own
// derivatives at the partner's registers back.  Between the barriers only the partner touches a
// wave's region.  Every wave of the block passes both barriers.
template <typename T, int L, class F, int NODE, int H, int NV>
__device__ __forceinline__ void x2h_swap_and_nodes(const X2Args &a, long long N, long long idx0, int rows_here,
                                                   cx<T> *own, cx<T> *other, int lane, cx<T> (&vals)[5][NV],
                                                   double &mloc, int &flag) {
    constexpr int NH = NV / 2, Q0 = NH * H, QP = NH * (1 - H);   // the own and the partner's registers
    constexpr bool D32 = NODE == X2N_D32, ALT = NODE == X2N_ALT || NODE == X2N_HESS_ALT;
    constexpr bool HESS = NODE == X2N_HESS || NODE == X2N_HESS_ALT;
    F::sync();   // the transforms' reads of the region precede the writes below
#pragma unroll
    for (int j = 0; j < 5; ++j)
#pragma unroll
        for (int k = 0; k < NH; ++k) own[(NH * j + k) * 64 + lane] = vals[j][QP + k];
    __syncthreads();
    static_for<NH>([&](auto K) __attribute__((always_inline)) {
        constexpr int k = K, i = Q0 + k;
        int p, e;
        const bool in = F::template out_pos<1>(i, p, e, lane);
        cx<T> oth[5];
#pragma unroll
        for (int j = 0; j < 5; ++j) oth[j] = other[(NH * j + k) * 64 + lane];
#pragma unroll
        for (int hr = 0; hr < 2; ++hr) {
            const bool ok = in && 2 * p + hr < rows_here;
            const unsigned node = (unsigned)((2 * p + hr) * L + e);
            typename std::conditional<D32, float, double>::type dn[DFT_NALPHA], dd[DFT_NALPHA];
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                dn[x2_half_field(H, j)] = hr == 0 ? vals[j][i].x : vals[j][i].y;
                dn[x2_half_field(1 - H, j)] = hr == 0 ? oth[j].x : oth[j].y;
            }
            if (ok) {
                if constexpr (D32) {
                    float nr[DFT_NALPHA];
#pragma unroll
                    for (int f = 0; f < DFT_NALPHA; ++f) nr[f] = ct::cld(at(a.nref + f * N + idx0, node * 4u));
                    x2_node_diff(nr, dn, dd, mloc, flag);
                } else {
                    x2_node<ALT, HESS, std::is_same<T, float>::value>(a, N, idx0, node, dn, dd, mloc, flag);
                }
            } else {
#pragma unroll
                for (int f = 0; f < DFT_NALPHA; ++f) dd[f] = 0;   // the missing partner row transforms as zero
            }
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                if (hr == 0) {
                    vals[j][i].x = T(dd[x2_half_field(H, j)]);
                    oth[j].x = T(dd[x2_half_field(1 - H, j)]);
                } else {
                    vals[j][i].y = T(dd[x2_half_field(H, j)]);
                    oth[j].y = T(dd[x2_half_field(1 - H, j)]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 5; ++j) other[(NH * j + k) * 64 + lane] = oth[j];
    });
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 5; ++j)
#pragma unroll
        for (int k = 0; k < NH; ++k) vals[j][QP + k] = own[(NH * j + k) * 64 + lane];
    F::sync();   // the reads above precede the transforms' writes to the same region
}

// Waves per SIMD that the registers allow without (or with few) spills, by the values a field has per
// lane (four, six or eight) and the nodewise form: FP32 differences 126 registers; FP64 about 200 at two waves.
// In FP64 three waves (168 registers) spill little enough at 96 and 192 only; us, two waves / three: 96^3 63 / 55,
// but 24 x 128 x 128 29.7 / 31.5, 36 x 96 x 96 31.7 / 34.4, 48 x 96 x 96 31.2 / 32.2, 72^3 32 / 44, 108^3 91 / 141,
// 216 x 96 x 96 131 / 288, 256^3 699 / 816; 54 x 81 x 81 35.5 / 34.5 and 144^3 204 / 166 would gain.
template <typename T, int L, int NODE>
struct XHalf {
    static constexpr int NV = XRow<L>::template F<T>::template nout<1>();
    static constexpr int WPE = NODE == X2N_D32 ? (NV <= 4 ? 4 : NV <= 6 ? 3 : 2)
                               : sizeof(T) == 4 ? 2
                                                : (NV > 6 ? 1 : (L == 96 || L == 192) ? 3 : 2);
};

template <typename T, int L, int NODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(XHalf<T, L, NODE>::WPE))) void
k_x2h(Geo g_in, X2Args a) {
    using X = XRow<L>;
    using F = typename X::template F<T>;
    constexpr int PW = X::PW, KX = X::KX;
    constexpr int NV = F::template nout<1>();
    static_assert(NV == F::template nin<-1>() && NV % 2 == 0, "registers of a node are the same in both directions");
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    constexpr int REGION = F::TILE > 5 * (NV / 2) * 64 ? F::TILE : 5 * (NV / 2) * 64;
    __shared__ cx<T> lds[4 * REGION];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), h = wave & 1;
    // the lane, opaque to the compiler: index arithmetic is redone after the nodewise work instead of
    // held in registers through it
    int lane = (int)threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    cx<T> *tile = lds + wave * REGION, *other = lds + (wave ^ 1) * REGION;
    const long long N = g.N, NC = g.NC;
    const long long rows = (long long)g.ny * g.nz;
    const long long pair0 = ((long long)blockIdx.x * 2 + (wave >> 1)) * PW;
    const int rows_here = (int)max(0LL, min((long long)(2 * PW), rows - 2 * pair0));   // real rows of the wave
    const cx<T> *tw = twp<T>(g, 0);
    const double dk0 = k_step<T>(g, 0);   // k_x step, read before any store
    HalfRows<T, L> half[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        const int f = h == 0 ? x2_half_field(0, j) : x2_half_field(1, j);
        // compact layout: n_V2,x = -i k_x n3 is formed below from field 3
        const bool skip = f == 7 && g.compact;
        half[j].load(reinterpret_cast<const cx<T> *>(a.specB) + (long long)f * NC + 2 * pair0 * KX, skip ? 0 : rows_here,
                     lane);
    }
    typename F::template TwReg<1> tri;
    F::template load_tw<1>(tri, tw, lane);
    cx<T> vals[5][NV];
    cx<T> v[F::V];
    cx<T> v3[F::template nin<1>()];   // inputs of field 3 (n3), the source of n_V2,x in the compact layout
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        if (h == 0 && j == 4 && g.compact) {
#pragma unroll
            for (int i = 0; i < F::template nin<1>(); ++i) {
                int p, e;
                F::template in_pos<1>(i, p, e, lane);
                const T kx = (X::EVEN && 2 * e == L) ? T(0) : T((e <= L / 2 ? e : e - L) * dk0);
                v[i] = mk<T>(kx * v3[i].y, -kx * v3[i].x);
            }
        } else {
            F::sync();
            half[j].put(tile, lane);
            F::sync();
            F::template get<F::template rad<1>(0)>(v, tile, lane);
            if (h == 0 && j == 3) {
#pragma unroll
                for (int i = 0; i < F::template nin<1>(); ++i) v3[i] = v[i];
            }
        }
        F::template run<1>(v, tile, lane, tri);
#pragma unroll
        for (int i = 0; i < NV; ++i) vals[j][i] = v[i];
    }
    double mloc = -INFINITY;
    int flag = 0;
    asm volatile("" : "+v"(lane));
    // the halves take constant register indices (a run-time choice would put vals in scratch)
    if (h == 0) x2h_swap_and_nodes<T, L, F, NODE, 0, NV>(a, N, 2 * pair0 * L, rows_here, tile, other, lane, vals, mloc, flag);
    else x2h_swap_and_nodes<T, L, F, NODE, 1, NV>(a, N, 2 * pair0 * L, rows_here, tile, other, lane, vals, mloc, flag);
    if (flag & 4) mloc = INFINITY;   // the n3 bound needs finite n3 only
    block_reduce_nt<true, 256>(mloc, flag, a.red.mpart + blockIdx.x, a.red.mflag + blockIdx.x);
    asm volatile("" : "+v"(lane));
    typename F::template TwReg<-1> trf;
    F::template load_tw<-1>(trf, tw, lane);
#pragma unroll
    for (int j = 0; j < 5; ++j) {
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = vals[j][i];
        F::template run<-1>(v, tile, lane, trf);
        F::sync();
#pragma unroll
        for (int i = 0; i < F::template nout<-1>(); ++i) {
            int p, e;
            if (F::template out_pos<-1>(i, p, e, lane)) tile[F::lidx(p, e)] = v[i];
        }
        F::sync();
        // compact layout: the x components of the vector derivatives leave multiplied by i k_x
        const int f = h == 0 ? x2_half_field(0, j) : x2_half_field(1, j);
        store_half_rows<T, L>(tile, reinterpret_cast<cx<T> *>(a.specB) + (long long)f * NC + 2 * pair0 * KX, rows_here,
                              lane, g.compact && (f == 4 || f == 7), dk0);
    }
}

// n3 only (the bound of the line search): inverse x of the one field in specB and its maximum.
// Four waves, each with its own pencils.
template <typename T, int L>
__global__ __launch_bounds__(256) void k_x2n(Geo g_in, X2Args a) {
    using X = XRow<L>;
    using F = typename X::template F<T>;
    constexpr int PW = X::PW, KX = X::KX;
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[4 * F::TILE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = (int)threadIdx.x & 63;
    cx<T> *tile = lds + w * F::TILE;
    const long long N = g.N;
    const long long rows = (long long)g.ny * g.nz;
    const long long pair0 = ((long long)blockIdx.x * 4 + w) * PW;
    const int rows_here = (int)max(0LL, min((long long)(2 * PW), rows - 2 * pair0));
    HalfRows<T, L> half;
    half.load(reinterpret_cast<const cx<T> *>(a.specB) + 2 * pair0 * KX, rows_here, lane);
    half.put(tile, lane);
    F::sync();
    cx<T> v[F::V];
    typename F::template TwReg<1> tri;
    F::template load_tw<1>(tri, twp<T>(g, 0));
    F::template get<F::template rad<1>(0)>(v, tile);
    int ph = lane;
    F::template run<1>(v, tile, ph, tri);
    double mloc = -INFINITY;
    int flag = 0;
#pragma unroll
    for (int i = 0; i < F::template nout<1>(); ++i) {
        int p, e;
        if (!F::template out_pos<1>(i, p, e, lane)) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const long long r = 2 * (pair0 + p) + h;
            if (2 * p + h >= rows_here) break;
            double n3 = h == 0 ? (double)v[i].x : (double)v[i].y;
            if (a.nref) n3 += (double)ct::cld(a.nref + 3 * N + r * L + e);
            if (!isfinite(n3)) flag |= 5;   // 1: evaluation non-finite, 4: n3 non-finite
            mloc = fmax(mloc, n3);
        }
    }
    if (flag & 4) mloc = INFINITY;   // the n3 bound needs finite n3 only
    block_reduce_nt<true, 256>(mloc, flag, a.red.mpart + blockIdx.x, a.red.mflag + blockIdx.x);
}

// Rule between the two kernels: one wave per field (k_x2w) while its blocks fit about once on the
// 256 CUs, where the pass lasts as long as one block does and short chains count; above, two waves
// per row pair (k_x2h), whose waves keep five fields of loads in flight and share the fixed work of a
// block among more of them.  Measured FP64, k_x2w against k_x2h: 24^3 (29 blocks) 13.6 / 19.1 us,
// 48^3 (231) 16.9 / 22.5, 384 x 16 x 16 (128) 26 / 37, 64^3 (512) 25.7 / 24.1, 96^3 (2304) 87 / 55,
// 256^3 1192 / 699; FP32 96^3 75 / 40, 128^3 135 / 62, 256^3 1077 / 433.
constexpr long long kX2WideBlocks = 384;

// Launches the full pass in nodewise form NODE; returns the number of blocks (each writes one
// n3-maximum partial).
template <typename T, int L, int NODE>
int launch_x2_form(const Geo &g, const X2Args &a, hipStream_t s) {
    constexpr int PW = XRow<L>::PW;
    const long long npairs = ((long long)g.ny * g.nz + 1) / 2;
    const long long nw = ct_cdiv(npairs, PW);
    // (eight FP64 values a field leave k_x2h one wave per SIMD with 372 registers: 384 x 96 x 96 345 us
    // with k_x2w, 319 with k_x2h; the longer rows, with as many, take k_x2w only)
    constexpr bool only_wide = sizeof(T) == 8 && L > 384;
    const bool wide = only_wide || nw * g.nprob <= kX2WideBlocks;
    const long long nb = wide ? nw : ct_cdiv(npairs, 2 * PW);
    if (nb > a.red.cap) throw std::runtime_error("x2: reduction buffer too small");
    const dim3 grid((unsigned)nb, 1, (unsigned)g.nprob);
    if (wide) hipLaunchKernelGGL((k_x2w<T, L, NODE>), grid, dim3(kX2WideThreads), 0, s, g, a);
    else if constexpr (!only_wide) hipLaunchKernelGGL((k_x2h<T, L, NODE>), grid, dim3(256), 0, s, g, a);
    ct_check("x2 (compiled length)");
    return (int)nb;
}

// Longest rows of the Hessian product: dft_adjoint and dft_newton refuse longer ones before any launch.
constexpr int kX2HessMax = 384;

// n3 only; returns the number of blocks (each writes one n3-maximum partial).
template <typename T, int L>
int launch_x2n_len(const Geo &g, const X2Args &a, hipStream_t s) {
    const long long nb = ct_cdiv(((long long)g.ny * g.nz + 1) / 2, 4 * XRow<L>::PW);
    if (nb > a.red.cap) throw std::runtime_error("x2: reduction buffer too small");
    hipLaunchKernelGGL((k_x2n<T, L>), dim3((unsigned)nb, 1, (unsigned)g.nprob), dim3(256), 0, s, g, a);
    ct_check("x2 (n3 only)");
    return (int)nb;
}

// The pass of one class and row length.  The classes but the first are kernels of their own, so the kernels of
// eq. (Phi) keep their register budget: the Hessian product (FP64 transforms) and the alternative hard-sphere
// functionals (Rosenfeld's original vector form, White Bear; FP64 nodewise work).
template <typename T, int CLASS, int L>
int launch_x2_len(const Geo &g, const X2Args &a, hipStream_t s) {
    if constexpr ((CLASS == X2C_HESS || CLASS == X2C_HESS_ALT) && L > kX2HessMax) {
        throw std::runtime_error("x2: the Hessian mode needs n_x <= 384");
    } else if constexpr (CLASS == X2C_HESS) return launch_x2_form<T, L, X2N_HESS>(g, a, s);
    else if constexpr (CLASS == X2C_ALT) return launch_x2_form<T, L, X2N_ALT>(g, a, s);
    else if constexpr (CLASS == X2C_HESS_ALT) return launch_x2_form<T, L, X2N_HESS_ALT>(g, a, s);
    else if (a.mode == X2_N3_ONLY) return launch_x2n_len<T, L>(g, a, s);
    // FP32 transforms act on differences from the reference
    else return launch_x2_form<T, L, std::is_same<T, float>::value && x2_fp32_nodes(L) ? X2N_D32 : X2N_FP64>(g, a, s);
}

}  // namespace dft
