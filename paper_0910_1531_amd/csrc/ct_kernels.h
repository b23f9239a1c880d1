// Pass kernels with the transform length fixed at compile time (fft_ct.h).  They compute
// the same transforms as the run-time-length kernels, and every launch shape of one length
// (tile width, threads, LDS buffering) performs the same arithmetic in the same order, so
// the choice among shapes never changes a result.
#pragma once

#include <stdexcept>
#include <string>
#include <type_traits>
#include <utility>

#include "dft_kernels.h"
#include "fft_ct.h"
#include "pass_util.h"

namespace dft {

// Threads per block: a power of two in [64, cap] near L P / per (per = values per thread).
constexpr int fit_threads(int L, int P, int per, int cap) {
    int t = 64;
    while (2 * t <= cap && 2 * t * per <= L * P) t *= 2;
    return t;
}

inline void ct_check(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw std::runtime_error(std::string(what) + ": " + hipGetErrorString(e));
}

inline long long ct_cdiv(long long a, long long b) { return (a + b - 1) / b; }

// f(integral_constant<int, i>) for i = 0..N-1: a loop whose index is a constant in every body,
// whatever the body's size (register arrays indexed by it stay in registers).
template <class Fn, int... I>
__device__ __forceinline__ void static_for_impl(Fn &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class Fn>
__device__ __forceinline__ void static_for(Fn &&f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Lengths whose y and z kernels come in the launch shapes the autotuner chooses among, and those
// compiled in one shape.
#define DFT_CT_LENGTHS(X) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(384)
#define DFT_CT_MORE_LENGTHS(X) \
    X(8) X(9) X(12) X(18) X(27) X(36) X(54) X(72) X(81) X(108) X(144) X(162) X(216) X(243) X(288) X(324) X(432) X(486) \
    X(512)

constexpr bool tuned_length(int L) {
    switch (L) {
#define DFT_CASE(n) case n: return true;
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

// Whether the z passes of length L in precision T form wavenumbers in FP64 and round them once, and take the
// pair factors from the FP64 tables: FP64 at every length, FP32 at the lengths compiled in one shape.  There the
// FP32 factors formed on the fly were up to three times further from 64 bits than those of the run-time-length
// kernels before them (pair factors at k R up to 100: 2.0e-7 to 3.4e-7 of their parts, from the tables at most
// 7.4e-8); the tables cost Z1 time on large grids (three species, us on the fly / tables: 24 x 24 x 162 24.9 / 23.9,
// 81^3 24.6 / 25.8, 108^3 52 / 61, 144^3 83 / 113, 96 x 96 x 288 90 / 104).  The tuned lengths form theirs on the fly.
template <typename T, int L>
constexpr bool z_fp64_factors() {
    return sizeof(T) == 8 || !tuned_length(L);
}

// Threads of a tile in the lengths compiled in one shape: of the multiples of 64 up to cap (and of P)
// that keep at most vcap values per thread in any stage and ocap after the last forward stage, the
// one that leaves the fewest threads idle over the stages, the larger of equals.
template <class SC>
constexpr int one_shape_threads(int P, int cap, int vcap, int ocap) {
    int best = 0;
    double least = 1e30;
    for (int t = 64; t <= cap; t += 64) {
        if (t % P) continue;
        bool ok = true;
        double spent = 0.0;
        for (int s = 0; s < SC::n; ++s) {
            const int R = SC::r(s), it = (SC::L * P / R + t - 1) / t;
            if (it * R > vcap || (s == SC::n - 1 && it * R > ocap)) ok = false;
            spent += (double)t * it * R;
        }
        if (ok && spent <= least) {
            least = spent;
            best = t;
        }
    }
    return best;
}

// ... of a z tile, whose products hold five or six sums of every value after the last forward stage:
// at most four values where 768 threads allow it, else eight; FP32 up to 162 six values and 512
// threads (144^3: 64 us either z pass with 192 threads of six values, 90 with 384 of three).
template <typename T, int L>
constexpr int z_one_threads(int P) {
    using SC = typename ct::PlanT<T, L>::type;
    constexpr int vcap = sizeof(T) == 4 ? 16 : 9;
    if (sizeof(T) == 4 && L <= 162) return one_shape_threads<SC>(P, 512, vcap, 6);
    const int few = one_shape_threads<SC>(P, 768, vcap, 4);
    return few ? few : one_shape_threads<SC>(P, 768, vcap, 8);
}

// z passes whose index arithmetic is redone at every exchange (Fft's OPQ) instead of held in registers
// through their seven to ten transforms: the lengths that otherwise spill or leave one wave per SIMD.
// Measured on 64 x 64 x n_z, three species, us held / redone: FP64 Z1 192 56 / 43, 384 109 / 96,
// 432 253 / 113, 144 55 / 50, 256 50 / 47 (256^3 788 / 773); Z2 192 71 / 51, 432 209 / 116,
// 96 28 / 46, 256^3 790 / 823; FP32 Z1 432 107 / 48, 324 67 / 58, 256 38 / 41; Z2 432 133 / 53,
// 512 69 / 54, 324 58 / 80.  On cubes, two and three species: FP64 Z1 96^3 45 / 37.5, 52 / 43.7, 128^3
// 65 / 59, 88 / 74; FP32 Z1 (with the waves of z1_waves) 128^3 47 / 41.7, 59 / 47.4, 192^3 108 / 100.6,
// 143 / 114.5, but 96^3 31.7 / 35.3 and 256^3 338 / 352.  Held is the better at the other lengths of one shape: FP64 72^3
// 29 / 33, 81^3 38 / 41, 108^3 77 / 78, 96 x 96 x 216 119 / 140, 72 x 72 x 243 93 / 107; FP32 (pair factors from the
// tables) 72^3 23.6 / 27.6, 96 x 96 x 216 85 / 98, 64 x 64 x 162 38 / 46, and at 108 and 144 by the size of the grid:
// 64 x 64 x 144 35 / 41 but 144^3 113 / 100.
template <typename T, int L>
constexpr bool z1_redo() {
    if (sizeof(T) == 8) return L == 96 || L == 128 || L == 144 || L == 162 || L == 192 || L == 256 || L == 384 || L == 432 || L == 486;
    return L == 128 || L == 192 || L == 324 || L == 432 || L == 486;
}
// Waves per SIMD Z1's registers are cut to (a few spills against more tiles in flight), by threads per
// block: the fewest the block needs, but FP32 128 five (96 VGPRs for 102; with four, 128^3 46.7 and 54.5 us
// where five take 41.7 and 47.4) and 192 four (121 and 138 us left alone, 100.6 and 114.5 with four).
template <typename T, int L, int NTB>
constexpr int z1_waves() {
    if (sizeof(T) == 4 && L == 128) return 5;
    if (sizeof(T) == 4 && L == 192) return 4;
    return (NTB + 255) / 256;
}
template <typename T, int L>
constexpr bool z2_redo() {
    if (sizeof(T) == 8) return L == 192 || L == 432 || L == 486;
    return L == 432 || L == 486 || L == 512;
}

// Grid step of k_x or k_y in the compact layout's x and y passes.  T(mode * step) is the FP64 wavenumber
// rounded once, or with Geo::fp64_k off the FP32 product of the mode and the rounded step (that product is
// exact in FP64).
template <typename T>
__device__ __forceinline__ double k_step(const Geo &g, int axis) {
    const double dk = axis == 0 ? g.cs->dk[0] : g.cs->dk[1];
    return std::is_same<T, double>::value || g.fp64_k ? dk : (double)(T)dk;
}

// ------------------------------------------------------------------ y / z plain transforms
// One block transforms P adjacent pencils of one field along y or z; the pencils' elements sit
// rs apart in HBM, and adjacent pencils of one row are adjacent in HBM.
// VEC = 1, 2: the y passes of the compact vector layout (Geo::compact), where a block of the
// n3 or nV1-sum slot makes two transforms (inverse: the field and -i k_y times it) and a block
// of a vector-derivative slot adds i k_y times the transform of the y component (forward).
template <typename T, int L, int P, int NTB, int NB, int VEC>
__global__ __launch_bounds__(NTB) void k_yc(Geo g_in, YArgs a) {
    using F = ct::Fft<T, typename ct::PlanT<T, L>::type, P, NTB, false, NB>;
    // blocks per problem: one per field, or per block type of the compact vector layout
    // (VEC = YArgs::vec, a template parameter so that the plain transforms keep their registers)
    const int ntypes = VEC == 1 ? 7 : (VEC == 2 ? 8 : a.nfield);
    const int prob = (int)blockIdx.z / ntypes;
    if (prob > 0) {
        const long long off = (long long)prob * g_in.pstride;
        g_in = shift(g_in, off);
        a = shift(a, off);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[F::LDS_ELEMS];
    const bool zax = a.axis == 2;
    const int Kx = g.Kx;
    // A tile is P consecutive pencils of the flattened plane of pencils, (y, kx) as y Kx + kx for
    // the z axis (as in the other z tiles), (z, kx) as z Kx + kx for the y axis, so no tile holds
    // a lone Nyquist column.  A thread keeps one pencil (p = threadIdx.x mod P) and its offset.
    static_assert(NTB % P == 0, "a thread keeps one pencil");
    int bx, unused;
    xcd_block(bx, unused);
    const int ncol = (zax ? g.ny : g.nz) * Kx;
    const int c0 = bx * P;
    const int Pact = min(P, ncol - c0);
    const int col = min(c0 + (int)threadIdx.x % P, ncol - 1);
    const int zc = zax ? 0 : col / Kx;
    const int jx = col - zc * Kx;   // k_x index of the pencil (y axis)
    const int f = (int)blockIdx.z % ntypes;
    if (f > 0 && n3_wanted(a.n3_only)) return;
    const long long rs = zax ? (long long)g.ny * Kx : (long long)Kx;
    cx<T> *spec = reinterpret_cast<cx<T> *>(a.spec) + (zax ? (long long)col : (long long)zc * g.ny * Kx + jx);
    const cx<T> *tw = twp<T>(g, zax ? 2 : 1);
    // grid steps of k_x, k_y read before any store (read later they would be reloaded after each)
    [[maybe_unused]] const double dkx = k_step<T>(g, 0), dky = k_step<T>(g, 1);
    cx<T> v[F::V];
    int ph = 0;
    auto body = [&](auto dirc) {
        constexpr int DIR = decltype(dirc)::value;
        auto load = [&](int slot, cx<T> *w) {
            const cx<T> *base = spec + (long long)slot * g.NC;
#pragma unroll
            for (int i = 0; i < F::template nin<DIR>(); ++i) {
                int p, e;
                const bool ok = F::template in_pos<DIR>(i, p, e);
                w[i] = (ok && p < Pact) ? ct::gld(base + e * rs) : mk<T>(T(0), T(0));
            }
        };
        // store slot, times -i k_x when mx (k_x of the column, zero on the Nyquist column)
        auto store = [&](int slot, const cx<T> *w, bool mx) {
            cx<T> *base = spec + (long long)slot * g.NC;
#pragma unroll
            for (int i = 0; i < F::template nout<DIR>(); ++i) {
                int p, e;
                const bool ok = F::template out_pos<DIR>(i, p, e);
                if (!(ok && p < Pact)) continue;
                cx<T> u = w[i];
                if (mx) {
                    const T kx = (g.nx % 2 == 0 && 2 * jx == g.nx) ? T(0) : T(jx * dkx);
                    u = mk<T>(kx * u.y, -kx * u.x);
                }
                ct::gst(base + e * rs, u);
            }
        };
        // k_y of element e of the pencil (zero on the Nyquist row)
        auto ky = [&](int e) {
            return (g.ny % 2 == 0 && 2 * e == g.ny) ? T(0) : T(signed_mode(e, g.ny) * dky);
        };
        if constexpr (VEC == 0) {
            load(f, v);
            F::template run<DIR>(v, lds, ph, tw);
            store(f, v, false);
        } else if constexpr (VEC == 1) {
            // inverse: slots 0-3 (n0..n3), 4 (nV1 sum), 6, 9 (z components) -> nine fields:
            // n3 also gives nV2_y = -i k_y n3, the nV1 sum gives nV1_x and nV1_y (slot 7,
            // nV2_x, is left to the x pass)
            const int slot = f < 5 ? f : (f == 5 ? 6 : 9);
            load(slot, v);
            if (slot == 3 || slot == 4) {
                cx<T> w[F::V];
#pragma unroll
                for (int i = 0; i < F::template nin<DIR>(); ++i) {
                    int p, e;
                    F::template in_pos<DIR>(i, p, e);
                    const T k = ky(e);
                    w[i] = mk<T>(k * v[i].y, -k * v[i].x);   // -i k_y
                }
                F::template run<DIR>(v, lds, ph, tw);
                store(slot, v, slot == 4);   // (n_V2,x = -i k_x n3 is formed by the x pass)
                F::template run<DIR>(w, lds, ph, tw);
                store(slot == 3 ? 8 : 5, w, false);
            } else {
                F::template run<DIR>(v, lds, ph, tw);
                store(slot, v, false);
            }
        } else {
            // forward: ten fields -> slots 0-3, 4 (i k_x dPhi_V1x + i k_y dPhi_V1y), 6, 7 (the same
            // for V2), 9; the x parts arrive multiplied by i k_x
            const int slot = f < 5 ? f : (f == 5 ? 6 : (f == 6 ? 7 : 9));
            load(slot, v);
            F::template run<DIR>(v, lds, ph, tw);
            if (slot == 4 || slot == 7) {
                cx<T> w[F::V];
                load(slot + 1, w);
                F::template run<DIR>(w, lds, ph, tw);
#pragma unroll
                for (int i = 0; i < F::template nout<DIR>(); ++i) {
                    int p, e;
                    F::template out_pos<DIR>(i, p, e);
                    const T k = ky(e);
                    v[i] = mk<T>(v[i].x - k * w[i].y, v[i].y + k * w[i].x);   // + i k_y w
                }
            }
            store(slot, v, false);
        }
    };
    if (a.dir < 0) body(std::integral_constant<int, -1>());
    else body(std::integral_constant<int, 1>());
}

// ------------------------------------------------------------------ z passes
// z tiles run over the plane of columns (y, kx) flattened as y Kx + kx: a tile is P consecutive
// columns, whatever row they fall in, so a plane of n_y Kx columns needs ceil(n_y Kx / P) tiles
// (none holding a lone Nyquist column) and, with n_y Kx a multiple of P, every tile's segment of
// a z plane starts on a P-element boundary.  In these tiles (pencil index fastest over threads,
// NTB a multiple of P) a thread keeps one column, p = threadIdx.x mod P.
struct ZTile {
    long long off;   // first column of the tile (offset of its segment in a z plane)
    int Pact;        // columns of the tile inside the plane
    int x, y;        // the thread's column (a valid column also for idle lanes of a ragged tile)
};
template <int P>
__device__ __forceinline__ ZTile z_tile(const Geo &g) {
    int t, unused;
    xcd_block(t, unused);
    const int ncol = g.ny * g.Kx;
    const int c0 = t * P;
    ZTile z;
    z.off = c0;
    z.Pact = min(P, ncol - c0);
    const int col = min(c0 + (int)threadIdx.x % P, ncol - 1);
    z.y = col / g.Kx;
    z.x = col - z.y * g.Kx;
    return z;
}

// Plane of the spectral tables for z element e: the tables are even in k_z and hold z <= L / 2 only, so
// a tile reads each value twice at close times, the second time from L2.  The z passes are bound by
// latency and bytes together, and these are 12 rows with three charged species (0.79 of the 2.55 GB of
// Z1 at 256^3, 0.40 of the 2.3 GB of Z2 when read in full).  Measured us, read in full and halved: 256^3
// Z1 758 / 709, Z2 791 / 760; 128^3 (two species) 74 / 65, 74 / 68; 108 x 72 x 81 39.5 / 37.3, 39.8 / 38.2.
// (Pairing the rows y and -y of a plane, to halve them again, breaks lines at the ends of the rows and
// costs more than it saves: Z1 955, and 30 in the y pass after it.)
template <int L>
__device__ __forceinline__ int z_tab(int e) {
    return e <= L / 2 ? e : L - e;
}

// Elements of a row of the tables (rs = n_y Kx, a z plane).
template <int L>
__device__ __forceinline__ long long z_tab_row(long long rs) {
    return spec_table_row(L / 2 + 1, rs);
}

// Wavenumbers of the elements of one z pencil: column (x, y), z index e.  Only the indices are
// kept per thread (the grid steps are uniform): the components are formed at each use, which
// costs a few instructions and no registers across the transforms.  U: the type they are formed in.
template <typename T, typename U = T>
struct ZWave {
    U dkx, dky, dkz;
    int x, y, nx, ny, nz;
    __device__ __forceinline__ ZWave(const Consts &c, int x_, int y_) : x(x_), y(y_) {
        dkx = U(c.dk[0]);
        dky = U(c.dk[1]);
        dkz = U(c.dk[2]);
        nx = c.nx;
        ny = c.ny;
        nz = c.nz;
    }
    __device__ __forceinline__ U kx() const { return U(x) * dkx; }
    __device__ __forceinline__ U ky() const { return U(signed_mode(y, ny)) * dky; }
    __device__ __forceinline__ U kz(int e) const { return U(signed_mode(e, nz)) * dkz; }
    __device__ __forceinline__ T kmag(int e) const {
        const U a = kx(), b = ky(), d = kz(e);
        return T(sqrt_r(a * a + b * b + d * d));
    }
    __device__ __forceinline__ bool zero(int e) const { return x == 0 && y == 0 && e == 0; }
    // component d of k, zero on the Nyquist plane of axis d
    __device__ __forceinline__ T comp(int e, int d) const {
        if (d == 0) return ((nx % 2 == 0) && 2 * x == nx) ? T(0) : T(kx());
        if (d == 1) return ((ny % 2 == 0) && 2 * y == ny) ? T(0) : T(ky());
        return ((nz % 2 == 0) && 2 * e == nz) ? T(0) : T(kz(e));
    }
};
template <typename T, int L>
using ZWaveOf = ZWave<T, typename std::conditional<z_fp64_factors<T, L>(), double, T>::type>;

// Eigenvalue of minus the 7-point Laplacian, sum_d 4 sin^2(k_d h_d / 2) / h_d^2, from the
// twiddle tables: k_d h_d = 2 pi j_d / n_d, and tw_d[j] = exp(-2 pi i j / n_d).  The x and y
// terms are those of one column (x, y).
template <typename T>
struct Poisson {
    const cx<T> *tz;
    T ih2z, dxy;
    __device__ __forceinline__ Poisson() : tz(nullptr), ih2z(0), dxy(0) {}
    __device__ __forceinline__ Poisson(const Geo &g, const Consts &c, int x, int y) {
        tz = twp<T>(g, 2);
        ih2z = T(1.0 / (c.h[2] * c.h[2]));
        const cx<T> wx = ct::cld(twp<T>(g, 0) + x), wy = ct::cld(twp<T>(g, 1) + y);
        dxy = two_omc<T>(wx.x, wx.y) * T(1.0 / (c.h[0] * c.h[0])) + two_omc<T>(wy.x, wy.y) * T(1.0 / (c.h[1] * c.h[1]));
    }
    __device__ __forceinline__ T denom(int e) const {
        const cx<T> wz = ct::cld(tz + e);
        return dxy + two_omc<T>(wz.x, wz.y) * ih2z;
    }
};

// Pair row of the spectral tables (Geo::tab64): K_ij, i <= j.
__device__ __forceinline__ int pair_row(int S, int i, int j) {
    const int a = min(i, j), b = max(i, j);
    return 2 * S + a * S - (a * (a - 1)) / 2 + (b - a);
}

// Z1: forward z transform of every species, then per element
//   (a) the five weighted sums of Appendix B spectra giving the ten n_alpha spectra (the
//       vector spectra are -i k times a w3 sum), each inverse z transformed into specB;
//   (b) with electrostatics (MS > 0 bounds S), per species i the linear electrostatic part
//       of the exponent sum_j K_ij(k) (rho_hat_j - N rho_b_j delta_k0), K_ij = C_ij(k) -
//       z_i z_j 4 pi l_B / D(k) (eqs. muESexpansion, potentialSolution), written
//       unnormalized over rho_hat in specA (z spectral order).
// FP64 takes the spectral factors from the setup-time tables.  FP32 (differences from the
// reference) evaluates them on the fly: sin and cos of k R once per species and, at the tuned
// lengths, the pair terms by the addition theorem and the Poisson denominator from the twiddle
// tables, which is cheaper than moving the tables; the other lengths read the pair terms from
// the tables (z_fp64_factors).  The products act on registers between
// the forward and inverse transforms.  Every Z1 kernel (fused or split, any tile width) does
// the same arithmetic in the same order, so the autotuner's choice does not change a result.

// Slot of the unordered species pair a <= b < MS.
template <int MS>
__device__ __forceinline__ constexpr int pair_slot(int a, int b) {
    return a * MS - (a * (a - 1)) / 2 + (b - a);
}

// The species and pair constants of the products in the arithmetic type, read once per block
// before any store (read at their uses they would be reloaded and converted after every store,
// which may alias them).  Pair p = pair_slot(a, b), a <= b.
template <typename T, int MS>
struct Z1Const {
    static constexpr int NPR = MS * (MS + 1) / 2;
    T R[MS], a0[MS], a1[MS], bath[MS];   // R_j, 1 / (4 pi R_j^2), 1 / (4 pi R_j), N rho_b,j
    T zz[NPR], scR[NPR], p1[NPR], p2[NPR], p3[NPR], p4[NPR];   // pair constants (FP32 only)
    T four_pi_lB;
    __device__ __forceinline__ explicit Z1Const(const Consts &c) {
        constexpr bool F32 = std::is_same<T, float>::value;
        static_for<MS>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = J;
            if constexpr (F32) {
                R[j] = c.f_R[j];
                a0[j] = c.f_i4piR2[j];
                a1[j] = c.f_i4piR[j];
                bath[j] = c.f_bath_N[j];
            } else {
                R[j] = c.R[j];
                a0[j] = c.i4piR2[j];
                a1[j] = c.i4piR[j];
                bath[j] = c.bath_N[j];
            }
        });
        static_for<MS>([&](auto IA) __attribute__((always_inline)) {
            static_for<MS>([&](auto IB) __attribute__((always_inline)) {
                constexpr int ia = IA, ib = IB;
                if constexpr (ib >= ia) {
                    constexpr int q = pair_slot<MS>(ia, ib), ij = ia * DFT_MAX_SPECIES + ib;
                    if constexpr (F32) {
                        zz[q] = c.f_zz[ij];
                        scR[q] = c.f_sc_R[ij];
                        p1[q] = c.f_sc_p1[ij];
                        p2[q] = c.f_sc_p2[ij];
                        p3[q] = c.f_sc_p3[ij];
                        p4[q] = c.f_sc_p4[ij];
                    } else {
                        // FP64 reads the pair factors from the spectral tables
                        zz[q] = c.z[ia] * c.z[ib];
                        scR[q] = p1[q] = p2[q] = p3[q] = p4[q] = T(0);
                    }
                }
            });
        });
        four_pi_lB = F32 ? c.f_four_pi_lB : c.four_pi_lB;
    }
};

// Products of one node with electrostatics (S <= MS): the species values u at the node (k_x
// column p of the tile, z element e; ti its offset in a row of TS elements of the spectral tables, ok whether it is a real
// column), the five weighted sums out in acc, and the node's sums over j of K_ij times the
// species spectra stored at dst + i NC.  Each unordered pair factor is formed once (K_ij = K_ji).
template <bool TAB, typename T, int MS, class ZW>
__device__ __forceinline__ void z1_node(const Z1Const<T, MS> &k, bool diff, const ZW &kw, const Poisson<T> &pd,
                                        const double *tab, long long TS, long long NC, int S, bool es, int e, bool ok,
                                        long long ti, const cx<T> (&u)[MS], cx<T> (&acc)[5], cx<T> *dst) {
    constexpr int NPR = MS * (MS + 1) / 2;
    T w2[MS], w3[MS], K[NPR];
    // every loop over species or pairs has constant indices (static_for), whatever its size
    if constexpr (TAB) {
        static_for<MS>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = J;
            w2[j] = w3[j] = T(0);
            if constexpr (std::is_same<T, double>::value) {
                if (ok && j < S) {
                    w2[j] = ct::cld(tab + (long long)j * TS + ti);
                    w3[j] = ct::cld(tab + (long long)(S + j) * TS + ti);
                }
            } else if (j < S) {
                weight_w2_w3<T>(kw.kmag(e), k.R[j], w2[j], w3[j]);
            }
        });
        static_for<MS>([&](auto IA) __attribute__((always_inline)) {
            static_for<MS>([&](auto IB) __attribute__((always_inline)) {
                constexpr int ia = IA, ib = IB;
                if constexpr (ib >= ia)
                    K[pair_slot<MS>(ia, ib)] =
                        (ok && es && ib < S) ? T(ct::cld(tab + (long long)pair_row(S, ia, ib) * TS + ti)) : T(0);
            });
        });
    } else {
        const T km = kw.kmag(e);
        T sn[MS], cs[MS];
        static_for<MS>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = J;
            sn[j] = T(0);
            cs[j] = T(1);
            w2[j] = w3[j] = T(0);
            if (j < S) {
                sincos_w(km * k.R[j], &sn[j], &cs[j]);
                weight_w2_w3_sc<T>(km, k.R[j], sn[j], cs[j], w2[j], w3[j]);
            }
        });
        static_for<MS>([&](auto IA) __attribute__((always_inline)) {
            static_for<MS>([&](auto IB) __attribute__((always_inline)) {
                constexpr int ia = IA, ib = IB;
                if constexpr (ib >= ia) {
                    T Kv = T(0);
                    if (es && ib < S) {
                        // sin, cos of k (R_a + R_b) by the addition theorem: the contact cutoff (the
                        // launcher sends the cutoff at lambda_a + lambda_b to the run-time-length kernel)
                        const T sp = sn[ia] * cs[ib] + cs[ia] * sn[ib];
                        const T cp = cs[ia] * cs[ib] - sn[ia] * sn[ib];
                        constexpr int q = pair_slot<MS>(ia, ib);
                        Kv = screening_hat_p<T>(km, k.scR[q], sp, cp, k.p1[q], k.p2[q], k.p3[q], k.p4[q]);
                    }
                    K[pair_slot<MS>(ia, ib)] = Kv;
                }
            });
        });
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) acc[m] = mk<T>(T(0), T(0));
    static_for<MS>([&](auto J) __attribute__((always_inline)) {
        constexpr int j = J;
        if (j < S) {
            const T a0 = k.a0[j], a1 = k.a1[j];
            const T m0 = w2[j] * a0, m1 = w2[j] * a1, m4 = w3[j] * a1;
            acc[0].x += u[j].x * m0; acc[0].y += u[j].y * m0;
            acc[1].x += u[j].x * m1; acc[1].y += u[j].y * m1;
            acc[2].x += u[j].x * w2[j]; acc[2].y += u[j].y * w2[j];
            acc[3].x += u[j].x * w3[j]; acc[3].y += u[j].y * w3[j];
            acc[4].x += u[j].x * m4; acc[4].y += u[j].y * m4;
        }
    });
    if (!(es && ok)) return;
    // the bath term enters the k = 0 element of the pair-correlation part only
    const bool z0 = !diff && kw.zero(e);
    T invD = T(0);
    if constexpr (!TAB)
        if (!kw.zero(e)) invD = k.four_pi_lB * rcp_r(pd.denom(e));
    static_for<MS>([&](auto IS) __attribute__((always_inline)) {
        constexpr int is = IS;
        if (is < S) {
            cx<T> ea = mk<T>(T(0), T(0));
            static_for<MS>([&](auto J) __attribute__((always_inline)) {
                constexpr int j = J;
                if (j < S) {
                    constexpr int q = is <= j ? pair_slot<MS>(is, j) : pair_slot<MS>(j, is);
                    const T Kij = K[q];
                    const T ux = z0 ? u[j].x - k.bath[j] : u[j].x;
                    if constexpr (TAB) {
                        ea.x += Kij * ux;
                        ea.y += Kij * u[j].y;
                    } else {
                        const T Pz = invD * k.zz[q];
                        ea.x += Kij * ux - Pz * u[j].x;
                        ea.y += (Kij - Pz) * u[j].y;
                    }
                }
            });
            ct::gst(dst + (long long)is * NC, ea);
        }
    });
}

// Products of one species at one node without electrostatics (species by species).
template <typename T, class ZW>
__device__ __forceinline__ void z1_species(const Consts &c, const ZW &kw, const double *tab, long long TS, int S,
                                           int jsp, int e, bool ok, long long ti, cx<T> u, cx<T> (&acc)[5]) {
    T w2, w3;
    if constexpr (std::is_same<T, double>::value) {
        w2 = ok ? ct::cld(tab + (long long)jsp * TS + ti) : T(0);
        w3 = ok ? ct::cld(tab + (long long)(S + jsp) * TS + ti) : T(0);
    } else {
        weight_w2_w3<T>(kw.kmag(e), T(c.R[jsp]), w2, w3);
    }
    const T a0 = T(c.i4piR2[jsp]), a1 = T(c.i4piR[jsp]);
    const T m0 = w2 * a0, m1 = w2 * a1, m4 = w3 * a1;
    acc[0].x += u.x * m0; acc[0].y += u.y * m0;
    acc[1].x += u.x * m1; acc[1].y += u.y * m1;
    acc[2].x += u.x * w2; acc[2].y += u.y * w2;
    acc[3].x += u.x * w3; acc[3].y += u.y * w3;
    acc[4].x += u.x * m4; acc[4].y += u.y * m4;
}

// The seven inverse transforms of Z1 and their stores.  Along a z pencil k_x and k_y are
// constant, so the x and y components of the vector densities are -i k_x and -i k_y times the
// transform of their scalar sum; only n0..n3, the two vector sums' k_z multiples and the nV1 sum
// are transformed.  Transform t, its source sum and whether it is multiplied by -i k_z:
//   t = 0..3: acc[t] (n0..n3; t = 3 also gives the x, y components of nV2)
//   t = 4: acc[4] (x, y components of nV1);  t = 5: -i k_z acc[4] (nV1_z);  t = 6: -i k_z acc[3] (nV2_z)
template <typename T, class F, int NO, class ZW>
__device__ __forceinline__ void z1_inverse(const Geo &g, const Z1Args &a, const ZW &kw, cx<T> *lds, int &ph,
                                           const cx<T> *tw, int Pact, long long rs, long long off,
                                           const cx<T> (&acc)[NO][5], bool n3) {
    const Consts &c = *g.cs;
    const long long NC = g.NC;
    const int ntr = n3 ? 1 : 7;
    const T invN = T(c.invN);
    cx<T> v[F::V];
    typename F::template TwReg<1> tri;   // inverse twiddles, shared by the output transforms
    F::template load_tw<1>(tri, tw);
    for (int t = 0; t < ntr; ++t) {
        const int src = n3 ? 3 : (t < 5 ? t : (t == 5 ? 4 : 3));
        const bool kzm = t >= 5;
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            // source sum selected with compile-time register indices
            cx<T> sm = acc[i][3];
#pragma unroll
            for (int m = 0; m < 5; ++m)
                if (m == src) sm = acc[i][m];
            if (kzm) {
                int p, e;
                F::template in_pos<1>(i, p, e);
                const T kd = kw.comp(e, 2);
                sm = mk<T>(kd * sm.y, -kd * sm.x);   // -i k_z s
            }
            v[i] = mk<T>(sm.x * invN, sm.y * invN);
        }
        F::template run<1>(v, lds, ph, tri);
        // store the transform as output o, times -i k_d for d = 0 (x) or 1 (y), plain for d < 0
        auto store = [&](int o, int d) {
            cx<T> *dst = reinterpret_cast<cx<T> *>(a.specB) + (long long)o * NC + off;
#pragma unroll
            for (int i = 0; i < F::template nout<1>(); ++i) {
                int p, e;
                const bool ok = F::template out_pos<1>(i, p, e);
                if (!(ok && p < Pact)) continue;
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
        } else if (g.compact) {
            // compact layout: n0..n3, the nV1 sum, nV1_z, nV2_z (the inverse y pass expands)
            store(t < 5 ? t : (t == 5 ? 6 : 9), -1);
        } else if (t < 4) {
            store(t, -1);
            if (t == 3) {
                store(7, 0);
                store(8, 1);
            }
        } else if (t == 4) {
            store(4, 0);
            store(5, 1);
        } else {
            store(t == 5 ? 6 : 9, -1);
        }
    }
}

template <typename T, int L, int P, int NTB, int MS>
__global__ __launch_bounds__(NTB, (z1_waves<T, L, NTB>())) void k_z1c(Geo g_in, Z1Args a) {
    using F = ct::Fft<T, typename ct::PlanT<T, L>::type, P, NTB, false, 2, 0, false, z1_redo<T, L>()>;
    constexpr int NO = F::template nout<-1>();
    static_assert(NO == F::template nin<1>(), "inverse must start where the forward ends");
    constexpr bool TAB = z_fp64_factors<T, L>();
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[F::LDS_ELEMS];
    const Consts &c = *g.cs;
    const int Kx = g.Kx, S = g.S;
    const long long NC = g.NC;
    static_assert(NTB % P == 0, "a thread keeps one column");
    const ZTile zt = z_tile<P>(g);
    const int Pact = zt.Pact;
    const long long rs = (long long)g.ny * Kx;
    const long long off = zt.off;
    const cx<T> *tw = twp<T>(g, 2);
    const bool n3 = n3_wanted(a.n3_only);
    const bool es = MS > 0 && c.es && !n3;
    const ZWaveOf<T, L> kw(c, zt.x, zt.y);
    // the products' constants, read before the first store
    [[maybe_unused]] const Z1Const<T, (MS > 0 ? MS : 1)> kc(c);
    const double *tab = TAB ? g.tab64 + off : nullptr;
    [[maybe_unused]] const long long TS = z_tab_row<L>(rs);
    cx<T> acc[NO][5];
    cx<T> v[F::V];
    int ph = 0;
    typename F::template TwReg<-1> trs;   // forward twiddles, shared by the species transforms
    F::template load_tw<-1>(trs, tw);
    // each species' inputs are fetched while the previous species transforms
    constexpr int NIN = F::template nin<-1>();
    cx<T> vin[NIN];
    auto load_species = [&](int jsp) {
        const cx<T> *src = reinterpret_cast<const cx<T> *>(a.specA) + (long long)jsp * NC + off;
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            int p, e;
            const bool ok = F::template in_pos<-1>(i, p, e);
            vin[i] = (ok && p < Pact) ? ct::gld(src + e * rs + p) : mk<T>(T(0), T(0));
        }
    };
    load_species(0);
    if constexpr (MS == 0) {
#pragma unroll
        for (int i = 0; i < NO; ++i)
#pragma unroll
            for (int m = 0; m < 5; ++m) acc[i][m] = mk<T>(T(0), T(0));
        for (int jsp = 0; jsp < S; ++jsp) {
#pragma unroll
            for (int i = 0; i < NIN; ++i) v[i] = vin[i];
            if (jsp + 1 < S) load_species(jsp + 1);
            F::template run<-1>(v, lds, ph, trs);
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                int p, e;
                const bool ok = F::template out_pos<-1>(i, p, e) && p < Pact;
                z1_species<T>(c, kw, tab, TS, S, jsp, e, ok, ok ? z_tab<L>(e) * rs + p : 0, v[i], acc[i]);
            }
        }
    } else {
        // all species transformed first (S <= MS), then the products node by node
        cx<T> us[MS][NO];
        static_for<MS>([&](auto J) __attribute__((always_inline)) {
            constexpr int jsp = J;
#pragma unroll
            for (int i = 0; i < NO; ++i) us[jsp][i] = mk<T>(T(0), T(0));
            if (jsp < S) {
#pragma unroll
                for (int i = 0; i < NIN; ++i) v[i] = vin[i];
                if (jsp + 1 < S) load_species(jsp + 1);
                F::template run<-1>(v, lds, ph, trs);
#pragma unroll
                for (int i = 0; i < NO; ++i) us[jsp][i] = v[i];
            }
        });
        Poisson<T> pd;
        if constexpr (!TAB) pd = Poisson<T>(g, c, zt.x, zt.y);
        static_for<NO>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = I;
            int p, e;
            const bool ok = F::template out_pos<-1>(i, p, e) && p < Pact;
            const long long ti = ok ? e * rs + p : 0;
            cx<T> u[MS];
#pragma unroll
            for (int j = 0; j < MS; ++j) u[j] = us[j][i];
            z1_node<TAB>(kc, a.diff != 0, kw, pd, tab, TS, NC, S, es, e, ok, ok ? z_tab<L>(e) * rs + p : 0, u, acc[i],
                           reinterpret_cast<cx<T> *>(a.specA) + off + ti);
        });
    }
    z1_inverse<T, F, NO>(g, a, kw, lds, ph, tw, Pact, rs, off, acc, n3);
}

// Z1 from z spectra: the same products and inverse transforms as k_z1c, for species spectra
// that the plain z pass has already transformed along z (the autotuner's split Z1 shapes).  With
// the forward transform in its own kernel, this one needs neither the prefetched inputs nor the
// forward twiddles in registers.  Each thread reads the species values at the positions it
// starts the inverse transforms from and overwrites them with the electrostatic spectra only
// after reading them.
template <typename T, int L, int P, int NTB, int MS>
__global__ __launch_bounds__(NTB, (z1_waves<T, L, NTB>())) void k_z1s(Geo g_in, Z1Args a) {
    using F = ct::Fft<T, typename ct::PlanT<T, L>::type, P, NTB, false, 2, 0, false, z1_redo<T, L>()>;
    constexpr int NO = F::template nin<1>();
    constexpr bool TAB = z_fp64_factors<T, L>();
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[F::LDS_ELEMS];
    const Consts &c = *g.cs;
    const int Kx = g.Kx, S = g.S;
    const long long NC = g.NC;
    static_assert(NTB % P == 0, "a thread keeps one column");
    const ZTile zt = z_tile<P>(g);
    const int Pact = zt.Pact;
    const long long rs = (long long)g.ny * Kx;
    const long long off = zt.off;
    const cx<T> *tw = twp<T>(g, 2);
    const bool n3 = n3_wanted(a.n3_only);
    const bool es = MS > 0 && c.es && !n3;
    const ZWaveOf<T, L> kw(c, zt.x, zt.y);
    // the products' constants, read before the first store
    [[maybe_unused]] const Z1Const<T, (MS > 0 ? MS : 1)> kc(c);
    const double *tab = TAB ? g.tab64 + off : nullptr;
    [[maybe_unused]] const long long TS = z_tab_row<L>(rs);
    cx<T> acc[NO][5];
    if constexpr (MS == 0) {
        // species by species, every node's input of a species in flight together
#pragma unroll
        for (int i = 0; i < NO; ++i)
#pragma unroll
            for (int m = 0; m < 5; ++m) acc[i][m] = mk<T>(T(0), T(0));
        for (int jsp = 0; jsp < S; ++jsp) {
            const cx<T> *src = reinterpret_cast<const cx<T> *>(a.specA) + (long long)jsp * NC + off;
            cx<T> uin[NO];
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                int p, e;
                const bool ok = F::template in_pos<1>(i, p, e) && p < Pact;
                uin[i] = ok ? ct::gld(src + e * rs + p) : mk<T>(T(0), T(0));
            }
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                int p, e;
                const bool ok = F::template in_pos<1>(i, p, e) && p < Pact;
                z1_species<T>(c, kw, tab, TS, S, jsp, e, ok, ok ? z_tab<L>(e) * rs + p : 0, uin[i], acc[i]);
            }
        }
    } else {
        Poisson<T> pd;
        if constexpr (!TAB) pd = Poisson<T>(g, c, zt.x, zt.y);
        static_for<NO>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = I;
            int p, e;
            const bool ok = F::template in_pos<1>(i, p, e) && p < Pact;
            const long long ti = ok ? e * rs + p : 0;
            cx<T> *src = reinterpret_cast<cx<T> *>(a.specA) + off + ti;
            cx<T> u[MS];
#pragma unroll
            for (int j = 0; j < MS; ++j) u[j] = (ok && j < S) ? ct::gld(src + (long long)j * NC) : mk<T>(T(0), T(0));
            z1_node<TAB>(kc, a.diff != 0, kw, pd, tab, TS, NC, S, es, e, ok, ok ? z_tab<L>(e) * rs + p : 0, u, acc[i], src);
        });
    }
    int ph = 0;
    z1_inverse<T, F, NO>(g, a, kw, lds, ph, tw, Pact, rs, off, acc, n3);
}

// Z2: forward z transform of the ten dPhi/dn spectra, back-convolution with conj(w_hat)
// (eq. muHS; the vector parts enter as +i k_d times a w3 weight), plus the electrostatic
// spectra Z1 left in specA, times 1/N, inverse z -> specA.  Z2_POISSON instead forms the
// potential of weighted source spectra.
// Weights: tables or on the fly (z_tables).
template <typename T, int L, int P, int NTB>
__global__ __launch_bounds__(NTB) void k_z2c(Geo g_in, Z2Args a) {
    using F = ct::Fft<T, typename ct::PlanT<T, L>::type, P, NTB, false, 2, 0, false, z2_redo<T, L>()>;
    constexpr int NO = F::template nout<-1>();
    static_assert(NO == F::template nin<1>(), "inverse must start where the forward ends");
    constexpr bool TAB = std::is_same<T, double>::value;
    const int prob = (int)blockIdx.z;
    if (prob > 0) {
        const long long o = (long long)prob * g_in.pstride;
        g_in = shift(g_in, o);
        a = shift(a, o);
    }
    const Geo &g = g_in;
    if (gated_off(a.gate)) return;
    __shared__ cx<T> lds[F::LDS_ELEMS];
    const Consts &c = *g.cs;
    const int Kx = g.Kx, S = g.S;
    const long long NC = g.NC;
    static_assert(NTB % P == 0, "a thread keeps one column");
    const ZTile zt = z_tile<P>(g);
    const int Pact = zt.Pact;
    const long long rs = (long long)g.ny * Kx;
    const long long off = zt.off;
    const cx<T> *tw = twp<T>(g, 2);
    const ZWaveOf<T, L> kw(c, zt.x, zt.y);
    [[maybe_unused]] const long long TS = z_tab_row<L>(rs);
    // position of output register i of the forward transforms (recomputed at each use: a few
    // instructions from the thread index instead of registers held through the kernel)
    auto ee = [&](int i) {
        int p, e;
        F::template out_pos<-1>(i, p, e);
        return e;
    };
    auto okk = [&](int i) {
        int p, e;
        return F::template out_pos<-1>(i, p, e) && p < Pact;
    };
    auto ti = [&](int i) {
        int p, e;
        const bool ok = F::template out_pos<-1>(i, p, e) && p < Pact;
        return ok ? e * rs + p : 0;
    };
    cx<T> v[F::V];
    int ph = 0;
    // FP32: the forward twiddles in registers, shared by the input transforms (in FP64 the
    // register budget is better spent on the transforms themselves)
    constexpr bool TWR = std::is_same<T, float>::value;
    typename F::template TwReg<-1> trf;
    if constexpr (TWR) F::template load_tw<-1>(trf, tw);
    auto fwd = [&]() {
        if constexpr (TWR) F::template run<-1>(v, lds, ph, trf);
        else F::template run<-1>(v, lds, ph, tw);
    };
    auto load_fwd = [&](const cx<T> *src) {
#pragma unroll
        for (int i = 0; i < F::template nin<-1>(); ++i) {
            int p, e;
            const bool ok = F::template in_pos<-1>(i, p, e);
            v[i] = (ok && p < Pact) ? ct::gld(src + e * rs + p) : mk<T>(T(0), T(0));
        }
        fwd();
    };
    auto inv_store = [&](cx<T> *dst) {
        F::template run<1>(v, lds, ph, tw);
#pragma unroll
        for (int i = 0; i < F::template nout<1>(); ++i) {
            int p, e;
            const bool ok = F::template out_pos<1>(i, p, e);
            if (ok && p < Pact) ct::gst(dst + e * rs + p, v[i]);
        }
    };

    if (a.mode == Z2_POISSON) {
        // phi_hat = 4 pi l_B (sum_j w_j src_j) / D(k), zero mode 0; x invN; output in specA[0].
        double acc[NO][2];
#pragma unroll
        for (int i = 0; i < NO; ++i) acc[i][0] = acc[i][1] = 0.0;
        for (int is = 0; is < a.nsrc; ++is) {
            load_fwd(reinterpret_cast<const cx<T> *>(a.specA) + (long long)is * NC + off);
            double wj = 0.0;   // a.wsrc[is] read with constant indices (no scratch copy of the arguments)
#pragma unroll
            for (int k = 0; k < DFT_MAX_SPECIES; ++k)
                if (k == is) wj = a.wsrc[k];
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                acc[i][0] += wj * (double)v[i].x;
                acc[i][1] += wj * (double)v[i].y;
            }
        }
        const Poisson<double> pd(g, c, zt.x, zt.y);
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            double m = 0.0;
            if (!kw.zero(ee(i))) m = c.four_pi_lB / pd.denom(ee(i)) * c.invN;
            v[i] = mk<T>(T(acc[i][0] * m), T(acc[i][1] * m));
        }
        inv_store(reinterpret_cast<cx<T> *>(a.specA) + off);
        return;
    }

    // six sums of the derivative spectra: u0..u3 and v1 = sum_d i k_d dPhi_V1,d, v2 likewise
    cx<T> u[6][NO];
#pragma unroll
    for (int m = 0; m < 6; ++m)
#pragma unroll
        for (int i = 0; i < NO; ++i) u[m][i] = mk<T>(T(0), T(0));
    // Eight forward transforms: along a z pencil k_x and k_y are constant, so the x and y parts of
    // each vector sum, i k_x dPhi_x + i k_y dPhi_y, are combined before one transform; the z parts
    // are transformed and multiplied by i k_z after.  Transform t: 0..3 the scalars (u0..u3);
    // 4, 6 the combined x, y parts of V1, V2; 5, 7 their z parts.
    // compact layout: slots 4 and 7 already hold i k_x dPhi_x + i k_y dPhi_y and all eight inputs
    // are plain spectra; in FP32 tiles of at most eight values per thread each is fetched while the
    // previous one transforms (FP64 tiles have no registers to spare for it)
    constexpr bool PF = std::is_same<T, float>::value && NO <= 8;
    constexpr int NIN = F::template nin<-1>();
    cx<T> vin[NIN];
    auto slot_of = [](int t) { return t < 4 ? t : (t == 4 ? 4 : (t == 5 ? 6 : (t == 6 ? 7 : 9))); };
    auto fetch = [&](int t) {
        const int al = slot_of(t);
        const cx<T> *src = reinterpret_cast<const cx<T> *>(a.specB) + (long long)al * NC + off;
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            int p, e;
            const bool ok = F::template in_pos<-1>(i, p, e);
            vin[i] = (ok && p < Pact) ? ct::gld(src + e * rs + p) : mk<T>(T(0), T(0));
        }
    };
    if (PF && g.compact) fetch(0);
    for (int t = 0; t < 8; ++t) {
        const int m = t < 4 ? t : (t < 6 ? 4 : 5);
        if (g.compact) {
            if constexpr (PF) {
#pragma unroll
                for (int i = 0; i < NIN; ++i) v[i] = vin[i];
                if (t + 1 < 8) fetch(t + 1);
                fwd();
            } else {
                load_fwd(reinterpret_cast<const cx<T> *>(a.specB) + (long long)slot_of(t) * NC + off);
            }
        } else if (t < 4 || t == 5 || t == 7) {
            const int al = t < 4 ? t : (t == 5 ? 6 : 9);
            load_fwd(reinterpret_cast<const cx<T> *>(a.specB) + (long long)al * NC + off);
        } else {
            const int al = t == 4 ? 4 : 7;
            const cx<T> *sx = reinterpret_cast<const cx<T> *>(a.specB) + (long long)al * NC + off;
            const cx<T> *sy = sx + NC;
#pragma unroll
            for (int i = 0; i < F::template nin<-1>(); ++i) {
                int p, e;
                const bool ok = F::template in_pos<-1>(i, p, e) && p < Pact;
                cx<T> w = mk<T>(T(0), T(0));
                if (ok) {
                    const cx<T> fx = ct::gld(sx + e * rs + p), fy = ct::gld(sy + e * rs + p);
                    const T kx = kw.comp(e, 0), ky = kw.comp(e, 1);
                    w = mk<T>(-(kx * fx.y + ky * fy.y), kx * fx.x + ky * fy.x);   // i k_x fx + i k_y fy
                }
                v[i] = w;
            }
            fwd();
        }
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            cx<T> w = v[i];
            if (t == 5 || t == 7) {
                const T kd = kw.comp(ee(i), 2);
                w = mk<T>(-kd * w.y, kd * w.x);   // + i k_z w
            }
#pragma unroll
            for (int mm = 0; mm < 6; ++mm)
                if (mm == m) { u[mm][i].x += w.x; u[mm][i].y += w.y; }
        }
    }
    const T invN = T(c.invN);
    constexpr int NOF = TAB ? 1 : NO;
    T kmag[NOF];
    if constexpr (!TAB) {
#pragma unroll
        for (int i = 0; i < NO; ++i) kmag[i] = kw.kmag(ee(i));
    }
    // FP32: the electrostatic spectra of species is + 1 fetched while species is transforms
    // (slot is + 1 is written only in the next iteration, after every read of it)
    cx<T> evn[NO];
    const bool es = c.es != 0;   // read once (a read after the stores below would be repeated)
    auto fetch_es = [&](int is) {
        const cx<T> *esrc = reinterpret_cast<const cx<T> *>(a.specA) + (long long)is * NC + off;
#pragma unroll
        for (int i = 0; i < NO; ++i) evn[i] = (es && okk(i)) ? ct::gld(esrc + ti(i)) : mk<T>(T(0), T(0));
    };
    if constexpr (PF) fetch_es(0);
    for (int is = 0; is < S; ++is) {
        const T Ri = T(c.R[is]), a0 = T(c.i4piR2[is]), a1 = T(c.i4piR[is]);
        if constexpr (!PF) fetch_es(is);
        cx<T> ev[NO];
#pragma unroll
        for (int i = 0; i < NO; ++i) ev[i] = evn[i];
        if (PF && is + 1 < S) fetch_es(is + 1);
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            T w2, w3;
            if constexpr (TAB) {
                int p, e;
                const bool ok = F::template out_pos<-1>(i, p, e) && p < Pact;
                const double *tab = g.tab64 + off + (ok ? z_tab<L>(e) * rs + p : 0);
                w2 = ct::cld(tab + (long long)is * TS);
                w3 = ct::cld(tab + (long long)(S + is) * TS);
            } else {
                weight_w2_w3<T>(kmag[i], Ri, w2, w3);
            }
            const T s2x = u[0][i].x * a0 + u[1][i].x * a1 + u[2][i].x;
            const T s2y = u[0][i].y * a0 + u[1][i].y * a1 + u[2][i].y;
            const T s3x = u[3][i].x + u[4][i].x * a1 + u[5][i].x;
            const T s3y = u[3][i].y + u[4][i].y * a1 + u[5][i].y;
            T ex = -(s2x * w2 + s3x * w3);
            T ey = -(s2y * w2 + s3y * w3);
            ex += ev[i].x;
            ey += ev[i].y;
            v[i] = mk<T>(ex * invN, ey * invN);
        }
        inv_store(reinterpret_cast<cx<T> *>(a.specA) + (long long)is * NC + off);
    }
}

}  // namespace dft
