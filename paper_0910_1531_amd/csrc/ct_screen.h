// Passes of the RFD screening operator in the compiled lengths (FP64): ball averages of the fields at
// several radii per launch.
#pragma once

#include "ct_rows.h"
#include "dft_screen.h"

namespace dft {

// Columns of a z tile: 128-byte segments of a z plane where the tile still fits the LDS twice.
constexpr int ball_width(int L) { return L >= 192 && L <= 256 ? 8 : 4; }

// Ball averages along z: the full spectra of two fields (blockIdx.z) in specA, times B(|k| R_m) / N for
// every radius of the batch, inverse z -> specB slot m S + field.  The spectra are read once per batch
// and stay in registers; the ball's transform is evaluated once for both fields.  One radius a launch
// repeated the forward z transform of the spectra for every radius.  128^3, two fields, five radii: 65 us
// (2.6 TB/s of writes), 116 before; bound by the writes and the FP64 sine and cosine.
template <int L, int P, int NTB>
__global__ __launch_bounds__(NTB) void k_ballc(Geo g, BallArgs a) {
    using F = ct::Fft<double, typename ct::PlanT<double, L>::type, P, NTB, false, 2, 0, false,
                      L == 216 || L == 243 || L == 432 || L == 486>;   // (index arithmetic redone where held it spills)
    constexpr int NI = F::template nin<1>();
    __shared__ cx<double> lds[F::LDS_ELEMS];
    const Consts &c = *g.cs;
    const ZTile zt = z_tile<P>(g);
    const long long rs = (long long)g.ny * g.Kx, NC = g.NC;
    const ZWave<double> kw(c, zt.x, zt.y);
    const int f0 = 2 * (int)blockIdx.z;
    const bool two = f0 + 1 < g.S;
    cx<double> sp[2][NI];
    double kmag[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        int p, e;
        const bool ok = F::template in_pos<1>(i, p, e) && p < zt.Pact;
        const cx<double> *src = reinterpret_cast<const cx<double> *>(a.specA) + f0 * NC + zt.off + (ok ? e * rs + p : 0);
        sp[0][i] = ok ? ct::gld(src) : mk<double>(0.0, 0.0);
        sp[1][i] = ok && two ? ct::gld(src + NC) : mk<double>(0.0, 0.0);
        kmag[i] = kw.kmag(e);
    }
    typename F::template TwReg<1> tw;
    F::template load_tw<1>(tw, twp<double>(g, 2));
    const double invN = c.invN;
    int ph = 0;
    for (int m = 0; m < a.nodes; ++m) {
        double ball[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) ball[i] = ball_mean<double>(kmag[i], a.R[m]) * invN;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1 && !two) break;
            cx<double> v[F::V];
#pragma unroll
            for (int i = 0; i < NI; ++i) v[i] = mk<double>(sp[h][i].x * ball[i], sp[h][i].y * ball[i]);
            F::template run<1>(v, lds, ph, tw);
            cx<double> *dst = reinterpret_cast<cx<double> *>(a.specB) + (long long)(m * g.S + f0 + h) * NC + zt.off;
#pragma unroll
            for (int i = 0; i < F::template nout<1>(); ++i) {
                int p, e;
                if (F::template out_pos<1>(i, p, e) && p < zt.Pact) ct::gst(dst + e * rs + p, v[i]);
            }
        }
    }
}

// Inverse x of the batch's slots with the interpolation in the radius: at every node the sum over the
// batch's radii of the barycentric weight of its own R_SC times the ball average, written to (or added
// to) f_ref.  Two fields (blockIdx.y) share the weights; up to four waves a block, each with its own row
// pairs; the next slot's rows are fetched while one transforms.  Replaces a pass that wrote the averages
// in real space and one that read them, f_ref and the weights for every radius: 128^3, two fields, five
// radii 75 us, 230 before.
template <int L>
__global__ __launch_bounds__(256) void k_ballx(Geo g, BallArgs a) {
    using X = XRow<L>;
    using F = typename X::template F<double>;
    constexpr int PW = X::PW, NO = F::template nout<1>();
    __shared__ cx<double> lds[4 * F::TILE];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = (int)threadIdx.x & 63;
    cx<double> *tile = lds + w * F::TILE;
    const long long rows = (long long)g.ny * g.nz;
    const long long pair0 = ((long long)blockIdx.x * (blockDim.x / 64) + w) * PW;
    const int rows_here = (int)max(0LL, min((long long)(2 * PW), rows - 2 * pair0));
    const int f0 = 2 * (int)blockIdx.y, nf = min(2, g.S - f0);
    const cx<double> *in = reinterpret_cast<const cx<double> *>(a.specB) + 2 * pair0 * X::KX;
    HalfRows<double, L> half;
    half.load(in + (long long)f0 * g.NC, rows_here, lane);
    typename F::template TwReg<1> tw;
    F::template load_tw<1>(tw, twp<double>(g, 0), lane);
    const long long node0 = 2 * pair0 * L;
    double r[NO][2], inv_den[NO][2], acc[2][NO][2];
    int hit[NO][2];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        int p, e;
        const bool in_tile = F::template out_pos<1>(i, p, e, lane);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool ok = in_tile && 2 * p + h < rows_here;
            const unsigned o = (unsigned)((2 * p + h) * L + e);
            r[i][h] = ok ? ct::cld(at(a.rsc + node0, o * 8u)) : 0.0;
            inv_den[i][h] = ok ? ct::cld(at(a.inv_den + node0, o * 8u)) : 0.0;
            hit[i][h] = ok ? ct::cld(at(a.hit + node0, o * 4u)) : -1;
            acc[0][i][h] = acc[1][i][h] = 0.0;
        }
    }
    for (int m = 0; m < a.nodes; ++m) {
        double l[NO][2];
#pragma unroll
        for (int i = 0; i < NO; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                l[i][h] = hit[i][h] >= 0 ? (hit[i][h] == a.m0 + m ? 1.0 : 0.0) : a.w[m] / (r[i][h] - a.R[m]) * inv_den[i][h];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (q >= nf) break;
            F::sync();
            half.put(tile, lane);
            const int next = q + 1 < nf ? m * g.S + f0 + 1 : (m + 1 < a.nodes ? (m + 1) * g.S + f0 : -1);
            if (next >= 0) half.load(in + (long long)next * g.NC, rows_here, lane);
            F::sync();
            cx<double> v[F::V];
            F::template get<F::template rad<1>(0)>(v, tile, lane);
            int ph = lane;
            F::template run<1>(v, tile, ph, tw);
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                acc[q][i][0] += l[i][0] * v[i].x;
                acc[q][i][1] += l[i][1] * v[i].y;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        int p, e;
        if (!F::template out_pos<1>(i, p, e, lane)) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (2 * p + h >= rows_here) break;
            const unsigned o = (unsigned)((2 * p + h) * L + e) * 8u;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (q >= nf) break;
                double *dst = at(a.out + (long long)(f0 + q) * g.N + node0, o);
                ct::gst(dst, a.first ? acc[q][i][h] : ct::gld(dst) + acc[q][i][h]);
            }
        }
    }
}

}  // namespace dft
