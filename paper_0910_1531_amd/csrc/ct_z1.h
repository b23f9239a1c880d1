// Launchers of the compiled-length Z1 pass, with the tile widths the autotuner chooses among.
#pragma once

#include "ct_kernels.h"

namespace dft {

template <typename T> constexpr int z_width(int v);
template <> constexpr int z_width<float>(int v) { return v == 0 ? 8 : v == 1 ? 4 : 16; }
template <> constexpr int z_width<double>(int v) { return v == 0 ? 4 : v == 1 ? 2 : 8; }

template <typename T, int L, int P, int NTB>
void launch_z1c_shape(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    const dim3 grid((unsigned)ct_cdiv(g.ny * g.Kx, P), 1, (unsigned)g.nprob);   // flattened (y, kx) columns
    if (!es) hipLaunchKernelGGL((k_z1c<T, L, P, NTB, 0>), grid, dim3(NTB), 0, s, g, a);
    else {
        // the pair accumulators are sized for the species count: fewer registers for S < 4
        if (g.S <= 2) hipLaunchKernelGGL((k_z1c<T, L, P, NTB, 2>), grid, dim3(NTB), 0, s, g, a);
        else if (g.S == 3) hipLaunchKernelGGL((k_z1c<T, L, P, NTB, 3>), grid, dim3(NTB), 0, s, g, a);
        else hipLaunchKernelGGL((k_z1c<T, L, P, NTB, 4>), grid, dim3(NTB), 0, s, g, a);
    }
    ct_check("z1 (compiled length)");
}

template <typename T, int L, int V>
void launch_z1c_var(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    constexpr int P = z_width<T>(V);
    launch_z1c_shape<T, L, P, fit_threads(L, P, 4, 512)>(g, a, es, s);
}

// The one shape of the lengths outside DFT_CT_LENGTHS: shape 0's columns, fused.
template <typename T, int L>
void launch_z1c_one(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    constexpr int P = z_width<T>(0), NTB = z_one_threads<T, L>(P);
    launch_z1c_shape<T, L, P, NTB>(g, a, es, s);
}

// Split shapes (V = 3, 4, 5 for the tile widths of V - 3): the plain z pass transforms the
// species spectra in place, then k_z1s forms the products and the inverse transforms.
template <typename T, int L, int V>
void launch_z1s_var(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    YArgs za{a.specA, g.S, -1, a.gate};
    za.axis = 2;
    launch_y<T>(g, za, s);
    constexpr int P = z_width<T>(V), NTB = fit_threads(L, P, 4, 512);
    dim3 grid((unsigned)ct_cdiv(g.ny * g.Kx, P), 1, (unsigned)g.nprob);   // flattened (y, kx) columns
    if (!es) hipLaunchKernelGGL((k_z1s<T, L, P, NTB, 0>), grid, dim3(NTB), 0, s, g, a);
    else if (g.S <= 2) hipLaunchKernelGGL((k_z1s<T, L, P, NTB, 2>), grid, dim3(NTB), 0, s, g, a);
    else if (g.S == 3) hipLaunchKernelGGL((k_z1s<T, L, P, NTB, 3>), grid, dim3(NTB), 0, s, g, a);
    else hipLaunchKernelGGL((k_z1s<T, L, P, NTB, 4>), grid, dim3(NTB), 0, s, g, a);
    ct_check("z1 from z spectra (compiled length)");
}

template <typename T, int L>
void launch_z1c_len(const Geo &g, const Z1Args &a, int es, hipStream_t s, int v) {
    if (v == 1) launch_z1c_var<T, L, 1>(g, a, es, s);
    else if (v == 2) launch_z1c_var<T, L, 2>(g, a, es, s);
    else if (v == 3) launch_z1s_var<T, L, 0>(g, a, es, s);
    else if (v == 4) launch_z1s_var<T, L, 1>(g, a, es, s);
    else if (v == 5) launch_z1s_var<T, L, 2>(g, a, es, s);
    else launch_z1c_var<T, L, 0>(g, a, es, s);
}

// The lengths compiled in one shape (a source of their own, for the compile time).
template <typename T>
bool launch_z1_more(const Geo &g, const Z1Args &a, int es, hipStream_t s);

template <typename T>
bool launch_z1_more_lengths(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    switch (g.nz) {
#define DFT_CASE(n) case n: launch_z1c_one<T, n>(g, a, es, s); return true;
        DFT_CT_MORE_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return false;
    }
}

template <typename T>
bool launch_z1_lengths(const Geo &g, const Z1Args &a, int es, hipStream_t s) {
    if (launch_z1_wide<T>(g, a, es, s)) return true;
    const int v = g.tune[TUNE_Z1][std::is_same<T, float>::value ? 1 : 0];
    switch (g.nz) {
#define DFT_CASE(n) case n: launch_z1c_len<T, n>(g, a, es, s, v); return true;
        DFT_CT_LENGTHS(DFT_CASE)
#undef DFT_CASE
        default: return launch_z1_more<T>(g, a, es, s);
    }
}

}  // namespace dft
