// One time step on the row layout: the 19 populations of lattice row
// r = y + ny z are stored as 19 consecutive runs of nx values, population a
// of node x at element (19 r + a) nx + x.
//
// A step then reads, for every row, parts of the 9 row groups r - e_y - ny e_z
// and writes one row group: a few compact regions instead of 38 planes spread
// over the whole buffer, which keeps the DRAM page and bank traffic of
// neighbouring waves together.
//
//   stream_collide_rows_flat   one thread per node, 64 consecutive nodes per wave,
//                         per-lane source addresses: no idle lanes at any
//                         width, no second launch or second round of loads for
//                         the faces.
//   stream_collide_rows_wide   the same with 64-bit offsets, for layers beyond
//                         the reach of 32-bit ones.
//   stream_collide_rows   large FP32 lattices: each wave covers 64 consecutive
//                         x of one row, so a direction's source is a uniform
//                         address plus the lane's x; rows on a y or z face
//                         take the wall rule by scalar selects, the lanes of
//                         the x faces by a second group of loads.
#include "clbm_rows.hpp"

namespace clbm {

// One thread per node, 64 consecutive nodes (x fastest, across rows and
// layers) per wave, so no lane is idle at any width.
//
// Bound: HBM for FP32 and FP64 (256^3: 448 us per step, 5.7 TB/s, and 880 us,
// 5.8 TB/s, against 6.55 of a copy; the kernel with one wave per run of a row
// and the faces in a second launch took 464 and 904), arithmetic for FP16
// (227 against 271 us; the hash of the stochastic rounding and the relaxation
// rate, 61 VGPRs and eight waves per SIMD), latency of one pass below about
// 10^5 nodes (64^3 FP32: 8.0 against 18.6 us, 48^3 5.0 against 9.3).  Rows that
// are not whole cache lines gain most, since the lines two runs share meet in
// one workgroup: 200 x 190 x 220 FP32 250 against 375 us.
template <typename S, typename T, bool Forced, int LdAux, int StAux, int Route, bool Far>
__global__ void __launch_bounds__(MaxThreads<T>::value)
stream_collide_rows_flat_kernel(const S *__restrict__ A, S *__restrict__ B, Geom g, Relax<T> p, FlatGrid L) {
    const FlatLane<S, Far> k(g, L);
    if (k.i >= (uint32_t)g.n) return;
    T d[Q];
    gather_flat<S, T, LdAux, Far>(A + k.r0 * g.row, k.own, g, p, k.x, k.y, k.z, d);
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    row_store_at<S, T, StAux>(row_rsrc(B + k.r0 * g.row, 0xFFFFFFFFu), k.own, (uint32_t)g.nx * (uint32_t)sizeof(S), d,
                              p.sr != 0, sr_base(k.i, p.step));
}

template <typename S, typename T, bool Forced, int LdAux, int StAux, int Route>
__global__ void __launch_bounds__(MaxThreads<T>::value)
stream_collide_rows_kernel(const S *__restrict__ A, S *__restrict__ B, Geom g, Relax<T> p, RowGrid R) {
    int x;
    uint32_t ri;
    if (!row_of(R, x, ri) || x >= g.nx) return;
    const int y = (int)(ri % (uint32_t)g.ny), z = (int)(ri / (uint32_t)g.ny);
    T d[Q];
    if (y >= 1 && y <= g.ny - 2 && z >= 1 && z <= g.nz - 2)
        row_gather<S, T, LdAux, false, XGroupRows<S>::value>(A, g, p, x, y, z, d);
    else
        row_gather<S, T, LdAux, true, XGroupRows<S>::value>(A, g, p, x, y, z, d);
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    const uint32_t node = (uint32_t)x + (uint32_t)g.nx * ri;
    row_store<S, T, StAux>(B, g, x, y, z, d, p.sr != 0, sr_base(node, p.step));
}

// The flat kernel for layers beyond the reach of 32-bit offsets, in FP64 and
// FP16, and in FP32 below 64 columns (a wave per row would leave its lanes idle
// and, from 2^26 rows, need more than the 2^32 threads that a launch can have:
// the runtime starts the remainder only, without an error).  us per step, against the kernel with a wave per row: ten layers of
// 20 x 195 000 FP64 2407 against 6150, 70 x 112 000 FP16 2874 against 8319,
// 2000 x 7 900 FP16 2205 against 4602.
template <typename S, typename T, bool Forced, int Route>
__global__ void __launch_bounds__(MaxThreads<T>::value)
stream_collide_rows_wide_kernel(const S *__restrict__ A, S *__restrict__ B, Geom g, Relax<T> p, FlatGrid L) {
    const FlatLane<S, true> k(g, L);
    if (k.i >= (uint32_t)g.n) return;
    const WideNode<S> w(g, k.x, k.y, k.z);
    T d[Q];
#pragma unroll
    for (int a = 0; a < Q; ++a) d[a] = (T)Conv<S, T>::load(A[w.at(a, a)]);
    if (w.f.wave_touches_lid()) {
#pragma unroll
        for (int a = 1; a < Q; ++a) d[a] = wall_value<T>(d[a], p, a, w.f.lid(a));
    }
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, k.i, p.step);
#pragma unroll
    for (int a = 0; a < Q; ++a) B[w.own + a * w.run] = Conv<S, T>::store(d[a]);
}

template <typename S, typename T, bool Forced, int LdAux, int StAux, int Route>
static hipError_t launch_rows_k(const S *a, S *b, const Geom &g, const Relax<T> &p, const StepLaunch &c,
                                hipStream_t st) {
    const int threads = (c.bx * c.by + 63) / 64 * 64;
    const FlatLaunch L = flat_launch(g, sizeof(S), threads, c.xcd_remap);
    // Beyond 1 GiB FP32 and FP64 run 0-6% faster with offsets from the wave's
    // own layer (300 x 280 x 290: 733 against 772 us FP32, 1220 against 1299
    // FP64), FP16 between 3% faster and 4% slower.  From 4 GiB FP32 runs 2-6%
    // faster with one wave per run of a row (512^3 3449 against 3524 us; 500^3,
    // whole rows per workgroup, 3569 against 3784; between 65 and 400 columns,
    // 5.2 GB, as fast: 1924 against 1893 us at 100), FP64 and FP16 1-14% slower.
    const bool prefer_far = !std::is_same<S, __half>::value && (uint64_t)Q * sizeof(S) * (uint64_t)g.n > (1ull << 30);
    const bool prefer_rows = std::is_same<S, float>::value && !L.near && g.nx >= 64;
    if (!prefer_rows && (L.near || L.far)) {
        if (L.near && !(L.far && prefer_far))
            hipLaunchKernelGGL((stream_collide_rows_flat_kernel<S, T, Forced, LdAux, StAux, Route, false>),
                               dim3(L.blocks), dim3(threads), 0, st, a, b, g, p, L.grid);
        else
            hipLaunchKernelGGL((stream_collide_rows_flat_kernel<S, T, Forced, LdAux, StAux, Route, true>),
                               dim3(L.blocks), dim3(threads), 0, st, a, b, g, p, L.grid);
        return hipGetLastError();
    }
    if (!prefer_rows) {
        hipLaunchKernelGGL((stream_collide_rows_wide_kernel<S, T, Forced, Route>), dim3(L.blocks), dim3(threads), 0, st, a,
                           b, g, p, L.grid);
        return hipGetLastError();
    }
    RowGrid R;
    const uint32_t blocks = all_rows(g, threads, c.xcd_remap, R);
    hipLaunchKernelGGL((stream_collide_rows_kernel<S, T, Forced, LdAux, StAux, Route>), dim3(blocks), dim3(threads), 0,
                       st, a, b, g, p, R);
    return hipGetLastError();
}

template <typename S, typename T, bool Forced, int Route>
static hipError_t launch_rows_f(const void *A, void *B, const Geom &g, const Relax<T> &p, const StepLaunch &c,
                                hipStream_t st) {
    const S *a = (const S *)A;
    S *b = (S *)B;
    if (Route != 0)     // the printed form and the comparison model: only the store hint is tunable
        return c.nt_stores ? launch_rows_k<S, T, Forced, 0, 2, Route>(a, b, g, p, c, st)
                           : launch_rows_k<S, T, Forced, 0, 0, Route>(a, b, g, p, c, st);
    switch ((c.nt_loads ? 1 : 0) | (c.nt_stores ? 2 : 0)) {
    case 0: return launch_rows_k<S, T, Forced, 0, 0, Route>(a, b, g, p, c, st);
    case 1: return launch_rows_k<S, T, Forced, 2, 0, Route>(a, b, g, p, c, st);
    case 2: return launch_rows_k<S, T, Forced, 0, 2, Route>(a, b, g, p, c, st);
    default: return launch_rows_k<S, T, Forced, 2, 2, Route>(a, b, g, p, c, st);
    }
}

template <typename S, typename T>
static hipError_t launch_rows_t(const void *A, void *B, const Geom &g, const Relax<T> &p, bool forced, int route,
                                const StepLaunch &c, hipStream_t st) {
    if (route == 2) return forced ? hipErrorInvalidValue : launch_rows_f<S, T, false, 2>(A, B, g, p, c, st);
    if (route == 0)
        return forced ? launch_rows_f<S, T, true, 0>(A, B, g, p, c, st) : launch_rows_f<S, T, false, 0>(A, B, g, p, c, st);
    return forced ? launch_rows_f<S, T, true, 1>(A, B, g, p, c, st) : launch_rows_f<S, T, false, 1>(A, B, g, p, c, st);
}

hipError_t launch_step_rows(int storage, const void *A, void *B, const Geom &g, const Relax<double> &pd,
                            const Relax<float> &pf, bool forced, int route, const StepLaunch &c, hipStream_t st) {
    switch (storage) {
    case 0: return launch_rows_t<double, double>(A, B, g, pd, forced, route, c, st);
    case 1: return launch_rows_t<float, float>(A, B, g, pf, forced, route, c, st);
    default: return launch_rows_t<__half, float>(A, B, g, pf, forced, route, c, st);
    }
}

}  // namespace clbm
