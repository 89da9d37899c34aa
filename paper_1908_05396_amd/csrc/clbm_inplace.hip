// In-place stepping with one state buffer: the AA access pattern.
//
// The buffer holds pre-collision populations in their natural slots (slot a
// of node x holds f_a(x)) before an even step.
//   even step: every node collides its own populations and stores f~_a into
//              its own slot opp(a);
//   odd step:  node x pulls f~_a(x - e_a) from slot opp(a) of x - e_a (where
//              the even step left it), collides, and pushes f~_a(x) to slot a
//              of x + e_a, its natural slot for the next even step.
// A pair of launches advances two time steps (collide, stream, collide,
// stream) with the same memory traffic per node update as the two-buffer
// pull, in half the memory.  Within a launch each node reads and then
// overwrites exactly the locations no other node touches: the odd step's read
// set {(opp(a), x - e_a)} equals its write set {(a, x + e_a)}.  Walls: a
// ghost source returns the node's own f~_opp(a), which the even step left in
// slot a of x, plus the lid term; a ghost target sends f~_a back into slot
// opp(a) of x with the lid term of direction opp(a) — the value the pull rule
// gives at the next step.  Periodic axes wrap.
#include "clbm_rows.hpp"

namespace clbm {

namespace {

__device__ inline bool wrap(int &c, int n, int periodic) {
    if (c >= 0 && c < n) return true;
    if (!periodic) return false;
    c = c < 0 ? c + n : c - n;
    return true;
}

__device__ inline void locate(const LaunchGrid &L, int &x, int &y, int &z) {
    uint32_t b = blockIdx.x;
    if (L.remap && b < L.aligned) b = (b & 7u) * (L.aligned >> 3) + (b >> 3);
    const uint32_t tx = b % L.gx;
    b /= L.gx;
    const uint32_t ty = b % L.gy;
    z = (int)(b / L.gy);
    x = (int)(tx * blockDim.x + threadIdx.x);
    y = (int)(ty * blockDim.y + threadIdx.y);
}

}  // namespace

// The even step writes back into the lines it has just read.
constexpr int EvenStAux = 0;

template <typename S, typename T, bool Forced, int Route>
__global__ void __launch_bounds__(MaxThreads<T>::value)
aa_even_kernel(S *__restrict__ A, Geom g, Relax<T> p, LaunchGrid L) {
    int x, y, z;
    locate(L, x, y, z);
    if (x >= g.nx || y >= g.ny) return;
    const uint32_t self = (uint32_t)x + (uint32_t)g.nx * (uint32_t)y + (uint32_t)g.nxy * (uint32_t)z;
    T d[Q];
#pragma unroll
    for (int a = 0; a < Q; ++a) d[a] = (T)Plane<S>::load(A, g, a, self);
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, self, p.step);
#pragma unroll
    for (int a = 0; a < Q; ++a) Plane<S, EvenStAux>::store(A, g, opp(a), self, d[a]);
}

// The odd step's pushes land one element off the wave's alignment along x:
// ordinary (cached) stores let L2 merge the partial lines of neighbouring waves.
constexpr int OddStAux = 0;

template <typename S, typename T, bool Forced, int Route>
__global__ void __launch_bounds__(MaxThreads<T>::value)
aa_odd_kernel(S *__restrict__ A, Geom g, Relax<T> p, LaunchGrid L) {
    int x, y, z;
    locate(L, x, y, z);
    if (x >= g.nx || y >= g.ny) return;
    const uint32_t self = (uint32_t)x + (uint32_t)g.nx * (uint32_t)y + (uint32_t)g.nxy * (uint32_t)z;
    const bool edge = x == 0 || x == g.nx - 1 || y == 0 || y == g.ny - 1 || z == 0 || z == g.nz - 1;
    T d[Q];
#pragma unroll
    for (int a = 0; a < Q; ++a) d[a] = (T)Plane<S>::load(A, g, opp(a), pull_offset(g, a, self));
    if (edge) {
#pragma unroll
        for (int a = 1; a < Q; ++a) {
            int sx = x - cx(a), sy = y - cy(a), sz = z - cz(a);
            const bool in_lid = ghost_in_lid(g, sx, sy, sz);
            const bool ok = wrap(sx, g.nx, g.px) & wrap(sy, g.ny, g.py) & wrap(sz, g.nz, g.pz);
            if (ok)
                d[a] = (T)Plane<S>::load(A, g, opp(a), (uint32_t)(sx + g.nx * sy + g.nxy * sz));
            else
                d[a] = wall_value<T>((T)Plane<S>::load(A, g, a, self), p, a, in_lid);
        }
    }
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, self, p.step);
    if (!edge) {
#pragma unroll
        for (int a = 0; a < Q; ++a)
            Plane<S, OddStAux>::store(A, g, a, self + (uint32_t)(cx(a) + cy(a) * g.nx + cz(a) * g.nxy), d[a]);
        return;
    }
    Plane<S, 2>::store(A, g, 0, self, d[0]);
#pragma unroll
    for (int a = 1; a < Q; ++a) {
        int tx = x + cx(a), ty = y + cy(a), tz = z + cz(a);
        const bool in_lid = ghost_in_lid(g, tx, ty, tz);
        const bool ok = wrap(tx, g.nx, g.px) & wrap(ty, g.ny, g.py) & wrap(tz, g.nz, g.pz);
        if (ok)
            Plane<S, 2>::store(A, g, a, (uint32_t)(tx + g.nx * ty + g.nxy * tz), d[a]);
        else
            Plane<S, 2>::store(A, g, opp(a), self, wall_value<T>(d[a], p, opp(a), in_lid));
    }
}

// f0 (FP64, unpadded planes; NULL: the rest state) written as deviations
// into the natural slots, without a collision.
template <typename S>
__global__ void __launch_bounds__(256) store_plain_kernel(const double *__restrict__ f0, S *__restrict__ A, Geom g) {
    const int64_t N = (int64_t)g.nx * g.ny * g.nz;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    using T = typename StoreCompute<S>::T;
#pragma unroll
    for (int a = 0; a < Q; ++a)
        A[elem_i(g, a, i)] = Conv<S, T>::store(f0 ? (T)(f0[(int64_t)a * N + i] - weight(a)) : T(0));
}

// ---------------------------------------------------------------------------
// The same pair of steps on the row layout, in waves of 64 consecutive nodes
// with the full wall logic by address selects (FlatNode).
// ---------------------------------------------------------------------------
// Even step: the node's own 19 runs, collided, each value stored in the run
// of the opposite direction.
template <typename S, typename T, bool Forced, int Route, bool Far>
__global__ void __launch_bounds__(MaxThreads<T>::value)
aa_even_flat_kernel(S *__restrict__ A, Geom g, Relax<T> p, FlatGrid L) {
    const FlatLane<S, Far> k(g, L);
    if (k.i >= (uint32_t)g.n) return;
    const uint32_t run = (uint32_t)g.nx * (uint32_t)sizeof(S);
    const __amdgpu_buffer_rsrc_t own = row_rsrc(A + k.r0 * g.row, 0xFFFFFFFFu);
    T d[Q];
#pragma unroll
    for (int a = 0; a < Q; ++a) d[a] = (T)RawBits<S>::template load<0>(own, k.own, (uint32_t)a * run);
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, k.i, p.step);
#pragma unroll
    for (int a = 0; a < Q; ++a) RawBits<S>::template store<EvenStAux>(own, k.own, d[a], (uint32_t)opp(a) * run);
}

// Odd step.  Pull: f~_a(x - e_a) from run opp(a) of the source, or beyond a
// wall the node's own f~_opp(a), which the even step left in run a.  Push:
// f~_a(x) to run a of x + e_a, or beyond a wall, with the lid term of the
// opposite direction, into the node's own run opp(a).  The target of a is the
// source of b = opp(a), so the store of a goes to exactly the address that
// direction b was loaded from.
//
// Bound: HBM through the vector memory pipe: 1.06 and 1.03 times the bytes
// needed are read and written, waves stand ready but not issued 69% of their
// time with the VALU 42% busy.  250 x 240 x 230 FP32 418 us per step, 5.0 TB/s (510 with
// one wave per run of a row, the x faces apart and the y and z faces in a second
// launch with a wait per direction).
template <typename S, typename T, bool Forced, int Route, bool Far>
__global__ void __launch_bounds__(MaxThreads<T>::value)
aa_odd_flat_kernel(S *__restrict__ A, Geom g, Relax<T> p, FlatGrid L) {
    const FlatLane<S, Far> k(g, L);
    if (k.i >= (uint32_t)g.n) return;
    S *Aw = A + k.r0 * g.row;
    T d[Q];
    auto far = [&](const FlatNode<S, Far> &f, int a) {
        return (S *)((char *)Aw + k.own + f.wrapped(g, a) + (int64_t)opp(a) * f.run);
    };
    auto offset = [&](const FlatNode<S, Far> &f, int a) {
        return f.wall(a) ? f.self + (uint32_t)(a - opp(a)) * f.run : f.source(a);
    };
    {
        const FlatNode<S, Far> f(g, k.own, k.x, k.y, k.z);
        const __amdgpu_buffer_rsrc_t rsrc = f.rsrc(Aw);
#pragma unroll
        for (int a = 0; a < Q; ++a)
            d[a] = (T)RawBits<S>::template load<0>(rsrc, offset(f, a), (uint32_t)opp(a) * f.run);
        if (f.wave_touches_lid()) {
#pragma unroll
            for (int a = 1; a < Q; ++a) d[a] = wall_value<T>(d[a], p, a, f.lid(a));
        }
        if constexpr (Far) {
            if (g.pz && (f.lo[2] || f.hi[2])) {
#pragma unroll
                for (int a = 1; a < Q; ++a)
                    if (cz(a) != 0 && f.wraps(a)) d[a] = (T)Conv<S, T>::load(*far(f, a));
            }
        }
    }
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, k.i, p.step);
    // the addresses once more: kept over the collision they cost 20 registers
    // (84 instead of 64 VGPRs in FP32)
    uint32_t own = k.own;
    int x = k.x, y = k.y, z = k.z;
    asm volatile("" : "+v"(own), "+v"(x), "+v"(y), "+v"(z));
    const FlatNode<S, Far> f(g, own, x, y, z);
    const __amdgpu_buffer_rsrc_t rsrc = f.rsrc(Aw);
    if (f.wave_touches_lid()) {
#pragma unroll
        for (int a = 1; a < Q; ++a) d[a] = wall_value<T>(d[a], p, opp(a), f.lid(opp(a)));
    }
#pragma unroll
    for (int a = 0; a < Q; ++a) {
        const int b = opp(a);
        // (Far: a lane that wraps in z points beyond the descriptor's range, so the store is dropped)
        const uint32_t o = Far && f.wraps(b) ? 0x80000000u : offset(f, b);
        RawBits<S>::template store<OddStAux>(rsrc, o, d[a], (uint32_t)a * f.run);
    }
    if constexpr (Far) {
        if (g.pz && (f.lo[2] || f.hi[2])) {
#pragma unroll
            for (int a = 1; a < Q; ++a)
                if (cz(a) != 0 && f.wraps(opp(a))) *far(f, opp(a)) = Conv<S, T>::store(d[a]);
        }
    }
}

// The same steps for layers beyond the reach of 32-bit offsets, one thread per
// node at any width (with a workgroup per run of a row, the lanes beyond the row
// idle, 2^24 narrow rows need more than the 2^32 threads that a launch can have,
// and the runtime starts the remainder only, without an error).  us per step of ten layers: 20 x 395 000 FP32
// 2753 against 8275, 70 x 56 000 FP64 2322 against 8047, 2000 x 7 900 FP16 2154
// against 4697.
template <typename S, typename T, bool Forced, int Route>
__global__ void __launch_bounds__(MaxThreads<T>::value)
aa_even_wide_kernel(S *__restrict__ A, Geom g, Relax<T> p, FlatGrid L) {
    const FlatLane<S, true> k(g, L);
    if (k.i >= (uint32_t)g.n) return;
    S *own = A + WideNode<S>(g, k.x, k.y, k.z).own;
    T d[Q];
#pragma unroll
    for (int a = 0; a < Q; ++a) d[a] = (T)Conv<S, T>::load(own[(int64_t)a * g.nx]);
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, k.i, p.step);
#pragma unroll
    for (int a = 0; a < Q; ++a) own[(int64_t)opp(a) * g.nx] = Conv<S, T>::store(d[a]);
}

template <typename S, typename T, bool Forced, int Route>
__global__ void __launch_bounds__(MaxThreads<T>::value)
aa_odd_wide_kernel(S *__restrict__ A, Geom g, Relax<T> p, FlatGrid L) {
    const FlatLane<S, true> k(g, L);
    if (k.i >= (uint32_t)g.n) return;
    T d[Q];
    {
        const WideNode<S> w(g, k.x, k.y, k.z);
#pragma unroll
        for (int a = 0; a < Q; ++a) d[a] = (T)Conv<S, T>::load(A[w.at(a, opp(a))]);
        if (w.f.wave_touches_lid()) {
#pragma unroll
            for (int a = 1; a < Q; ++a) d[a] = wall_value<T>(d[a], p, a, w.f.lid(a));
        }
    }
    collide<T, Forced, Route, NewtonSteps<S>::value>(d, p, nullptr);
    round_state<S, T>(d, p, k.i, p.step);
    int x = k.x, y = k.y, z = k.z;      // the addresses once more, as in aa_odd_flat_kernel
    asm volatile("" : "+v"(x), "+v"(y), "+v"(z));
    const WideNode<S> w(g, x, y, z);
    if (w.f.wave_touches_lid()) {
#pragma unroll
        for (int a = 1; a < Q; ++a) d[a] = wall_value<T>(d[a], p, opp(a), w.f.lid(opp(a)));
    }
#pragma unroll
    for (int a = 0; a < Q; ++a) A[w.at(opp(a), a)] = Conv<S, T>::store(d[a]);
}

template <typename S, typename T, bool Forced, int Route, bool Far>
static hipError_t aa_pair_flat(void *A, const Geom &g, const Relax<T> &p, const FlatLaunch &L, int threads,
                               hipStream_t st) {
    Relax<T> q = p;             // the odd step is the next collision
    q.step = p.step + 1u;
    hipLaunchKernelGGL((aa_even_flat_kernel<S, T, Forced, Route, Far>), dim3(L.blocks), dim3(threads), 0, st, (S *)A, g,
                       p, L.grid);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((aa_odd_flat_kernel<S, T, Forced, Route, Far>), dim3(L.blocks), dim3(threads), 0, st, (S *)A, g,
                       q, L.grid);
    return hipGetLastError();
}

template <typename S, typename T, bool Forced, int Route>
static hipError_t aa_pair_f(void *A, const Geom &g, const Relax<T> &p, const StepLaunch &c, hipStream_t st) {
    if (g.rows) {
        const int threads = (c.bx * c.by + 63) / 64 * 64;
        const FlatLaunch F = flat_launch(g, sizeof(S), threads, c.xcd_remap);
        if (F.near) return aa_pair_flat<S, T, Forced, Route, false>(A, g, p, F, threads, st);
        if (F.far) return aa_pair_flat<S, T, Forced, Route, true>(A, g, p, F, threads, st);
        Relax<T> q = p;         // the odd step is the next collision
        q.step = p.step + 1u;
        hipLaunchKernelGGL((aa_even_wide_kernel<S, T, Forced, Route>), dim3(F.blocks), dim3(threads), 0, st, (S *)A, g, p,
                           F.grid);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((aa_odd_wide_kernel<S, T, Forced, Route>), dim3(F.blocks), dim3(threads), 0, st, (S *)A, g, q,
                           F.grid);
        return hipGetLastError();
    }
    LaunchGrid L;
    L.gx = (g.nx + c.bx - 1) / c.bx;
    L.gy = (g.ny + c.by - 1) / c.by;
    L.gz = g.nz;
    const uint32_t nb = (uint32_t)L.gx * L.gy * L.gz;
    L.aligned = nb & ~7u;
    L.remap = c.xcd_remap;
    dim3 grid(nb), block(c.bx, c.by);
    Relax<T> q = p;             // the odd step is the next collision
    q.step = p.step + 1u;
    hipLaunchKernelGGL((aa_even_kernel<S, T, Forced, Route>), grid, block, 0, st, (S *)A, g, p, L);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((aa_odd_kernel<S, T, Forced, Route>), grid, block, 0, st, (S *)A, g, q, L);
    return hipGetLastError();
}

template <typename S, typename T>
static hipError_t aa_pair_t(void *A, const Geom &g, const Relax<T> &p, bool forced, int route, const StepLaunch &c,
                            hipStream_t st) {
    if (route == 2) return forced ? hipErrorInvalidValue : aa_pair_f<S, T, false, 2>(A, g, p, c, st);
    if (route == 1) return forced ? aa_pair_f<S, T, true, 1>(A, g, p, c, st) : aa_pair_f<S, T, false, 1>(A, g, p, c, st);
    return forced ? aa_pair_f<S, T, true, 0>(A, g, p, c, st) : aa_pair_f<S, T, false, 0>(A, g, p, c, st);
}

hipError_t launch_aa_pair(int storage, void *A, const Geom &g, const Relax<double> &pd, const Relax<float> &pf,
                          bool forced, int route, const StepLaunch &c, hipStream_t st) {
    switch (storage) {
    case 0: return aa_pair_t<double, double>(A, g, pd, forced, route, c, st);
    case 1: return aa_pair_t<float, float>(A, g, pf, forced, route, c, st);
    default: return aa_pair_t<__half, float>(A, g, pf, forced, route, c, st);
    }
}

hipError_t launch_store_plain(int storage, const double *f0, void *A, const Geom &g, hipStream_t st) {
    const int64_t N = (int64_t)g.nx * g.ny * g.nz;
    dim3 grid((unsigned)((N + 255) / 256)), block(256);
    switch (storage) {
    case 0: hipLaunchKernelGGL(store_plain_kernel<double>, grid, block, 0, st, f0, (double *)A, g); break;
    case 1: hipLaunchKernelGGL(store_plain_kernel<float>, grid, block, 0, st, f0, (float *)A, g); break;
    default: hipLaunchKernelGGL(store_plain_kernel<__half>, grid, block, 0, st, f0, (__half *)A, g); break;
    }
    return hipGetLastError();
}

}  // namespace clbm
