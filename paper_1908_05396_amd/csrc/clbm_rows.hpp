// Row layout helpers shared by the single-lattice, in-place, flagged and batch kernels.
//
// Row layout: the 19 populations of lattice row r = y + ny z are 19
// consecutive runs of nx values, population a of node x at element
// (19 r + a) nx + x (Geom::plane = nx, Geom::row = 19 nx).  A row kernel
// runs waves of 64 consecutive x of one row (blockDim.x a multiple of 64),
// so every direction's source or target run has a uniform (scalar) base and
// one lane offset serves all of them.
#pragma once

#include "clbm_internal.hpp"

namespace clbm {

__device__ inline __amdgpu_buffer_rsrc_t row_rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, kBufferFlags);
}

// The work of a launch is a list of wave items, (row, run of 64 x) in x-fastest
// order; workgroup b takes the items b W .. b W + W - 1 of its W waves, so a
// lattice of any width fills whole workgroups and the runs of a row, which
// share cache lines where they meet, stay together.
struct RowGrid {
    uint32_t gx;            // runs of 64 x per row
    uint32_t rows;          // rows handled by the launch
    uint32_t aligned;       // largest multiple of 8 <= number of workgroups
    int32_t remap;          // XCD-contiguous workgroup order
};

// Column of the lane and row index of the wave.
__device__ inline bool row_of(const RowGrid &R, int &x, uint32_t &ri) {
    uint32_t b = blockIdx.x;
    if (R.remap && b < R.aligned) b = (b & 7u) * (R.aligned >> 3) + (b >> 3);
    const uint32_t item = __builtin_amdgcn_readfirstlane(b * (blockDim.x >> 6) + (threadIdx.x >> 6));
    ri = item / R.gx;
    x = (int)((item - ri * R.gx) * 64u + (threadIdx.x & 63u));
    return ri < R.rows;
}

// Quotient of a 32-bit value below 2^31 by a divisor fixed at launch, by one
// high multiplication: with s = ceil(log2 d) and m = ceil(2^(31 + s) / d) <
// 2^32, floor(m i / 2^(31 + s)) = floor(i / d) for i < 2^31 (the excess of m,
// below d, adds less than i / 2^(31 + s) <= 1 / d to the quotient).
struct Divisor {
    uint32_t m, s;
    static Divisor make(uint32_t d) {
        uint32_t s = 0;
        while ((1ull << s) < d) ++s;
        return {(uint32_t)(((1ull << (31 + s)) + d - 1) / d), s};
    }
    __device__ uint32_t quotient(uint32_t i) const { return (uint32_t)(((uint64_t)m * i) >> 31 >> s); }
};

struct FlatGrid {
    Divisor by_nx, by_ny;
    uint32_t aligned;       // largest multiple of 8 <= number of workgroups
    int32_t remap;          // XCD-contiguous workgroup order
};

// Workgroups of `threads` threads (a multiple of 64) over every row of the lattice.
inline uint32_t all_rows(const Geom &g, int threads, int remap, RowGrid &R) {
    R.gx = ((uint32_t)g.nx + 63u) / 64u;
    R.rows = (uint32_t)g.ny * (uint32_t)g.nz;
    R.remap = remap;
    const uint32_t waves = (uint32_t)threads / 64u;
    const uint32_t blocks = (uint32_t)(((uint64_t)R.gx * R.rows + waves - 1) / waves);
    R.aligned = blocks & ~7u;
    return blocks;
}

// Row kernels group the x-face bounce-back loads of a wave (row_gather's
// XGroup) with FP32 storage: at 512^3 the one-step launch runs 1.3% and the
// two-step one 2.9% faster.  FP16 storage, bound by its arithmetic, ran 3%
// slower that way and keeps the per-direction path.
template <typename S> struct XGroupRows { static constexpr bool value = std::is_same<S, float>::value; };

// Pull of node x of row (y, z) with the wall rules into d; y and z uniform
// over the wave; Face: the row may lie on a y or z face; XGroup: the x-face
// bounce-back loads of a wave issued together (below).
//
// Nine source rows (one per e_y, e_z), each with a descriptor whose base lies
// one value before the row group; direction a's run at the scalar offset
// a nx.  The lane offset selects x - cx(a) + 1, wrapped on a periodic x axis;
// it is shared by the directions of one cx.
template <typename S, typename T, int LdAux, bool Face, bool XGroup = false>
__device__ inline void row_gather(const S *__restrict__ A, const Geom &g, const Relax<T> &p, int x, int y, int z,
                                  T (&d)[Q]) {
    constexpr uint32_t es = sizeof(S);
    // On a non-periodic x face the source column x - cx(a) = -1 or nx is a
    // ghost, whose value the x-face rule below supplies: those lanes take an
    // offset beyond every descriptor's range, so the load returns 0 without
    // touching memory (and the cache line past the run is not fetched for
    // them).  (the lengths pass through readfirstlane so that the compiler
    // keeps them in scalar registers; run offsets stay below 2^31 bytes)
    const uint32_t run = __builtin_amdgcn_readfirstlane((uint32_t)g.nx * es);
    const uint32_t range = (uint32_t)(Q * run) + 2 * es;
    constexpr uint32_t outside = 0x80000000u;
    const uint32_t o0 = (uint32_t)(x + 1) * es;
    const uint32_t op = x == 0 ? (g.px ? run : outside) : (uint32_t)x * es;                  // cx = +1
    const uint32_t om = x == g.nx - 1 ? (g.px ? es : outside) : (uint32_t)(x + 2) * es;      // cx = -1
    auto lane_off = [&](int a) { return cx(a) == 1 ? op : (cx(a) == -1 ? om : o0); };
    const int64_t row = g.row, layer = (int64_t)g.ny * g.row;
    const S *own = A + ((int64_t)z * layer + (int64_t)y * row) - 1;
    // source ghosts beyond the y and z walls (index c + 1 for c = -1, 0, +1)
    const int ylo = y == 0, yhi = y == g.ny - 1, zlo = z == 0, zhi = z == g.nz - 1;
    const int gy[3] = {yhi & (g.py ^ 1), 0, ylo & (g.py ^ 1)};
    const int gz[3] = {zhi & (g.pz ^ 1), 0, zlo & (g.pz ^ 1)};
    auto row_wall = [&](int a) { return Face && ((gy[cy(a) + 1] | gz[cz(a) + 1]) != 0); };
    if constexpr (!Face) {
#pragma unroll
        for (int a = 0; a < Q; ++a)
            d[a] = (T)RawBits<S>::template load<LdAux>(row_rsrc(own - cy(a) * row - cz(a) * layer, range), lane_off(a),
                                                       (uint32_t)a * run);
    } else {
        // per direction (uniformly) the source row is inside, wrapped on a
        // periodic axis, or a ghost: half-way bounce-back returns the node's
        // own population opposite to a, plus the moving-wall term for a ghost
        // in the lid plane.  Which run is read is a scalar select, so the 19
        // loads go out together and the wave waits for memory once; the lid
        // terms are added afterwards.
        const int64_t dy[3] = {yhi ? row - layer : row, 0, ylo ? layer - row : -row};
        const int64_t lattice = (int64_t)g.nz * layer;
        const int64_t dz[3] = {zhi ? layer - lattice : layer, 0, zlo ? lattice - layer : -layer};
#pragma unroll
        for (int a = 0; a < Q; ++a) {
            const bool wall = row_wall(a);
            const S *src = own + (wall ? 0 : dy[cy(a) + 1] + dz[cz(a) + 1]);
            const uint32_t o = cx(a) == 0 ? o0 : (wall ? o0 : lane_off(a));
            d[a] = (T)RawBits<S>::template load<LdAux>(row_rsrc(src, range), o, (uint32_t)(wall ? opp(a) : a) * run);
            // (each direction's scalars end with its load: all of them together
            // would not fit the scalar registers)
            __builtin_amdgcn_sched_barrier(0);
        }
        // the lid is one face, so a ghost lies in its plane through one axis
        const int m = g.lid_mask;
        auto lid_y = [&](int c) {
#pragma unroll
            for (int a = 1; a < Q; ++a)
                if (cy(a) == c) d[a] = wall_value<T>(d[a], p, a, true);
        };
        auto lid_z = [&](int c) {
#pragma unroll
            for (int a = 1; a < Q; ++a)
                if (cz(a) == c) d[a] = wall_value<T>(d[a], p, a, true);
        };
        if ((m & 4) && ylo) lid_y(1);
        if ((m & 8) && yhi) lid_y(-1);
        if ((m & 16) && zlo) lid_z(1);
        if ((m & 32) && zhi) lid_z(-1);
        if (m & 3) {
            // lid on an x face: its lanes' ghosts beyond a y or z wall lie in its plane too
#pragma unroll
            for (int a = 1; a < Q; ++a) {
                if (cx(a) == 0) continue;
                const bool in_lid = row_wall(a) && (cx(a) == 1 ? (m & 1) && x == 0 : (m & 2) && x == g.nx - 1);
                d[a] = wall_value<T>(d[a], p, a, in_lid);
            }
        }
    }
    // lanes on a non-periodic x face: directions whose source row is inside
    // the lattice but whose source column is a ghost take the bounce-back of
    // the node's own opposite population (those whose source row is a ghost
    // have bounced back above, with the lid term of every ghost coordinate).
    // XGroup: the wave issues these loads all together, the lanes without such
    // a ghost taking an out-of-range offset, i.e. no memory access, and selects
    // the wall values afterwards, so that it waits for memory once instead of
    // once per direction.
    if (g.px) return;
    const bool lo = x == 0, hi = x == g.nx - 1;
    const __amdgpu_buffer_rsrc_t own_rsrc = row_rsrc(own, range);
    auto bounce = [&](int a, uint32_t o) {
        return (T)RawBits<S>::template load<LdAux>(own_rsrc, o, (uint32_t)opp(a) * run);
    };
    if constexpr (!XGroup) {
        if (lo || hi) {
#pragma unroll
            for (int a = 1; a < Q; ++a) {
                if (cx(a) == 0 || !(cx(a) == 1 ? lo : hi) || row_wall(a)) continue;
                d[a] = wall_value<T>(bounce(a, o0), p, a, (g.lid_mask & (cx(a) == 1 ? 1 : 2)) != 0);
            }
        }
    } else if (__builtin_amdgcn_ballot_w64(lo || hi) != 0) {       // uniform over the wave
        const uint32_t ol = lo ? o0 : outside, oh = hi ? o0 : outside;
        T o[Q];
#pragma unroll
        for (int a = 1; a < Q; ++a)
            if (cx(a) != 0) o[a] = bounce(a, cx(a) == 1 ? ol : oh);
#pragma unroll
        for (int a = 1; a < Q; ++a) {
            if (cx(a) == 0) continue;
            const bool ghost = (cx(a) == 1 ? lo : hi) && !row_wall(a);
            const T w = wall_value<T>(o[a], p, a, (g.lid_mask & (cx(a) == 1 ? 1 : 2)) != 0);
            d[a] = ghost ? w : d[a];
        }
    }
}

// Store of the 19 populations at lane byte offset `lane` of `out`, the run of
// direction a at the scalar offset a * run.  FP16 with stochastic rounding (sr):
// rounded in the store itself with the seeds of round_state (sr_base =
// sr_base(node, step)).
template <typename S, typename T, int StAux>
__device__ __forceinline__ void row_store_at(__amdgpu_buffer_rsrc_t out, uint32_t lane, uint32_t run, const T (&d)[Q], bool sr,
                                    uint32_t seed_base) {
    if constexpr (std::is_same<S, __half>::value) {
        if (sr) {
            // each conversion keeps the high half of its first operand: the
            // previous direction's result (stored already) serves, so no
            // register is cleared per value; the stored low halves are those
            // of sr_to_f16_bits
            typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
            half2_t h = __builtin_bit_cast(half2_t, (float)d[0]);
#pragma unroll
            for (int a = 0; a < Q; ++a) {
                h = __builtin_amdgcn_cvt_sr_f16_f32(h, (float)d[a], seed_base + (uint32_t)a * kWeyl, false);
                __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, h[0]), out, (int)lane,
                                                      (int)((uint32_t)a * run), StAux);
            }
            return;
        }
    }
#pragma unroll
    for (int a = 0; a < Q; ++a) RawBits<S>::template store<StAux>(out, lane, d[a], (uint32_t)a * run);
}

// Store at node x of row (y, z) (y, z uniform).
template <typename S, typename T, int StAux>
__device__ inline void row_store(S *__restrict__ B, const Geom &g, int x, int y, int z, const T (&d)[Q],
                                 bool sr = false, uint32_t seed_base = 0) {
    constexpr uint32_t es = sizeof(S);
    const uint32_t run = __builtin_amdgcn_readfirstlane((uint32_t)g.nx * es);
    const __amdgpu_buffer_rsrc_t out =
        row_rsrc(B + ((int64_t)z * g.ny + y) * g.row, (uint32_t)Q * run);
    row_store_at<S, T, StAux>(out, (uint32_t)x * es, run, d, sr, seed_base);
}

// ---------------------------------------------------------------------------
// Waves of 64 consecutive nodes (x fastest, across rows and layers): each lane
// addresses its sources with the full wall logic (Eq. cascaded streaming with
// the rules of Sec. 4): periodic wrap, half-way bounce-back, moving lid.
// Which value a direction reads - the source's, or the node's own beyond a
// wall - is a select on its address, so the 19 loads go out together and the
// wave waits for memory once; the lid terms are added afterwards, in waves that
// touch the lid.
//
// `own` is the byte offset of the node's own row group plus its x from the
// base that the loads use, and every source lies within 32 bits of it: loads
// go through one descriptor that starts K = layer + row + one value before that
// base (no access falls before it), which keeps the lane offsets positive.
// Far: the lattice itself is larger; the base is the layer of the wave's first
// node, and lanes that pull across a periodic z face address in 64 bits.
//
// Waves without a face node could use one lane offset and 19 scalar ones.
// Their loads then issue back to back, which the memory serves worse than
// loads a few instructions apart: 200 x 190 x 220 FP32 304 us per step with
// that path against 250 without, 256^3 FP16 233 against 227; not kept.
// ---------------------------------------------------------------------------
template <typename S, bool Far> struct FlatNode {
    uint32_t run, layer, self;          // bytes; self: own + K
    uint32_t xm, xp, ym, yp, zm, zp;    // byte distance to the (wrapped) source for c = -1 (m) and +1 (p)
    bool lo[3], hi[3], per[3];          // on the low and high face of an axis; periodic
    int lid_mask;

    __device__ __forceinline__ FlatNode(const Geom &g, uint32_t own, int x, int y, int z) {
        constexpr uint32_t es = sizeof(S);
        run = (uint32_t)g.nx * es;
        const uint32_t row = Q * run;
        layer = row * (uint32_t)g.ny;
        self = own + lead();
        lo[0] = x == 0; lo[1] = y == 0; lo[2] = z == 0;
        hi[0] = x == g.nx - 1; hi[1] = y == g.ny - 1; hi[2] = z == g.nz - 1;
        per[0] = g.px != 0; per[1] = g.py != 0; per[2] = g.pz != 0;
        lid_mask = g.lid_mask;
        // (Far: lanes wrapping in z point at their own layer)
        const uint32_t wrap = Far ? layer : layer * (uint32_t)g.nz;
        xm = hi[0] ? es - run : es;
        xp = lo[0] ? run - es : 0u - es;
        ym = hi[1] ? row - layer : row;
        yp = lo[1] ? layer - row : 0u - row;
        zm = hi[2] ? layer - wrap : layer;
        zp = lo[2] ? wrap - layer : 0u - layer;
    }
    __device__ uint32_t lead() const { return layer + Q * run + (uint32_t)sizeof(S); }
    __device__ __amdgpu_buffer_rsrc_t rsrc(const S *base) const { 
        // (Far: offsets stay below 2^31, so that 0x80000000 lies outside whether or not scalar offsets count)
        return row_rsrc((const char *)base - lead(), Far ? 0x80000000u : 0xFFFFFFFFu);
    }
    __device__ bool ghost(int axis, int c) const { return c != 0 && !per[axis] && (c == 1 ? lo[axis] : hi[axis]); }
    __device__ bool wall(int a) const { return ghost(0, cx(a)) | ghost(1, cy(a)) | ghost(2, cz(a)); }
    // lane offset of the source of direction a (run 0 of its row group)
    __device__ uint32_t source(int a) const { return self + dxy(a) + (cz(a) == 0 ? 0u : cz(a) == 1 ? zp : zm); }
    __device__ uint32_t dxy(int a) const {
        return (cx(a) == 0 ? 0u : cx(a) == 1 ? xp : xm) + (cy(a) == 0 ? 0u : cy(a) == 1 ? yp : ym);
    }
    // the source of direction a is a ghost in the lid plane (edges and corners of it included)
    __device__ bool lid(int axis, int c) const {
        return c != 0 && (c == 1 ? ((lid_mask >> (2 * axis)) & 1) && lo[axis]
                                 : ((lid_mask >> (2 * axis + 1)) & 1) && hi[axis]);
    }
    __device__ bool lid(int a) const { return lid(0, cx(a)) | lid(1, cy(a)) | lid(2, cz(a)); }
    __device__ bool wave_touches_lid() const {
        const bool any = lid(0, 1) | lid(0, -1) | lid(1, 1) | lid(1, -1) | lid(2, 1) | lid(2, -1);
        return __builtin_amdgcn_ballot_w64(any) != 0;
    }
    // Far: direction a's source lies across a periodic z face, at this byte
    // distance from the node's own row group
    __device__ bool wraps(int a) const { return Far && per[2] && cz(a) != 0 && (cz(a) == 1 ? lo[2] : hi[2]) && !wall(a); }
    __device__ int64_t wrapped(const Geom &g, int a) const {
        return (int64_t)(int32_t)dxy(a) + cz(a) * (int64_t)(g.nz - 1) * (int64_t)layer;
    }
};

template <typename S, typename T, int LdAux, bool Far>
__device__ __forceinline__ void gather_flat(const S *__restrict__ A, uint32_t own, const Geom &g, const Relax<T> &p,
                                            int x, int y, int z, T (&d)[Q]) {
    const FlatNode<S, Far> f(g, own, x, y, z);
    const __amdgpu_buffer_rsrc_t rsrc = f.rsrc(A);
#pragma unroll
    for (int a = 0; a < Q; ++a) {
        d[a] = (T)RawBits<S>::template load<LdAux>(
            rsrc, f.wall(a) ? f.self + (uint32_t)(opp(a) - a) * f.run : f.source(a), (uint32_t)a * f.run);
        // (each lane address next to its load: the scheduler would otherwise
        // collect the loads into bursts; the 64-cavity batch runs 638 against
        // 650 us per step in FP32, 397 against 409 in FP16)
        __builtin_amdgcn_sched_barrier(0x4);    // scalar arithmetic may cross
    }
    if (f.wave_touches_lid()) {
#pragma unroll
        for (int a = 1; a < Q; ++a) d[a] = wall_value<T>(d[a], p, a, f.lid(a));
    }
    if constexpr (Far) {
        if (g.pz && (f.lo[2] || f.hi[2])) {
#pragma unroll
            for (int a = 1; a < Q; ++a)
                if (cz(a) != 0 && f.wraps(a))
                    d[a] = (T)Conv<S, T>::load(
                        *(const S *)((const char *)A + own + f.wrapped(g, a) + (int64_t)a * f.run));
        }
    }
}

// Workgroups over the nodes of a lattice, and whether 32-bit offsets reach
// the whole of it (near) or the layers of a wave's nodes and their sources
// (far).
struct FlatLaunch {
    FlatGrid grid;
    uint32_t blocks;
    bool near, far;
};

inline FlatLaunch flat_launch(const Geom &g, uint64_t value_bytes, int threads, int remap) {
    FlatLaunch L;
    const uint64_t row = (uint64_t)Q * value_bytes * (uint64_t)g.nx, layer = row * (uint64_t)g.ny;
    L.near = layer * (uint64_t)g.nz + layer + 2 * row < 0xFFFFFF00ull;
    L.far = layer * (uint64_t)(64 / g.nxy + 5) + 2 * row < 0x80000000ull;
    L.blocks = (uint32_t)(((int64_t)g.n + threads - 1) / threads);
    L.grid.by_nx = Divisor::make((uint32_t)g.nx);
    L.grid.by_ny = Divisor::make((uint32_t)g.ny);
    L.grid.aligned = L.blocks & ~7u;
    L.grid.remap = remap;
    return L;
}

// The lane's node of a flat launch: its coordinates, the first row of the
// base that 32-bit offsets count from (0, or Far: of the layer of the wave's
// first node) and its own offset from there.
template <typename S, bool Far> struct FlatLane {
    uint32_t i, own;
    int64_t r0;
    int x, y, z;
    __device__ __forceinline__ FlatLane(const Geom &g, const FlatGrid &L) {
        uint32_t b = blockIdx.x;
        if (L.remap && b < L.aligned) b = (b & 7u) * (L.aligned >> 3) + (b >> 3);
        i = b * blockDim.x + threadIdx.x;
        if (i >= (uint32_t)g.n) return;
        const uint32_t r = L.by_nx.quotient(i), zr = L.by_ny.quotient(r);
        x = (int)(i - r * (uint32_t)g.nx);
        y = (int)(r - zr * (uint32_t)g.ny);
        z = (int)zr;
        const uint32_t first = Far ? __builtin_amdgcn_readfirstlane(zr) * (uint32_t)g.ny : 0u;
        r0 = first;
        own = (r - first) * (Q * (uint32_t)g.nx * (uint32_t)sizeof(S)) + (uint32_t)x * (uint32_t)sizeof(S);
    }
};

// Layers beyond the reach of 32-bit offsets (430 MB and more): the same selects
// on 64-bit element offsets from the start of the state.
template <typename S> struct WideNode {
    FlatNode<S, true> f;                    // faces, walls and lid
    int64_t run, own, xm, xp, ym, yp, zm, zp;   // elements
    __device__ __forceinline__ WideNode(const Geom &g, int x, int y, int z) : f(g, 0u, x, y, z) {
        run = g.nx;
        const int64_t row = g.row, layer = row * g.ny, lattice = layer * g.nz;
        own = z * layer + y * row + x;
        xm = f.hi[0] ? 1 - run : 1;
        xp = f.lo[0] ? run - 1 : -1;
        ym = f.hi[1] ? row - layer : row;
        yp = f.lo[1] ? layer - row : -row;
        zm = f.hi[2] ? layer - lattice : layer;
        zp = f.lo[2] ? lattice - layer : -layer;
    }
    // run `slot` of the source of direction a; beyond a wall the node's own run of the opposite direction
    __device__ __forceinline__ int64_t at(int a, int slot) const {
        const int64_t d = (cx(a) == 0 ? 0 : cx(a) == 1 ? xp : xm) + (cy(a) == 0 ? 0 : cy(a) == 1 ? yp : ym) +
                          (cz(a) == 0 ? 0 : cz(a) == 1 ? zp : zm);
        return own + (f.wall(a) ? opp(slot) * run : d + slot * run);
    }
};

}  // namespace clbm
