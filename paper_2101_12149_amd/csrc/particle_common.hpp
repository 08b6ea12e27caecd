// Device helpers shared by the particle kernels: particle state, tiles and
// their LDS regions, guests and strays, the full-window deposit.
#pragma once

#include "pic_device.hpp"
#include "pic_types.hpp"

namespace pic {

template <typename T>
__device__ inline void gatomic_add(T *p, T v)
{
    unsafeAtomicAdd(p, v);
}

template <typename T>
__device__ inline void latomic_add(T *p, T v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ inline int wrap_once(int v, int n)
{
    return v < 0 ? v + n : (v >= n ? v - n : v);
}

__device__ inline int wrap_any(int v, int n)
{
    int r = v % n;
    return r < 0 ? r + n : r;
}

// momentum update of the push: Boris or Vay (uniform across the launch)
template <typename T>
__device__ inline void push_momentum(const PConst<T> &pc, const T *u, const T *E, const T *B, T *u1)
{
    if (pc.vay) {
        vay(pc.h, pc.inv_c2, u, E, B, u1);
    } else {
        BorisTape<T> tp;
        boris(pc.h, pc.inv_c2, u, E, B, u1, tp);
    }
}

template <typename T>
__device__ inline bool finite3(const T *u)
{
    return isfinite(u[0]) & isfinite(u[1]) & isfinite(u[2]);
}

// Load a particle and check its state; returns false (and flags err) for a
// cell outside [0,n), an offset outside [0,1) or a non-finite momentum.
// the state words of particle p, unchecked
template <typename T>
__device__ __attribute__((always_inline)) inline void load_state(const PArr<T> &in, int64_t p, int *c, T *f, T *u)
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        c[d] = in.cell[d][p];
        f[d] = in.off[d][p];
        u[d] = in.u[d][p];
    }
}

// true for a valid state (cell in the grid, offsets in [0,1), finite
// momentum); an invalid one sets bit 0 of the error word
template <typename T>
__device__ inline bool check_state(const int *n, const int *c, const T *f, const T *u, int *err)
{
    // no short-circuit branches: a branch between the loads of load_state
    // and their uses lets the compiler move later loads behind earlier checks
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        ok = ok & (c[d] >= 0) & (c[d] < n[d]) & (f[d] >= T(0)) & (f[d] < T(1));
    ok = ok & finite3(u);
    if (!ok)
        atomicOr(err, 1);
    return ok;
}

template <typename T>
__device__ inline bool load_particle(const PArr<T> &in, int64_t p, const int *n, int *c, T *f, T *u, int *err)
{
    load_state(in, p, c, f, u);
    return check_state(n, c, f, u, err);
}

template <typename T>
__device__ inline void copy_particle(const PArr<T> &in, const PArr<T> &out, int64_t p)
{
    if (in.cell[0] == out.cell[0])
        return;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        out.cell[d][p] = in.cell[d][p];
        out.off[d][p] = in.off[d][p];
        out.u[d][p] = in.u[d][p];
    }
    if (out.w)
        out.w[p] = in.w[p];
}

// ---------------------------------------------------------------------------
// tiles

template <typename T>
__device__ inline FieldSrc<T> global_fields(const FieldPtrs<T> &fp)
{
    FieldSrc<T> gf;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        gf.c[m] = fp.E[m];
        gf.c[3 + m] = fp.B[m];
    }
    return gf;
}

struct TileSpan {
    int t;       // logical tile index (x fastest)
    int t0[3];
    int64_t ps, pe;
};

__device__ inline TileSpan tile_span(const TileGeo &tg, const int *tile_start, int64_t N)
{
    const int ntiles = tg.nt[0] * tg.nt[1] * tg.nt[2];
    int t = blockIdx.x;
    if (tg.xcd_map)
        t = (t & 7) * (ntiles >> 3) + (t >> 3);
    TileSpan s;
    s.t = t;
    s.t0[0] = (t % tg.nt[0]) * tg.t[0];
    s.t0[1] = ((t / tg.nt[0]) % tg.nt[1]) * tg.t[1];
    s.t0[2] = (t / (tg.nt[0] * tg.nt[1])) * tg.t[2];
    int64_t ps = tile_start[t], pe = tile_start[t + 1];
    ps = ps < 0 ? 0 : (ps > N ? N : ps);
    pe = pe < ps ? ps : (pe > N ? N : pe);
    s.ps = ps;
    s.pe = pe;
    return s;
}

// cell position relative to the tile origin, periodic; true when inside
__device__ inline bool tile_local(const TileGeo &tg, const int *n, const int *t0, const int *c, int *l)
{
    bool inside = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        int v = c[d] - t0[d];
        v += v < -tg.slack ? n[d] : (v >= tg.t[d] + tg.slack ? -n[d] : 0);
        l[d] = v;
        inside = inside & (v >= -tg.slack) & (v < tg.t[d] + tg.slack);
    }
    return inside;
}

// logical tile of a cell, and the first cell of a tile
__device__ __attribute__((always_inline)) inline int cell_tile(const TileGeo &tg, const int *c)
{
    return c[0] / tg.t[0] + tg.nt[0] * (c[1] / tg.t[1] + tg.nt[1] * (c[2] / tg.t[2]));
}

__device__ __attribute__((always_inline)) inline void tile_origin(const TileGeo &tg, int t, int *t0)
{
    t0[0] = (t % tg.nt[0]) * tg.t[0];
    t0[1] = ((t / tg.nt[0]) % tg.nt[1]) * tg.t[1];
    t0[2] = (t / (tg.nt[0] * tg.nt[1])) * tg.t[2];
}

// Status of a moved particle for the next step: 0 if its new cell c1 is in
// its home tile's region (or no list slot is free, which leaves it to the
// stray kernel), 1 once it is listed as a guest of the tile holding c1.
__device__ __attribute__((always_inline)) inline unsigned char guest_next(const GuestArgs &g, const TileGeo &tg, const int *n, int64_t p, int home,
                                           const int *home_t0, const int *c1)
{
    int l[3];
    if (tile_local(tg, n, home_t0, c1, l) || p > 0x7fffffff)
        return 0;
    const int host = cell_tile(tg, c1);
    const int slot = atomicAdd(g.cnt_next + host, 1);
    if (slot >= g.cap)
        return 0;
    g.list_next[(int64_t)host * g.cap + slot] = make_int2((int)p, home);
    return 1;
}

// Walk of a tile region (ex x ey x ez cells from t0 - lo, x fastest, LDS row
// pitch px >= ex) by the whole workgroup without integer divisions in the
// loop: a thread keeps one x (its position in a group of LX lanes, LX the
// power of two >= ex) and steps over the rows (y, z) by blockDim.x / LX,
// carrying y into z.  region_cells: fn(x, y, z, global index) runs once per
// cell; region_walk: fn(local index, global index).
// With once, every axis of the region wraps at most once around the grid
// (see region_wraps_once), else each row takes the general wrap.
template <typename Fn>
__device__ __attribute__((always_inline)) inline void region_cells(const int *n, const int *t0, int lo, int ex,
                                                                    int ey, int ez, bool once, Fn &&fn)
{
    const int lb = ex > 1 ? 32 - __clz(ex - 1) : 0;
    const int x = (int)threadIdx.x & ((1 << lb) - 1);
    const int step = (int)blockDim.x >> lb;   // >= 1: regions are at most 64 cells wide
    if (x >= ex || step == 0)
        return;
    int row = (int)threadIdx.x >> lb;
    int y = row % ey, z = row / ey;
    const int sy = step % ey, sz = step / ey;
    const int gx = wrap_any(t0[0] - lo + x, n[0]);
    const int nrow = ey * ez;
    for (; row < nrow; row += step) {
        const int vy = t0[1] - lo + y, vz = t0[2] - lo + z;
        const int gy = once ? wrap_once(vy, n[1]) : wrap_any(vy, n[1]);
        const int gz = once ? wrap_once(vz, n[2]) : wrap_any(vz, n[2]);
        fn(x, y, z, gx + n[0] * (gy + n[1] * gz));
        y += sy;
        z += sz;
        if (y >= ey) {
            y -= ey;
            ++z;
        }
    }
}

template <typename Fn>
__device__ __attribute__((always_inline)) inline void region_walk(const int *n, const int *t0, int lo, int ex,
                                                                   int ey, int ez, int px, bool once, Fn &&fn)
{
    region_cells(n, t0, lo, ex, ey, ez, once, [&](int x, int y, int z, int gi) { fn(x + px * (y + ey * z), gi); });
}

// A tile region's values of NV fields copied by the whole workgroup:
// load(global index, v) reads them, store(x, y, z, v) puts them down.  R rows
// per thread are requested before the first is stored, with no branch between
// the loads (a lane or row past the region reads its last value and stores
// nothing): a branch there makes a wave wait out the memory latency at each
// row, with the values in scratch.
template <int R, int NV, typename V, typename LoadFn, typename StoreFn>
__device__ __attribute__((always_inline)) inline void region_stage(const int *n, const int *t0, int lo, int ex,
                                                                    int ey, int ez, bool once, LoadFn &&load,
                                                                    StoreFn &&store)
{
    if (once) {
        const int lb = ex > 1 ? 32 - __clz(ex - 1) : 0;
        const int x = (int)threadIdx.x & ((1 << lb) - 1), step = (int)blockDim.x >> lb;
        const int gx = wrap_once(t0[0] - lo + (x < ex ? x : ex - 1), n[0]);
        int y = ((int)threadIdx.x >> lb) % ey, z = ((int)threadIdx.x >> lb) / ey;
        const int sy = step % ey, sz = step / ey;
        for (int r = 0; r < ey * ez; r += R * step) {
            V v[R][NV];
            int ay[R], az[R];
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const int gy = wrap_once(t0[1] - lo + y, n[1]);
                const int gz = wrap_once(t0[2] - lo + (z < ez ? z : ez - 1), n[2]);
                load(gx + n[0] * (gy + n[1] * gz), v[t]);
                ay[t] = y;
                az[t] = z;
                y += sy;
                z += sz;
                const bool over = y >= ey;
                y -= over ? ey : 0;
                z += over ? 1 : 0;
            }
#pragma unroll
            for (int t = 0; t < R; ++t)
                if (x < ex && az[t] < ez)
                    store(x, ay[t], az[t], v[t]);
        }
    } else {
        region_cells(n, t0, lo, ex, ey, ez, false, [&](int x, int y, int z, int gi) {
            V v[NV];
            load(gi, v);
            store(x, y, z, v);
        });
    }
}

// true when the region of extents e starting lo cells below a tile of
// extents t wraps each axis of the grid at most once (wrap_once suffices)
__device__ inline bool region_wraps_once(const int *n, const int *t, int lo, const int *e)
{
    bool ok = true;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        ok = ok && lo <= n[d] && e[d] - t[d] - lo <= n[d];
    return ok;
}

// E and B of a tile's field region into LDS: component m of (x, y, z) at
// sF[m * pm + x + py * y + pz * z].  R rows per thread at a time (first-order
// regions have hardly more rows than a workgroup takes at once).
template <int R, typename T>
__device__ __attribute__((always_inline)) inline void stage_fields(const FieldPtrs<T> &fp, const int *n,
                                                                    const TileGeo &tg, const int *t0, T *sF, int pm,
                                                                    int py, int pz)
{
    region_stage<R, 6, T>(
        n, t0, tg.lo_f, tg.rf[0], tg.rf[1], tg.rf[2], region_wraps_once(n, tg.t, tg.lo_f, tg.rf),
        [&](int gi, T *v) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                v[m] = fp.E[m][gi];
                v[3 + m] = fp.B[m][gi];
            }
        },
        [&](int x, int y, int z, const T *v) {
            T *s = sF + x + py * y + pz * z;
#pragma unroll
            for (int m = 0; m < 6; ++m)
                s[m * pm] = v[m];
        });
}

// An index into rows of 16 values, the halves of every second row exchanged:
// sixteen lanes that add to eight cells of two neighbouring rows then fall on
// all the LDS banks, as they would not at any pitch below 24.  fold is LDS_FOLD,
// or 0 for rows of another pitch.
constexpr int LDS_FOLD = 8;

__device__ inline int lds_fold(int i, int fold)
{
    return i ^ ((i >> 1) & fold);
}

// A list of strays on the device, appended to by the tile kernels (one
// atomic per wave) and worked through by the stray kernels; cnt is cleared
// before the tile kernel runs.  cap >= the particle count.
struct StrayList {
    int *p;
    int *cnt;
    int cap;
};

// appends p for every lane with `want`; call with the whole wave converged
__device__ inline void stray_append(bool want, int p, const StrayList &sl)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long m = __ballot(want);
    if (m == 0)
        return;   // uniform across the wave
    const int leader = __ffsll((long long)m) - 1;
    int base = 0;
    if (lane == leader)
        base = atomicAdd(sl.cnt, __popcll(m));
    base = __shfl(base, leader);
    if (want) {
        const int i = base + __popcll(m & ((1ull << lane) - 1ull));
        if (i < sl.cap)
            sl.p[i] = p;
    }
}

// Esirkepov full-window current of component M into the component's LDS
// accumulator
template <typename T, int O, int M>
__device__ __attribute__((always_inline)) inline void deposit_local_comp(const PConst<T> &pc, const T *f0, const T *f1,
                                                                         const int *kap, const int *l, int lo_j,
                                                                         const int *sj, T w, double *sA)
{
    constexpr int NW = Shape<O, T>::NW;
    EskAxis<O, T> e[3];
    T K[3];
    int jo[3][NW + 1];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        esk_axis<O>(f0[d], f1[d], kap[d], e[d]);
        K[d] = pc.jk[d] * w;
        axis_offsets_local<NW + 1>(l[d] + lo_j, e[d].lo, sj[d], jo[d]);
    }
    const int *const jx[2] = {jo[0], jo[0]};
    esk_scatter<O, T, double, M>(e, jo, jx, K, [&](int, int idx, double v) { latomic_add(sA + idx, v); });
}

// Esirkepov full-window current straight into global memory (a crosser
// that found the queue full)
template <typename T, int O>
__device__ __attribute__((always_inline)) inline void deposit_global_full(const PConst<T> &pc, const FieldPtrs<T> &fp,
                                                                          const int *c, const T *f0, const T *f1,
                                                                          const int *kap, T w)
{
    constexpr int NW = Shape<O, T>::NW;
    const int gs[3] = {1, pc.n[0], pc.n[0] * pc.n[1]};
    EskAxis<O, T> e[3];
    T K[3];
    int jo[3][NW + 1];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        esk_axis<O>(f0[d], f1[d], kap[d], e[d]);
        K[d] = pc.jk[d] * w;
        axis_offsets_global<NW + 1>(c[d], e[d].lo, pc.n[d], gs[d], jo[d]);
    }
    const int *const jx[2] = {jo[0], jo[0]};
    esk_scatter<O, T, T>(e, jo, jx, K, [&](int m, int idx, T v) { gatomic_add(fp.J[m] + idx, v); });
}

}  // namespace pic
