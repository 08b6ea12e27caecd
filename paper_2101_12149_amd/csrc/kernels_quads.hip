// The FP32 third-order tile step on the matrix cores.
//
// The gather of a particle is a contraction of a 4-wide (5-wide on a
// staggered axis) window of six field components with weights along three
// axes, and its deposit an outer product of the same shape.  Particles of
// one cell share the window, so a group of up to four of them (a quad: four
// consecutive lanes) forms one 4x4 block of v_mfma_f32_4x4x1_16b, whose 16
// blocks hold 16 quads:
//
//  gather   columns: the quad's particles; rows: four window nodes along one
//           nodal axis; the matrix core sums over the taps of a second axis.
//           A lane reads one row of the window for the whole quad, so a
//           wave reads 135 values per lane from LDS instead of 384, at
//           fixed positions relative to the cell (a staggered axis takes the
//           five nodes either half of the cell reaches, with a zero weight
//           on one), which a row pitch of 8 or 24 modulo 32 words spreads
//           over all banks.  Every lane then holds its own particle's four
//           rows and sums the remaining two axes with its own weights.
//  deposit  rows: the running sums P along the component's axis; columns:
//           four nodes along a second axis; one instruction per particle and
//           node of the third.  A quad's lanes evaluate one node's weights
//           each for the particle in turn.
//
// Particles are grouped by cell with a counting sort in LDS.  A particle
// that changes cells deposits the full window after the loop.
//
// Against one thread per particle (k_particles_tile; k_particles_cells from 6
// per cell on), particle kernels per step: 256^3, 8 per cell 15.1 -> 12.5 ms;
// 128 x 128 x 1024 laser box, 2 per cell, with a laser pulse 6.4 -> 4.9 ms;
// 512^3, 2 per cell, hot 60 -> 43 ms; 128^3 in 4^3 tiles, 2 per cell 3.1 ->
// 1.1 ms.  What is left is latency: at 256^3 (one workgroup of 16 waves on a
// CU) the vector units are busy 58 % of the time, the LDS 52 %, the matrix cores
// 12 %, in the laser box (two workgroups of 8) 69, 46 and 14 %; HBM is at 1.8
// TB/s and 1.4 TB/s.
#include <type_traits>

#include "particle_common.hpp"

namespace pic {

typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int QD_THREADS = 1024;   // threads of a workgroup, at most
constexpr int QD_WAVES = QD_THREADS / 64;
constexpr int QD_SLOTS = 4;        // cells (with the slack's) per thread, at most
constexpr int QD_BATCH = 5;        // sparse tiles: batches of sixteen groups per wave and round
constexpr int QD_MIN_ROUND = 256;  // particles of a round, at least
constexpr int QD_RESTAGE = 4096;   // cells that a tile of several rounds stages in all, at most
constexpr int QD_CELLS = 640;      // cells of a tile, at most
constexpr int QD_CUS = 256;        // compute units: so many tiles or fewer have one each
constexpr int QD_STAGE = 4;        // rows of the field staging in flight together

// Row pitches (in words) that spread a quad's columns over the LDS banks:
// eight cells along x times four rows (or planes) fall on 32 banks.
__host__ __device__ inline int bank_pitch(int n)
{
    int p = (n + 7) / 8 * 8;
    return (p & 15) == 8 ? p : p + 8;
}

// LDS layouts of k_particles_quads, shared by the launcher.  The six field
// components interleaved by row; the three FP64 current components; the cell
// counts (16 bits), the groups and the round's list of particles by cell; the
// scan's scratch and counters; the queue of cell-changing particles.
// Sparse tiles (`share`): the currents take the place of the fields and the
// lists once these are done with, so that two workgroups fit a CU.  Dense
// tiles: fields and currents side by side, and the queue in the place of the
// groups.
struct QuadLds {
    int pr, ps;          // pitch of a row of six components, of a plane
    int ej[3][3];        // extents of the current components
    int pj[3];           // and pitches of their planes
    int oj[3];           // first value of each
    int jvol;            // values of all
    int qcap, gcap;      // entries of the queue and groups
    unsigned j, cnt, sh, list, desc, q, total;   // byte offsets
};

inline QuadLds quad_lds(const TileGeo &tg, int round, int nth, bool share)
{
    QuadLds L;
    L.pr = bank_pitch(6 * tg.rf[0]);
    L.ps = bank_pitch(L.pr * tg.rf[1]);
    int v = 0;
    for (int m = 0; m < 3; ++m) {
        L.oj[m] = v;
        for (int d = 0; d < 3; ++d)
            // along its own axis a component has one node less
            L.ej[m][d] = tg.rj[d] - (d == m ? 1 : 0);
        // eight cells along x times two planes fall on all banks (where the
        // LDS has room)
        const int plane = L.ej[m][0] * L.ej[m][1];
        L.pj[m] = plane + (share ? ((8 - plane % 16) + 16) % 16 : 0);
        v += L.pj[m] * L.ej[m][2];
    }
    L.jvol = v;
    const unsigned jbytes = (unsigned)(v * (int)sizeof(double));
    const int slots = (tg.t[0] + 2 * tg.slack) * (tg.t[1] + 2 * tg.slack) * (tg.t[2] + 2 * tg.slack);
    // groups: a full one per four particles and a partial one per cell, or
    // what the waves keep
    L.gcap = share ? nth / 64 * QD_BATCH * 16 : round / 4 + (round < slots ? round : slots) * 3 / 4 + 2;
    unsigned o = (unsigned)(L.ps * tg.rf[2] * (int)sizeof(float));
    if (!share) {
        L.j = (o + 15) & ~15u;
        o = L.j + jbytes;
    }
    L.cnt = o;
    o += 4u * ((slots + 1) / 2);
    L.desc = o;
    o += 4u * L.gcap;
    L.list = o;
    o += 2u * round;
    o = (o + 15) & ~15u;
    if (share) {
        L.j = 0;
        o = o > jbytes ? o : jbytes;
    }
    L.sh = o;
    o += 4 * (2 * QD_WAVES + 8);
    L.q = share ? o : L.desc;
    L.qcap = share ? round : 2 * L.gcap;
    o += share ? 2u * round : 0u;
    L.total = (o + 15) & ~15u;
    return L;
}

// Element i of a global array of 4-byte values at a uniform base.  N: the byte
// offset fits 32 bits (at most 2^30 values), so that an access takes one
// address register beside the scalar base.
template <bool N, typename V>
__device__ __attribute__((always_inline)) inline V &elem(V *base, int i)
{
    static_assert(sizeof(V) == 4, "4-byte elements");
    using C = typename std::conditional<std::is_const<V>::value, const char, char>::type;
    return N ? *reinterpret_cast<V *>(reinterpret_cast<C *>(base) + ((unsigned)i << 2)) : base[i];
}

template <int CTRL>
__device__ inline float quad_perm(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// the value of lane R of the quad
template <int R>
__device__ inline float quad_lane(float v)
{
    return quad_perm<R * 0x55>(v);
}

// The six field components at the quad's particles.  Columns of a matrix
// product are the particles (weights wk of the summed axis, this lane's own
// particle's), rows the nodes whose values the lanes read at row[m] (this
// lane's); one product per node of the looped axis (weights wl), then the row
// axis is summed with the weights wr.  The taps of a product are read two
// products ahead, as a wave would otherwise wait out the LDS latency at each of
// the 29.
struct QuadComp {
    int nk, nl;         // taps of the summed and of the looped axis
    int k, l, r;        // their axes and the row axis
    bool ks, ls;        // staggered: the five-tap weights
};

// staggering: E_x(s,n,n) E_y(n,s,n) E_z(n,n,s) B_x(n,s,s) B_y(s,n,s) B_z(s,s,n)
__device__ constexpr QuadComp QCOMP[6] = {
    {5, 4, 0, 2, 1, true, false}, {4, 5, 0, 1, 2, false, true}, {4, 5, 0, 2, 1, false, true},
    {5, 5, 1, 2, 0, true, true},  {5, 5, 0, 2, 1, true, true},  {5, 5, 0, 1, 2, true, true},
};
constexpr int QSTEPS = 29;   // products: 4 + 5 * 5

__device__ __attribute__((always_inline)) inline void quad_gather(const float *const *row, int PR, int PS,
                                                                  const float (*wn)[4], const float (*ww)[5],
                                                                  float *out)
{
    const int st[3] = {1, PR, PS};
    float x[3][5], v[4];
    auto load = [&](int s, float *t) {
        const int m = s < 4 ? 0 : (s + 1) / 5, k = s < 4 ? s : (s + 1) % 5;
#pragma unroll
        for (int i = 0; i < 5; ++i)
            if (i < QCOMP[m].nk)
                t[i] = row[m][k * st[QCOMP[m].l] + i * st[QCOMP[m].k]];
    };
    load(0, x[0]);
    load(1, x[1]);
#pragma unroll
    for (int s = 0; s < QSTEPS; ++s) {
        const int m = s < 4 ? 0 : (s + 1) / 5, k = s < 4 ? s : (s + 1) % 5;
        const QuadComp q = QCOMP[m];
        if (s + 2 < QSTEPS)
            load(s + 2, x[(s + 2) % 3]);
        __builtin_amdgcn_sched_barrier(1);   // the reads stay here
        f4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 5; ++i)
            if (i < q.nk)
                d = __builtin_amdgcn_mfma_f32_4x4x1f32(x[s % 3][i], q.ks ? ww[q.k][i] : wn[q.k][i], d, 0, 0, 0);
        const float wl = q.ls ? ww[q.l][k] : wn[q.l][k];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[r] = k == 0 ? wl * d[r] : __builtin_fmaf(wl, d[r], v[r]);
        if (k == q.nl - 1)
            out[m] = wn[q.r][0] * v[0] + wn[q.r][1] * v[1] + wn[q.r][2] * v[2] + wn[q.r][3] * v[3];
    }
}

// Shapes of one axis for the particle in turn (offsets d0 -> d1 in its
// cell), at this lane's node: S0 = w(d0), DS = w(d1) - w(d0) as (d1 - d0)
// times the divided difference, from the node's polynomial coefficients.
// The polynomials have whole coefficients and are scaled at the end, as the
// shapes of the other kernels are: the rounding of 1/6 enters at the same place.
struct NodePoly {
    float c0, c1, c2, c3;   // w(d) = (c0 + d (c1 + d (c2 + d c3))) / 6
    float qa, qb, qc, qs;   // divided difference: (qa + qb (a + b) + qc (a^2 + a b + b^2)) qs
};

__device__ inline NodePoly node_poly(int j)
{
    NodePoly p;
    p.c0 = j == 1 ? 4.f : j == 3 ? 0.f : 1.f;
    p.c1 = j == 0 ? -3.f : j == 2 ? 3.f : 0.f;
    p.c2 = j == 1 ? -6.f : j == 3 ? 0.f : 3.f;
    p.c3 = j == 0 ? -1.f : j == 1 ? 3.f : j == 2 ? -3.f : 1.f;
    p.qa = j == 0 ? -3.f : j == 2 ? 1.f : 0.f;
    p.qb = j == 0 ? 3.f : j == 1 ? -2.f : j == 2 ? 1.f : 0.f;
    p.qc = j == 0 || j == 2 ? -1.f : 1.f;
    p.qs = j == 0 || j == 3 ? 1.f / 6.f : 0.5f;
    return p;
}

// One component of the deposit of particle R of the quad, node C of the
// looped axis: the matrix product of the running sums P along the component's
// axis and the profile over the other two, with this lane's node of each.
// The columns (the lanes of the result) lie along z for every component: for
// J_x and J_y the profile's nodes, for J_z the running sums, so that
// neighbouring quads, whose cells follow along x, add to distinct addresses
// (atomics to one address are served one after the other).
template <int M, int C>
__device__ __attribute__((always_inline)) inline f4 quad_deposit(float P, float S0, float DS, float Aq, float Bq, f4 acc)
{
    const float c = __builtin_fmaf(quad_lane<C>(Bq), DS, quad_lane<C>(Aq) * S0);
    return M == 2 ? __builtin_amdgcn_mfma_f32_4x4x1f32(c, P, acc, 0, 0, 0)
                  : __builtin_amdgcn_mfma_f32_4x4x1f32(P, c, acc, 0, 0, 0);
}

// this lane's particle along one axis: old offset, sum and difference of the
// offsets, a^2 + a b + b^2, and the component's prefactor times the weight
struct QuadMove {
    float a[3], sm[3], p2[3], dd[3], K[3];
};

template <int R>
__device__ __attribute__((always_inline)) inline void quad_deposit_particle(const NodePoly &np, const QuadMove &v,
                                                                            float m1, float m2, f4 (*acc)[4])
{
    float S0[3], DS[3], A[3], B[3], P[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const float a = quad_lane<R>(v.a[d]);
        S0[d] = (np.c0 + a * (np.c1 + a * (np.c2 + a * np.c3))) * (1.f / 6.f);
        DS[d] = quad_lane<R>(v.dd[d]) *
                ((np.qa + np.qb * quad_lane<R>(v.sm[d]) + np.qc * quad_lane<R>(v.p2[d])) * np.qs);
        A[d] = S0[d] + 0.5f * DS[d];
        B[d] = 0.5f * S0[d] + (1.f / 3.f) * DS[d];
        // running sum over the quad's nodes
        const float t = __builtin_fmaf(quad_perm<0x90>(DS[d]), m1, DS[d]);   // lanes 0,0,1,2
        P[d] = quad_lane<R>(v.K[d]) * __builtin_fmaf(quad_perm<0x44>(t), m2, t);   // lanes 0,1,0,1
    }
    // J_x: profile nodes along z, loop along y; J_y: z, loop x; J_z: profile
    // nodes along x, loop y
#define PIC_QUAD_NODE(c)                                                                \
    acc[0][c] = quad_deposit<0, c>(P[0], S0[2], DS[2], A[1], B[1], acc[0][c]);          \
    acc[1][c] = quad_deposit<1, c>(P[1], S0[2], DS[2], A[0], B[0], acc[1][c]);          \
    acc[2][c] = quad_deposit<2, c>(P[2], S0[0], DS[0], A[1], B[1], acc[2][c]);
    PIC_QUAD_NODE(0)
    PIC_QUAD_NODE(1)
    PIC_QUAD_NODE(2)
    PIC_QUAD_NODE(3)
#undef PIC_QUAD_NODE
}

struct QuadArgs {
    PConst<float> pc;
    TileGeo tg;
    QuadLds L;
    PArr<float> in, out;
    FieldPtrs<float> fp;
    const int *tile_start;
    StrayList strays;
    GuestArgs g;
    float *f0[3];   // old offsets of the particles that change cells (in.off when the step is not in place)
    int round;      // particles per round, at most
    int *err;
};

// a member added to the arguments, or to a struct among them, that these
// kernels use has to be copied below: it would be uninitialised there
static_assert(sizeof(QuadArgs) == 640, "quad_args copies the members that the kernels use: look it over");

// The kernel's arguments, read again from the argument segment: each phase
// of the kernel takes its own copy, so that it holds only what it uses in
// scalar registers (all of them at once spill to vector registers, and those
// to memory).
__device__ __attribute__((always_inline)) inline QuadArgs quad_args()
{
    const uint64_t v = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    asm volatile("" : "+s"(lo), "+s"(hi));
    // (marked uniform, and read member by member from the constant address
    // space, so that these are scalar loads of pointers to global memory)
    lo = __builtin_amdgcn_readfirstlane(lo);
    hi = __builtin_amdgcn_readfirstlane(hi);
    const auto p = (const __attribute__((address_space(4))) QuadArgs *)((uint64_t)hi << 32 | lo);
    QuadArgs a;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        a.pc.n[d] = p->pc.n[d];
        a.pc.dtd[d] = p->pc.dtd[d];
        a.pc.jk[d] = p->pc.jk[d];
        a.tg.t[d] = p->tg.t[d];
        a.tg.nt[d] = p->tg.nt[d];
        a.tg.rf[d] = p->tg.rf[d];
        a.tg.rj[d] = p->tg.rj[d];
#pragma unroll
        for (int m = 0; m < 3; ++m)
            a.L.ej[m][d] = p->L.ej[m][d];
        a.L.oj[d] = p->L.oj[d];
        a.L.pj[d] = p->L.pj[d];
        a.in.cell[d] = p->in.cell[d];
        a.in.off[d] = p->in.off[d];
        a.in.u[d] = p->in.u[d];
        a.out.cell[d] = p->out.cell[d];
        a.out.off[d] = p->out.off[d];
        a.out.u[d] = p->out.u[d];
        a.fp.E[d] = p->fp.E[d];
        a.fp.B[d] = p->fp.B[d];
        a.fp.J[d] = p->fp.J[d];
        a.f0[d] = p->f0[d];
    }
    a.pc.h = p->pc.h;
    a.pc.inv_c2 = p->pc.inv_c2;
    a.pc.w0 = p->pc.w0;
    a.pc.lj = p->pc.lj;
    a.pc.vay = p->pc.vay;
    a.tg.slack = p->tg.slack;
    a.tg.lo_f = p->tg.lo_f;
    a.tg.lo_j = p->tg.lo_j;
    a.tg.jp = p->tg.jp;
    a.tg.xcd_map = p->tg.xcd_map;
    a.tg.qcap = p->tg.qcap;
    a.L.pr = p->L.pr;
    a.L.ps = p->L.ps;
    a.L.jvol = p->L.jvol;
    a.L.qcap = p->L.qcap;
    a.L.gcap = p->L.gcap;
    a.L.j = p->L.j;
    a.L.cnt = p->L.cnt;
    a.L.sh = p->L.sh;
    a.L.list = p->L.list;
    a.L.desc = p->L.desc;
    a.L.q = p->L.q;
    a.L.total = p->L.total;
    a.in.w = p->in.w;
    a.in.n = p->in.n;
    a.out.w = p->out.w;
    a.out.n = p->out.n;
    a.tile_start = p->tile_start;
    a.strays.p = p->strays.p;
    a.strays.cnt = p->strays.cnt;
    a.strays.cap = p->strays.cap;
    a.g.cnt = p->g.cnt;
    a.g.list = p->g.list;
    a.g.flag = p->g.flag;
    a.g.cnt_next = p->g.cnt_next;
    a.g.list_next = p->g.list_next;
    a.g.flag_next = p->g.flag_next;
    a.g.cap = p->g.cap;
    a.round = p->round;
    a.err = p->err;
    return a;
}

// a round of a tile: particles [jb, je) of its own (np) and guests
struct QuadRound {
    int jb, je, np, total;
};

// index in the particle arrays of particle j of a tile (own ones first)
template <bool G>
__device__ __attribute__((always_inline)) inline int quad_index(const QuadArgs &A, const TileSpan &ts, int np, int j)
{
    return !G || j < np ? (int)ts.ps + j : A.g.list[(int64_t)ts.t * A.g.cap + (j - np)].x;
}

// Field staging.  QD_STAGE rows per thread are requested before the first is
// stored, without branches between the loads (a lane or row past the region
// reads its last value and stores nothing), as region_stage does; written out
// here because that took 100 x 84 x 175 at 4 per cell from 3.90 to 4.08 ms for
// four steps.
template <int PRC, int PSC, int RFX>
__device__ __attribute__((always_inline)) inline void quad_stage(const TileSpan &ts, float *sF)
{
    constexpr bool N = RFX > 0;
    const QuadArgs A = quad_args();
    const TileGeo &tg = A.tg;
    const int tid = threadIdx.x, nth = blockDim.x;
    const int rfx = RFX ? RFX : tg.rf[0], rfy = tg.rf[1], PR = PRC ? PRC : A.L.pr, PS = PSC ? PSC : A.L.ps;
    if (region_wraps_once(A.pc.n, tg.t, tg.lo_f, tg.rf)) {
        const int lb = 32 - __clz(rfx - 1);
        const int x = tid & ((1 << lb) - 1), step = nth >> lb, rfz = tg.rf[2];
        const int gx = wrap_once(ts.t0[0] - tg.lo_f + (x < rfx ? x : rfx - 1), A.pc.n[0]);
        int y = (tid >> lb) % rfy, z = (tid >> lb) / rfy;
        const int sy = step % rfy, sz = step / rfy;
        for (int r = 0; r < rfy * rfz; r += QD_STAGE * step) {
            float v[QD_STAGE][6];
            int at[QD_STAGE];
#pragma unroll
            for (int t = 0; t < QD_STAGE; ++t) {
                const bool in = x < rfx && z < rfz;
                const int gy = wrap_once(ts.t0[1] - tg.lo_f + y, A.pc.n[1]);
                const int gz = wrap_once(ts.t0[2] - tg.lo_f + (z < rfz ? z : rfz - 1), A.pc.n[2]);
                const int gi = gx + A.pc.n[0] * (gy + A.pc.n[1] * gz);
                at[t] = in ? x + PR * y + PS * z : -1;
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    v[t][m] = elem<N>(A.fp.E[m], gi);
                    v[t][3 + m] = elem<N>(A.fp.B[m], gi);
                }
                y += sy;
                z += sz;
                const bool over = y >= rfy;
                y -= over ? rfy : 0;
                z += over ? 1 : 0;
            }
#pragma unroll
            for (int t = 0; t < QD_STAGE; ++t)
                if (at[t] >= 0) {
#pragma unroll
                    for (int m = 0; m < 6; ++m)
                        sF[at[t] + m * rfx] = v[t][m];
                }
        }
    } else {
        region_cells(A.pc.n, ts.t0, tg.lo_f, rfx, rfy, tg.rf[2], false, [&](int x, int y, int z, int gi) {
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                sF[x + m * rfx + PR * y + PS * z] = elem<N>(A.fp.E[m], gi);
                sF[x + (3 + m) * rfx + PR * y + PS * z] = elem<N>(A.fp.B[m], gi);
            }
        });
    }
}

// Groups the round's particles by cell: fills the list and the groups, puts
// the particles outside the region (or with a corrupt cell, which that
// kernel reports) on the stray kernel's list.  When there are more groups
// than there is room for, the round is halved.  Counters: queued cell
// changes, batches taken, third and later groups, all groups, listed
// particles.  Begins with a barrier and ends with one.
template <bool G, bool N, int PER>
__device__ __attribute__((always_inline)) inline void quad_lists(const TileSpan &ts, QuadRound &R,
                                                                 unsigned char *smem)
{
    const QuadArgs A = quad_args();
    const TileGeo &tg = A.tg;
    const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = nth >> 6;
    unsigned *cnt = reinterpret_cast<unsigned *>(smem + A.L.cnt);   // two cells per word
    unsigned short *cnt16 = reinterpret_cast<unsigned short *>(cnt);
    int *sh = reinterpret_cast<int *>(smem + A.L.sh), *ctr = sh + 2 * QD_WAVES;
    unsigned *desc = reinterpret_cast<unsigned *>(smem + A.L.desc);
    unsigned short *list = reinterpret_cast<unsigned short *>(smem + A.L.list);
    const int sl = tg.slack, ex = tg.t[0] + 2 * sl, ey = tg.t[1] + 2 * sl;
    const int slots = ex * ey * (tg.t[2] + 2 * sl), sper = (slots + nth - 1) / nth;
    // this thread's particles: the slot of their cell, or -1 (no particle, or
    // a guest that another tile moves), or -2 for the stray kernel's
    int key[PER];
    {
        // (no branches between the loads: a thread without a particle reads
        // the round's last one)
        int c[PER][3], p[PER], fl[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = R.jb + k * nth + tid < R.je ? R.jb + k * nth + tid : R.je - 1;
            p[k] = (int)ts.ps + j;
            if (G && R.total > R.np)
                p[k] = j < R.np ? p[k] : A.g.list[(int64_t)ts.t * A.g.cap + (j < R.np ? 0 : j - R.np)].x;
            fl[k] = 0;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                c[k][d] = elem<N>(A.in.cell[d], p[k]);
        if (G && A.g.flag) {
#pragma unroll
            for (int k = 0; k < PER; ++k)
                fl[k] = R.jb + k * nth + tid < R.np ? A.g.flag[p[k]] : 0;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int j = R.jb + k * nth + tid;
            bool ok = true;
#pragma unroll
            for (int d = 0; d < 3; ++d)
                ok = ok & (c[k][d] >= 0) & (c[k][d] < A.pc.n[d]);
            int l[3];
            const bool in = tile_local(tg, A.pc.n, ts.t0, c[k], l);
            key[k] = ok & in ? l[0] + sl + ex * (l[1] + sl + ey * (l[2] + sl)) : -2;
            // (a guest's cell cannot be outside: its list was built from it in
            // this call)
            if (G && key[k] == -2 && j >= R.np && j < R.je) {
                atomicOr(A.err, 2);
                key[k] = -1;
            }
            if (j >= R.je || fl[k])
                key[k] = -1;
        }
    }
    int rank[PER];
    for (;;) {
        for (int i = tid; 2 * i < slots; i += nth)
            cnt[i] = 0;
        if (tid < 5)
            ctr[tid] = 0;
        __syncthreads();   // also: the field tile is staged
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (key[k] >= 0 && R.jb + k * nth + tid < R.je) {
                const int h = 16 * (key[k] & 1);
                rank[k] = (int)((atomicAdd(cnt + (key[k] >> 1), 1u << h) >> h) & 0xffff);
            }
        __syncthreads();
        // First one group of every occupied cell, then a second one of the
        // cells that hold more, so that neighbouring quads sit in different
        // cells; third and later groups take the places after them in any
        // order.  A thread counts sper consecutive cells.
        int n[QD_SLOTS];
        unsigned v = 0;
        int v2 = 0, more = 0;
#pragma unroll
        for (int i = 0; i < QD_SLOTS; ++i) {
            const int s = tid * sper + i;
            n[i] = i < sper && s < slots ? cnt16[s] : 0;
            v += (unsigned)n[i] | (n[i] > 0 ? 1u << 16 : 0u);
            v2 += n[i] > 4 ? 1 : 0;
            more += n[i] > 8 ? (n[i] - 5) / 4 : 0;
        }
        unsigned x = v;
        int x2 = v2 | more << 16;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned y = __shfl_up(x, o, 64);
            const int y2 = __shfl_up(x2, o, 64);
            if (lane >= o) {
                x += y;
                x2 += y2;
            }
        }
        if (lane == 63) {
            sh[wv] = (int)x;
            sh[QD_WAVES + wv] = x2;
        }
        __syncthreads();
        // totals of the waves before this one, and of all
        unsigned before = 0, all = 0;
        int before2 = 0, all2 = 0;
        for (int w = 0; w < nw; ++w) {
            const unsigned t = (unsigned)sh[w];
            const int t2 = sh[QD_WAVES + w];
            before += w < wv ? t : 0u;
            before2 += w < wv ? t2 : 0;
            all += t;
            all2 += t2;
        }
        const int g1 = (int)(all >> 16), g2 = g1 + (all2 & 0xffff), g3 = g2 + (all2 >> 16);
        if (g3 > A.L.gcap) {
            R.je = R.jb + (R.je - R.jb + 1) / 2;   // uniform
            __syncthreads();
            continue;
        }
        unsigned first = before + x - v;
        int at2 = g1 + ((before2 + x2) & 0xffff) - v2;
#pragma unroll
        for (int i = 0; i < QD_SLOTS; ++i) {
            if (n[i] > 0) {
                const int sid = tid * sper + i;
                const unsigned s = first & 0xffff;
                cnt16[sid] = (unsigned short)s;
                const unsigned cell = (unsigned)(sid % ex) << 16 | (unsigned)((sid / ex) % ey) << 21 |
                                      (unsigned)(sid / (ex * ey)) << 26;
                desc[first >> 16] = s | (unsigned)(n[i] < 4 ? n[i] : 4) << 13 | cell;
                if (n[i] > 4)
                    desc[at2++] = (s + 4) | (unsigned)(n[i] < 8 ? n[i] - 4 : 4) << 13 | cell;
                for (int r = 8; r < n[i]; r += 4)
                    desc[g2 + atomicAdd(ctr + 2, 1)] = (s + r) | (unsigned)(n[i] - r < 4 ? n[i] - r : 4) << 13 | cell;
                first += (unsigned)n[i] | 1u << 16;
            }
        }
        if (tid == 0) {
            ctr[3] = g3;
            ctr[4] = (int)(all & 0xffff);
        }
        break;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int j = R.jb + k * nth + tid;
        if (key[k] >= 0 && j < R.je)
            list[cnt16[key[k]] + rank[k]] = (unsigned short)(j - R.jb);
        stray_append(key[k] == -2 && j < R.je, (int)ts.ps + j, A.strays);
    }
    __syncthreads();
}

// A lane's particle of a batch of sixteen groups: its group (0: none), its
// index in the arrays (-1: none) and in the round, its state.
struct QuadParticle {
    unsigned d;
    int p, jc;
    float f[3], u[3], w;
};

template <bool G, bool N>
__device__ __attribute__((always_inline)) inline void quad_fetch(const QuadArgs &A, const TileSpan &ts,
                                                                 const QuadRound &R, const unsigned *desc,
                                                                 const unsigned short *list, int gi, int ngr,
                                                                 QuadParticle &q)
{
    const int jj = threadIdx.x & 3;
    q.d = gi < ngr ? desc[gi] : 0u;
    q.p = -1;
    q.jc = 0;
    q.w = A.pc.w0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        q.f[k] = 0.5f;
        q.u[k] = 0.f;
    }
    if (jj < (int)((q.d >> 13) & 7)) {
        q.jc = list[(q.d & 0x1fff) + jj];
        q.p = quad_index<G>(A, ts, R.np, R.jb + q.jc);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            q.f[k] = elem<N>(A.in.off[k], q.p);
            q.u[k] = elem<N>(A.in.u[k], q.p);
        }
        if (A.in.w)
            q.w = elem<N>(A.in.w, q.p);
    }
}

// Gather, push and move of a batch (the whole wave converged); q.w becomes 0
// and the new offsets f1 a half where nothing is deposited with the narrow
// window: no particle, one that changed cells (queued for the full window by
// cross(i), and its old offsets kept where the step runs in place) or a
// rejected one.
template <bool G, int PRC, int PSC, int RFX, typename CrossFn>
__device__ __attribute__((always_inline)) inline void quad_advance(const QuadArgs &A, const TileSpan &ts,
                                                                   const QuadRound &R, const float *sF,
                                                                   QuadParticle &q, float *f1, CrossFn &&crossed)
{
    using S = Shape<3, float>;
    constexpr int NW = S::NW, NB = S::NB;
    constexpr bool N = RFX > 0;
    const TileGeo &tg = A.tg;
    const PArr<float> &in = A.in, &out = A.out;
    const int jj = threadIdx.x & 3;
    const int rfx = RFX ? RFX : tg.rf[0], PR = PRC ? PRC : A.L.pr, PS = PSC ? PSC : A.L.ps, sl = tg.slack;
    const int l[3] = {(int)((q.d >> 16) & 31) - sl, (int)((q.d >> 21) & 31) - sl, (int)(q.d >> 26) - sl};
    const int p = q.p;
    bool live = p >= 0;
    int bad = 0;
    {
        bool ok = finite3(q.u);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            ok = ok & (q.f[k] >= 0.f) & (q.f[k] < 1.f);
        bad = ok ? 0 : 1;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            q.f[k] = ok ? q.f[k] : 0.5f;
            q.u[k] = ok ? q.u[k] : 0.f;
        }
    }
    float E[3], B[3];
    {
        float wn[3][NW], ww[3][NW + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            S::w(q.f[k], wn[k]);
            float ws[NW];
            const bool up = q.f[k] >= 0.5f;
            S::w(up ? q.f[k] - 0.5f : q.f[k] + 0.5f, ws);
            ww[k][0] = up ? 0.f : ws[0];
#pragma unroll
            for (int i = 1; i < NW; ++i)
                ww[k][i] = up ? ws[i - 1] : ws[i];
            ww[k][NW] = up ? ws[NW - 1] : 0.f;
        }
        // first nodal node of the window; a staggered axis starts one lower
        const float *F = sF + (l[0] + tg.lo_f + NB) + PR * (l[1] + tg.lo_f + NB) + PS * (l[2] + tg.lo_f + NB);
        const float *Fx = F + jj, *Fy = F + PR * jj, *Fz = F + PS * jj;   // this lane's row
        const float *row[6] = {Fy - 1,
                               Fz + rfx - PR,
                               Fy + 2 * rfx - PS,
                               Fx + 3 * rfx - PR - PS,
                               Fy + 4 * rfx - 1 - PS,
                               Fz + 5 * rfx - 1 - PR};
        float eb[6];
        quad_gather(row, PR, PS, wn, ww, eb);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            E[k] = eb[k];
            B[k] = eb[3 + k];
        }
    }
    float u1[3];
    push_momentum(A.pc, q.u, E, B, u1);
    const float ig = 1.f / sqrtf(1.f + (u1[0] * u1[0] + u1[1] * u1[1] + u1[2] * u1[2]) * A.pc.inv_c2);
    int kap[3];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float disp = A.pc.dtd[k] * u1[k] * ig;
        ok = ok & (fabsf(disp) < 1.f);
        move_axis(q.f[k], disp, f1[k], kap[k]);
    }
    bad |= ok ? 0 : 2;
    if (live && bad) {
        atomicOr(A.err, bad & 1);
        // a corrupt offset or momentum, or a move of a cell or more (also from
        // a field that is not finite at the one node of a five-tap window
        // that is not the particle's): the stray kernel's, which reports it
        const int i = atomicAdd(A.strays.cnt, 1);
        if (i < A.strays.cap)
            A.strays.p[i] = p;
        live = false;
    }
    const bool cross = (kap[0] | kap[1] | kap[2]) != 0;
    if (live) {
        const bool inplace = in.cell[0] == out.cell[0];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            elem<N>(out.off[k], p) = f1[k];
            elem<N>(out.u[k], p) = u1[k];
        }
        if (out.w && out.w != in.w)
            elem<N>(out.w, p) = q.w;
        int c1[3] = {0, 0, 0};
        if (cross || !inplace) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                c1[k] = wrap_once(wrap_once(ts.t0[k] + l[k], A.pc.n[k]) + kap[k], A.pc.n[k]);
                elem<N>(out.cell[k], p) = c1[k];
            }
        }
        if (cross) {
            crossed();
            if (inplace) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    elem<N>(A.f0[k], p) = q.f[k];
            }
        }
        if (G) {
            // a particle that changed cells, or a guest, gets its status for
            // the next step
            unsigned char gn = 0;
            const bool own = R.jb + q.jc < R.np;
            if (cross || !own) {
                int ht0[3] = {ts.t0[0], ts.t0[1], ts.t0[2]}, home = ts.t;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    c1[k] = wrap_once(wrap_once(ts.t0[k] + l[k], A.pc.n[k]) + kap[k], A.pc.n[k]);
                if (!own) {
                    home = A.g.list[(int64_t)ts.t * A.g.cap + (R.jb + q.jc - R.np)].y;
                    tile_origin(tg, home, ht0);
                }
                gn = guest_next(A.g, tg, A.pc.n, p, home, ht0, c1);
            }
            A.g.flag_next[p] = gn;
        }
    }
    const bool still = live && !cross;
    q.w = still ? q.w : 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        f1[k] = still ? f1[k] : 0.5f;
}

// Narrow-window deposit of a batch: groups d, offsets a -> e, weights w (0:
// nothing).
__device__ __attribute__((always_inline)) inline void quad_deposit_batch(const QuadArgs &A, double *sJ, unsigned d,
                                                                         const float *a, const float *e, float w,
                                                                         const NodePoly &poly)
{
    constexpr int NW = 4, NB = -1;
    const int jj = threadIdx.x & 3, sl = A.tg.slack, lo = A.tg.lo_j + NB;
    const float m1 = jj >= 1 ? 1.f : 0.f, m2 = jj >= 2 ? 1.f : 0.f;
    QuadMove mv;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        mv.a[k] = a[k];
        mv.sm[k] = a[k] + e[k];
        mv.p2[k] = a[k] * a[k] + a[k] * e[k] + e[k] * e[k];
        mv.dd[k] = e[k] - a[k];
        mv.K[k] = A.pc.jk[k] * w;
    }
    f4 acc[3][4];
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            acc[m][k] = f4{0.f, 0.f, 0.f, 0.f};
    // Particles that no group of the wave holds are passed over (the first groups
    // of all cells come first, so at low density whole waves hold one or two
    // each): 96^3, 1 per cell, cold 245 -> 234 us a step, 256^3, 8 per cell 12.6
    // -> 12.5 ms.
    const int count = (int)((d >> 13) & 7);
    quad_deposit_particle<0>(poly, mv, m1, m2, acc);
    if (__ballot(count > 1)) {
        quad_deposit_particle<1>(poly, mv, m1, m2, acc);
        if (__ballot(count > 2)) {
            quad_deposit_particle<2>(poly, mv, m1, m2, acc);
            quad_deposit_particle<3>(poly, mv, m1, m2, acc);
        }
    }
    if (d != 0) {
        const int o[3] = {(int)((d >> 16) & 31) - sl + lo, (int)((d >> 21) & 31) - sl + lo, (int)(d >> 26) - sl + lo};
        double *a0[3];
        int py[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            py[m] = A.L.ej[m][0];
            a0[m] = sJ + A.L.oj[m] + o[0] + py[m] * o[1] + A.L.pj[m] * (o[2] + jj);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < NW - 1; ++i) {
                latomic_add(a0[0] + py[0] * k + i, (double)acc[0][k][i]);
                latomic_add(a0[1] + k + py[1] * i, (double)acc[1][k][i]);
            }
        if (jj < NW - 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < NW; ++i)
                    latomic_add(a0[2] + py[2] * k + i, (double)acc[2][k][i]);
        }
    }
}

// The queued cell-changing particles, one lane per particle and component
// (component-major, so that a wave mostly takes one).
template <bool G, bool N>
__device__ __attribute__((always_inline)) inline void quad_crossers(const QuadArgs &A, const TileSpan &ts,
                                                                    const QuadRound &R, const unsigned short *queue,
                                                                    int nq, double *sJ)
{
    const TileGeo &tg = A.tg;
    for (int i = threadIdx.x; i < 3 * nq; i += blockDim.x) {
        const int m = i / nq, p = quad_index<G>(A, ts, R.np, R.jb + queue[i - m * nq]);
        int cn[3], l[3], kap[3];
        float f0[3], f1[3], u1[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            cn[k] = elem<N>(A.out.cell[k], p);
            f0[k] = elem<N>(A.f0[k], p);
            f1[k] = elem<N>(A.out.off[k], p);
            u1[k] = elem<N>(A.out.u[k], p);
        }
        const float w = A.in.w ? elem<N>(A.in.w, p) : A.pc.w0;
        // The cell it left: the displacement again, from the new momentum, is
        // the difference of the offsets but for whole cells.  (Its last bits
        // may differ from the first time's, so the cell change is rounded
        // from the stored offsets and never taken from a second move.)
        const float ig = 1.f / sqrtf(1.f + (u1[0] * u1[0] + u1[1] * u1[1] + u1[2] * u1[2]) * A.pc.inv_c2);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            kap[k] = (int)rintf(f0[k] + A.pc.dtd[k] * u1[k] * ig - f1[k]);
            cn[k] = wrap_once(cn[k] - kap[k], A.pc.n[k]);
        }
        tile_local(tg, A.pc.n, ts.t0, cn, l);
        if (m == 0) {
            const int sj[3] = {1, A.L.ej[0][0], A.L.pj[0]};
            deposit_local_comp<float, 3, 0>(A.pc, f0, f1, kap, l, tg.lo_j, sj, w, sJ + A.L.oj[0]);
        } else if (m == 1) {
            const int sj[3] = {1, A.L.ej[1][0], A.L.pj[1]};
            deposit_local_comp<float, 3, 1>(A.pc, f0, f1, kap, l, tg.lo_j, sj, w, sJ + A.L.oj[1]);
        } else {
            const int sj[3] = {1, A.L.ej[2][0], A.L.pj[2]};
            deposit_local_comp<float, 3, 2>(A.pc, f0, f1, kap, l, tg.lo_j, sj, w, sJ + A.L.oj[2]);
        }
    }
}

__device__ __attribute__((always_inline)) inline void quad_clear(double *sJ)
{
    const QuadArgs A = quad_args();
    for (int r = threadIdx.x; r < A.L.jvol; r += blockDim.x)
        sJ[r] = 0.0;
}

// adds the tile's currents to global memory
template <bool N>
__device__ __attribute__((always_inline)) inline void quad_flush(const TileSpan &ts, const double *sJ)
{
    const QuadArgs A = quad_args();
    const TileGeo &tg = A.tg;
    region_cells(A.pc.n, ts.t0, tg.lo_j, tg.rj[0], tg.rj[1], tg.rj[2],
                 region_wraps_once(A.pc.n, tg.t, tg.lo_j, tg.rj), [&](int x, int y, int z, int gi) {
                     const int at[3] = {x, y, z};
#pragma unroll
                     for (int m = 0; m < 3; ++m) {
                         if (at[m] >= A.L.ej[m][m])
                             continue;
                         const float v = (float)sJ[A.L.oj[m] + x + A.L.ej[m][0] * y + A.L.pj[m] * z];
                         if (v != 0.f)
                             gatomic_add(&elem<N>(A.fp.J[m], gi), v);
                     }
                 });
}

// A tile's span, its particles and guests (G: the kernel also builds the next
// step's guest lists) and the size of its rounds; false for an empty tile.
template <bool G>
__device__ __attribute__((always_inline)) inline bool quad_tile(TileSpan &ts, QuadRound &R, int &chunk)
{
    const QuadArgs A = quad_args();
    ts = tile_span(A.tg, A.tile_start, A.in.n);
    const int ng = (G && A.g.cnt) ? (A.g.cnt[ts.t] < A.g.cap ? A.g.cnt[ts.t] : A.g.cap) : 0;
    R.np = (int)(ts.pe - ts.ps);
    R.total = R.np + ng;
    const int n = (R.total + A.round - 1) / A.round;
    chunk = n > 0 ? (R.total + n - 1) / n : 0;
    return R.total > 0;
}

}  // namespace

// PRC, PSC, RFX > 0: the pitches and the row length of the field region known
// at compile time (the window's taps become constant offsets); else from
// the arguments.
//
// Sparse tiles: rounds of up to `round` particles (mostly one).  Every wave
// gathers and moves up to QD_BATCH batches, keeping what their deposit needs
// in registers; then the currents take the fields' place in LDS and the
// batches are deposited.  Of the 148k clocks that a workgroup of the laser box
// took (clock counters between the phases, in a copy of the kernel), staging was
// 15k, the lists 37k, the batches 36k, the deposit 22k, the cell-changing
// particles 13k and the flush 10k: latencies in turn, which two workgroups on a
// CU overlap.
template <bool G, int PRC, int PSC, int RFX>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) k_particles_quads(QuadArgs)
{
    constexpr bool N = RFX > 0;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    TileSpan ts;
    QuadRound R;
    int chunk;
    if (!quad_tile<G>(ts, R, chunk))
        return;   // uniform across the workgroup
    for (R.jb = 0, R.je = 0; R.jb < R.total; R.jb = R.je) {
        R.je = R.total < R.jb + chunk ? R.total : R.jb + chunk;
        quad_stage<PRC, PSC, RFX>(ts, reinterpret_cast<float *>(smem_raw));
        quad_lists<G, N, 4>(ts, R, smem_raw);
        // per batch, the last one first: group, old and new offsets, weight
        unsigned rd[QD_BATCH];
        float r0[QD_BATCH][3], r1[QD_BATCH][3], rw[QD_BATCH];
        int mine = 0;
        {
            const QuadArgs A = quad_args();
            int *ctr = reinterpret_cast<int *>(smem_raw + A.L.sh) + 2 * QD_WAVES;
            const unsigned *desc = reinterpret_cast<const unsigned *>(smem_raw + A.L.desc);
            const unsigned short *list = reinterpret_cast<const unsigned short *>(smem_raw + A.L.list);
            unsigned short *queue = reinterpret_cast<unsigned short *>(smem_raw + A.L.q);
            const int ngr = __builtin_amdgcn_readfirstlane(ctr[3]), nb = (ngr + 15) >> 4;
            for (int b = wv; b < nb; b += nw) {
                QuadParticle q;
                quad_fetch<G, N>(A, ts, R, desc, list, b * 16 + (lane >> 2), ngr, q);
                float f1[3];
                quad_advance<G, PRC, PSC, RFX>(A, ts, R, reinterpret_cast<const float *>(smem_raw), q, f1, [&]() {
                    queue[atomicAdd(ctr, 1)] = (unsigned short)q.jc;
                });
#pragma unroll
                for (int i = QD_BATCH - 1; i > 0; --i) {
                    rd[i] = rd[i - 1];
                    rw[i] = rw[i - 1];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        r0[i][k] = r0[i - 1][k];
                        r1[i][k] = r1[i - 1][k];
                    }
                }
                rd[0] = q.d;
                rw[0] = q.w;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    r0[0][k] = q.f[k];
                    r1[0][k] = f1[k];
                }
                ++mine;
            }
        }
        __syncthreads();   // the fields and the lists are done with
        double *sJ = reinterpret_cast<double *>(smem_raw);
        quad_clear(sJ);
        __syncthreads();
        {
            const QuadArgs A = quad_args();
            const NodePoly poly = node_poly(lane & 3);
            for (int b = 0; b < mine; ++b) {
                quad_deposit_batch(A, sJ, rd[0], r0[0], r1[0], rw[0], poly);
#pragma unroll
                for (int i = 0; i < QD_BATCH - 1; ++i) {
                    rd[i] = rd[i + 1];
                    rw[i] = rw[i + 1];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        r0[i][k] = r0[i + 1][k];
                        r1[i][k] = r1[i + 1][k];
                    }
                }
            }
        }
        {
            const QuadArgs A = quad_args();
            const int nq = *(reinterpret_cast<const int *>(smem_raw + A.L.sh) + 2 * QD_WAVES);
            quad_crossers<G, N>(A, ts, R, reinterpret_cast<const unsigned short *>(smem_raw + A.L.q), nq, sJ);
        }
        __syncthreads();
        quad_flush<N>(ts, sJ);
        __syncthreads();   // the next round stages its fields in the same place
    }
}

// Dense tiles: fields and currents side by side in LDS, so that a tile's
// particles need one staging and one flush; a batch is deposited right after
// its move, and the waves draw batches from a counter and request the next
// one's state before they work on the present one.
template <bool G, int PRC, int PSC, int RFX>
__global__ void __launch_bounds__(1024) k_particles_quads_dense(QuadArgs)
{
    constexpr bool N = RFX > 0;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = nth >> 6;
    TileSpan ts;
    QuadRound R;
    int chunk;
    if (!quad_tile<G>(ts, R, chunk))
        return;   // uniform across the workgroup
    quad_stage<PRC, PSC, RFX>(ts, reinterpret_cast<float *>(smem_raw));
    {
        const QuadArgs A = quad_args();
        quad_clear(reinterpret_cast<double *>(smem_raw + A.L.j));
    }
    for (R.jb = 0, R.je = 0; R.jb < R.total; R.jb = R.je) {
        R.je = R.total < R.jb + chunk ? R.total : R.jb + chunk;
        quad_lists<G, N, 5>(ts, R, smem_raw);
        {
            const QuadArgs A = quad_args();
            double *sJ = reinterpret_cast<double *>(smem_raw + A.L.j);
            int *ctr = reinterpret_cast<int *>(smem_raw + A.L.sh) + 2 * QD_WAVES;
            const unsigned *desc = reinterpret_cast<const unsigned *>(smem_raw + A.L.desc);
            unsigned short *list = reinterpret_cast<unsigned short *>(smem_raw + A.L.list);
            const NodePoly poly = node_poly(lane & 3);
            const int ngr = __builtin_amdgcn_readfirstlane(ctr[3]), nb = (ngr + 15) >> 4;
            QuadParticle nx;
            quad_fetch<G, N>(A, ts, R, desc, list, wv * 16 + (lane >> 2), ngr, nx);
            for (int b = wv; b < nb;) {
                QuadParticle q = nx;
                int t = 0;
                if (lane == 0)
                    t = atomicAdd(ctr + 1, 1);
                b = nw + __builtin_amdgcn_readfirstlane(t);
                quad_fetch<G, N>(A, ts, R, desc, list, b * 16 + (lane >> 2), ngr, nx);
                float f1[3];
                // one that changes cells is marked in the list
                quad_advance<G, PRC, PSC, RFX>(A, ts, R, reinterpret_cast<const float *>(smem_raw), q, f1, [&]() {
                    list[(q.d & 0x1fff) + (lane & 3)] = (unsigned short)(q.jc | 0x8000);
                });
                quad_deposit_batch(A, sJ, q.d, q.f, f1, q.w, poly);
            }
        }
        __syncthreads();
        // The marked particles are collected in the groups' place, which
        // holds them all at once unless most of a large round change cells.
        {
            const QuadArgs A = quad_args();
            double *sJ = reinterpret_cast<double *>(smem_raw + A.L.j);
            int *ctr = reinterpret_cast<int *>(smem_raw + A.L.sh) + 2 * QD_WAVES;
            const unsigned short *list = reinterpret_cast<const unsigned short *>(smem_raw + A.L.list);
            unsigned short *queue = reinterpret_cast<unsigned short *>(smem_raw + A.L.q);
            const int listed = ctr[4];
            for (int i0 = 0; i0 < listed; i0 += A.L.qcap) {
                if (i0 > 0) {
                    __syncthreads();   // the collected entries are worked off
                    if (tid == 0)
                        ctr[0] = 0;
                    __syncthreads();
                }
                const int ie = listed < i0 + A.L.qcap ? listed : i0 + A.L.qcap;
                for (int i = i0; i < ie; i += nth) {
                    const int e = i + tid < ie ? list[i + tid] : 0;
                    const bool mark = (e & 0x8000) != 0;
                    const unsigned long long mk = __ballot(mark);
                    int at = 0;
                    if (lane == 0 && mk)
                        at = atomicAdd(ctr, __popcll(mk));
                    at = __builtin_amdgcn_readfirstlane(at);
                    if (mark)
                        queue[at + __popcll(mk & ((1ull << lane) - 1ull))] = (unsigned short)(e & 0x7fff);
                }
                __syncthreads();
                quad_crossers<G, N>(A, ts, R, queue, ctr[0], sJ);
            }
        }
        __syncthreads();   // the next round reuses the lists
    }
    {
        const QuadArgs A = quad_args();
        quad_flush<N>(ts, reinterpret_cast<const double *>(smem_raw + A.L.j));
    }
}

// Threads, particles per round and layout of a launch.
struct QuadPlan {
    bool ok, share;
    int nth, round;
};

static QuadPlan quad_plan_as(const TileGeo &tg, int64_t want, int64_t ntiles, int slots, bool share)
{
    QuadPlan P{false, share, 0, 0};
    // the shared layout on half a CU's LDS: two workgroups
    const size_t limit = (share ? 80 : 160) * 1024;
    const int per = share ? 4 : 5, most = share ? 512 : 1024;
    // tiles of few particles take fewer threads where several share a CU; a
    // tile with a CU to itself ends sooner with all (16 x 20 x 35 in 80 tiles, 2
    // per cell: 39.6 us a step with 256 threads, 33.6 with 512; 32^3 in 512
    // tiles, 1 per cell: 32.9 / 35.8 us)
    P.nth = want <= 400 && ntiles > QD_CUS && slots <= 256 * QD_SLOTS ? 256 : (want <= 1600 || most == 512) ? 512 : 1024;
    if (slots > P.nth * QD_SLOTS)
        P.nth = most;
    if (slots > P.nth * QD_SLOTS)
        return P;
    int64_t r = want < QD_MIN_ROUND ? QD_MIN_ROUND : want;
    r = r > per * P.nth ? per * P.nth : r;
    const int64_t least = share ? (r < 1024 ? r : 1024) : (r < 2048 ? r : 2048);
    while (r >= least && quad_lds(tg, (int)r, P.nth, share).total > limit)
        r -= 32;
    P.round = (int)r;
    P.ok = r >= least;
    return P;
}

// The shared layout stages and flushes its regions once a round, so it takes
// the tiles of one round, and of a few where the regions are small and the two
// workgroups on a CU overlap (14 x 21 x 16 in 24 tiles, 12 per cell: 85.3 us a
// step in two rounds, 63.0 dense).  Shared
// against dense, particle kernel of four steps: 160^3, 8^3 tiles, 3 / 4 / 6
// per cell (one round, then two) 5.5 / 9.2 / 10.3 against 6.8 / 7.8 / 9.9 ms;
// 128^3, 8 x 8 x 4 tiles, 4 / 8 / 12 per cell 3.9 / 7.0 / 9.7 against
// 5.5 / 7.6 / 10.1 ms; 4^3 tiles, 2 per cell 4.6 against 7.0 ms.
// Tiles of more than QD_CELLS cells, which only a caller's own choice gives,
// are left to the other kernels (160^3, 16 x 8 x 8 tiles, 2 / 4 / 8 per cell:
// 5.4 / 9.3 / 16.5 ms there, 5.8 / 10.1 / 16.8 dense).
static QuadPlan quad_plan(const TileGeo &tg, int64_t n)
{
    int slots = 1, cells = 1, region = 1;
    for (int d = 0; d < 3; ++d) {
        if (tg.t[d] + 2 * tg.slack > 31)
            return QuadPlan{false, false, 0, 0};
        slots *= tg.t[d] + 2 * tg.slack;
        cells *= tg.t[d];
        region *= tg.rf[d];
    }
    if (cells > QD_CELLS)
        return QuadPlan{false, false, 0, 0};
    const int64_t ntiles = (int64_t)tg.nt[0] * tg.nt[1] * tg.nt[2];
    // With a CU for each tile a step takes the latency of its longest tile, and
    // groups of one or two particles need more batches than a workgroup has
    // waves.  One particle per thread / groups, us a step: 42 x 20 x 35 in 120
    // tiles, 1 per cell 32.6 / 37.6, 2 per cell 35.5 / 38.1; 14 x 21 x 16 in 24
    // tiles, 2 per cell 33.8 / 35.8, 4 per cell 42.8 / 36.4; 16^3 in 64 tiles, 1
    // per cell 30.5 / 26.1.
    if (ntiles <= QD_CUS && cells > 512 / 64 * 16 && 2 * n < 5 * cells * ntiles)
        return QuadPlan{false, false, 0, 0};
    // what a tile holds on average, with room for uneven ones
    const int64_t want = (n + ntiles - 1) / ntiles * 9 / 8 + 64;
    const QuadPlan S = quad_plan_as(tg, want, ntiles, slots, true);
    if (S.ok && (want <= S.round ||
                 (ntiles > QD_CUS && (want + S.round - 1) / S.round * region <= QD_RESTAGE)))
        return S;
    return quad_plan_as(tg, want, ntiles, slots, false);
}

template <bool G, int PRC, int PSC, int RFX>
static hipError_t launch_quads(const QuadArgs &a, const QuadPlan &P, unsigned ntiles, hipStream_t st)
{
    static bool attr = false;
    if (!attr) {
        for (const void *k : {reinterpret_cast<const void *>(&k_particles_quads<G, PRC, PSC, RFX>),
                              reinterpret_cast<const void *>(&k_particles_quads_dense<G, PRC, PSC, RFX>)})
            hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        attr = true;
    }
    if (P.share)
        hipLaunchKernelGGL((k_particles_quads<G, PRC, PSC, RFX>), dim3(ntiles), dim3(P.nth), a.L.total, st, a);
    else
        hipLaunchKernelGGL((k_particles_quads_dense<G, PRC, PSC, RFX>), dim3(ntiles), dim3(P.nth), a.L.total, st, a);
    return hipGetLastError();
}

bool quads_fit(const TileGeo &tg, int64_t n)
{
    return quad_plan(tg, n).ok;
}

hipError_t launch_particles_quads(const PConst<float> &pc, const TileGeo &tg, const PArr<float> &in,
                                  const PArr<float> &out, const FieldPtrs<float> &f, const int *tile_start,
                                  int *stray_list, int *stray_cnt, const GuestArgs &g, float *const scratch[3],
                                  int *err, hipStream_t st)
{
    const QuadPlan P = quad_plan(tg, in.n);
    if (!P.ok)
        return hipErrorInvalidValue;
    QuadArgs a{};
    a.pc = pc;
    a.tg = tg;
    a.L = quad_lds(tg, P.round, P.nth, P.share);
    a.in = in;
    a.out = out;
    a.fp = f;
    a.tile_start = tile_start;
    a.strays = StrayList{stray_list, stray_cnt, (int)in.n};
    a.g = g;
    for (int d = 0; d < 3; ++d)
        a.f0[d] = in.off[d] == out.off[d] ? scratch[d] : in.off[d];
    a.round = P.round;
    a.err = err;
    const unsigned ntiles = (unsigned)(tg.nt[0] * tg.nt[1] * tg.nt[2]);
    // tiles of 8 x 8 cells (any height) with one cell of slack, the automatic
    // choice on large grids, have compile-time pitches and 32-bit offsets
    const int64_t lim = int64_t(1) << 30, ncell = (int64_t)pc.n[0] * pc.n[1] * pc.n[2];
    if (a.L.pr == 88 && a.L.ps == 1240 && tg.rf[0] == 14 && in.n <= lim && ncell <= lim)
        return g.flag_next ? launch_quads<true, 88, 1240, 14>(a, P, ntiles, st)
                           : launch_quads<false, 88, 1240, 14>(a, P, ntiles, st);
    return g.flag_next ? launch_quads<true, 0, 0, 0>(a, P, ntiles, st)
                       : launch_quads<false, 0, 0, 0>(a, P, ntiles, st);
}

}  // namespace pic
