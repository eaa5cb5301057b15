// dss_lists.hpp -- windows of time steps on pair lists.
//
// Most pairs of one time step are the pairs of the next: the particles move by about 1e-3 of a
// radius per step.  dss_step therefore takes runs of steps as windows.  A window of n steps from
// a committed state is
//   k_list_begin          the pairs inside the cutoff plus a margin (skin) at the window's first
//                         state, with their stored stretches, and the first kick and drift (with
//                         size-class stencils k_list_search finds the pairs first);
//   k_list x n            one launch per step: the pair physics over the lists, the Stokes terms,
//                         the finishing kick and the next kick, drift and wrap; the last one writes
//                         the state, the force records and the sorted history rows (beside the
//                         committed ones) instead;
//   a counting sort       of the last state (k_predict's cell ids alone, k_scan, k_scatter, and
//                         k_history_move for the rows) over the committed one, which leaves the
//                         order, cells, rows and records of an ordinary step.  (A full step at the end instead cost 61 us
//                         against 47 at N = 100k, and 2.3 ms against 0.3 at N = 500k, size ratio 10.)
// The listed-pair test of every step is the FP64 one at the step's own positions: the list only
// holds more candidates than the test accepts, so the pair set, forces and history are those of a
// search at every step (up to the order of sums).
//
// Validity.  With A = 1 + gdot dt e_x e_y the separation of two particles (or of a particle and
// an image across the sheared faces) advances as r' = A r + d_j - d_i, d the displacement of a
// particle in the step beyond the ambient gdot y dt.  So after n steps, with g = gdot n dt and
// s+- = sqrt(1 + g^2 / 4) +- g / 2 the singular values of A^n,
//   |r_n| >= s- |r_0| - s+ (D_i + D_j),  D_i = sum_k |d_i,k|,
// and no pair outside the list is inside its cutoff while s- (rc + skin) - 2 s+ D >= rc for the
// largest cutoff rc of the box and every D.  Each particle's sum is kept beside its record (a
// maximum over the box instead, by an atomic of every workgroup on one word, took 50 of the 76 us
// of a step of 100k particles); a particle that finds the next step beyond the bound (or a list, a
// history row or a force out of range) sets a flag in
// the clock's error word, every later kernel of the stream's queue then returns at once, and the
// committed state at the window's start, which only the sort writes, is where the host resumes
// (dss_api.hip, settle).  (A history row may overflow in the last list step too, with the owners that
// the pairs had at the window's start where those of the step itself would fit.)  The searches, which set the flag too, run beside
// workgroups of their own launch that are still to start: one lane of a workgroup reads it, and after a
// barrier all go on or all return (read by each wavefront, some would leave and the others find the
// counters and queues in LDS unset, and take them for indices).
//
// Work split.  One workgroup per block of consecutive sorted slots (about one x-row of cells; the
// blocks of one box never span another).  It evaluates the pairs inside its block once and
// every pair that crosses its border on its own side, so a particle's force is complete in its
// workgroup's LDS and the integration follows in the same launch: no partner records (192 B per
// particle written and read back each step by the row tiles), no second launch.  A pair that
// crosses blocks is evaluated by both workgroups from the same inputs in the same orientation, so
// both hold the same stretch to the bit.
// Measured (FP64, a sheared box): N = 100k, 21 to 23 us per list step against 64 us for a full step
// (k_pairs 40, k_predict 9, k_scatter 6, k_scan 4, and their launches); N = 500k, 81 to 88 against
// 360 us; N = 1000, 6 against 27 us.
#pragma once

#include "dss_kernels.hpp"

namespace dss {

constexpr int kListBlock = 192;       // lanes of k_list: four workgroups per CU at up to 168 VGPRs
constexpr int kBeginBlock = 256;      // lanes of k_list_begin
constexpr int kBeginLanes = 8;        // lanes that take a run of candidates together
constexpr int kBeginRuns = 2;         // runs of a lane in flight
constexpr int kBeginRows = 1024;      // (particle, cell row) pairs of a batch of its search
constexpr int kListOwnMax = 128;      // particles of a block
constexpr int kListPerOwn = 24;       // list entries allotted per particle (more for a large one)
constexpr int kListSpare = 64;        // and per block
constexpr int kListCapMax = kListPerOwn * kListOwnMax + kListSpare;

// One particle in a window: (x, y, z, a), (u, box), (w, id); a neighbour gather is one 96-byte record.
struct ListRec {
    double4 p, v, w;
};

// A block of consecutive slots of one box (and of one size class); its list has room for cap
// entries from e0.
struct ListBlock {
    int start, n, box, cls, e0, cap;
};

// A list entry.  x: partner slot, kEntSwap when the partner is the pair's first member (the pair is
// evaluated in that orientation), kEntHas when a stretch is stored.  y: the own particle's index in
// the block, and for a pair inside the block the partner's (from bit 8) and kEntIn.
constexpr int kEntSlot = 0x1fffffff;
constexpr int kEntSwap = 0x20000000;
constexpr int kEntHas = 0x40000000;
constexpr int kEntIn = 0x40000000;
constexpr int kEntIdx = 0xff;
constexpr int kEntIdxBits = 8;
constexpr int kClasses = 5;  // contacts inside the block and across, listed pairs across and inside, margin

struct ListView {
    const ListBlock *blocks;
    int2 *ent;
    double *xi, *xr;      // 3 per entry; xr only with rolling resistance
    int *n;               // entries of each block
    const int *of;        // block of a slot (with size-class stencils)
    double *dsum;         // displacement sum D of the bound above, by slot
    // electro-chemical pairs beyond the lubrication list (ec_split): the partners of each slot
    // within their ranges plus the margin, far_cap per slot, and their force on it (3 per slot)
    int *far, *far_n;
    double *far_f;
    int far_cap;
    int *cross;           // y-face crossings of the window by slot
    int *x_used;          // whether the evaluation before the window used the atomic force record
    int own_cap;          // largest block
};

// The committed state of a handle, read by k_list_begin, and the state after the last list step, in the
// same slots (before the sort).
struct CommittedView {
    const double4 *pa, *vel, *omg;
    ForceBufs B;    // of the evaluation before the window
    double4 *pa_end, *vel_end, *omg_end;
    double *own_end;
};

// After a window that stopped: the flag and the lists' counts are cleared, and what follows runs.
__global__ void __launch_bounds__(kBeginBlock) k_list_resume(int nblock, int *__restrict__ n, DevClock *__restrict__ clk)
{
    const int k = blockIdx.x * kBeginBlock + threadIdx.x;
    if (k < nblock) n[k] = 0;
    if (k == 0) clk->err &= ~kErrListMask;
}

// Largest displacement sum of a particle with which the lists hold every pair after n steps.
__device__ __forceinline__ double list_budget(const DevParams &P, const BoxParams &G, double skin, int n)
{
    const double g = fabs(G.gd) * P.dt * (double)n;
    const double q = sqrt(1.0 + 0.25 * g * g);
    // largest cutoff; with ec_split that of the far pairs, whose lists have the same margin
    const double rc = P.ec_split ? 2.0 * G.amax + P.rext : pair_cutoff(P, 2.0 * G.amax);
    return ((q - 0.5 * g) * (rc + skin) - rc * (1.0 + 1e-12)) / (2.0 * (q + 0.5 * g));
}

// Periodic difference b - a of two cell coordinates in (-n/2, n/2], 0 for the ambiguous half.
__device__ __forceinline__ int cell_diff(int a, int b, int n)
{
    int d = b - a;
    if (2 * d > n) d -= n;
    if (2 * d < -n) d += n;
    return 2 * d == n || 2 * d == -n ? 0 : d;
}

// Whether i is the pair's first member, as in the pair kernels: with size-class stencils the larger
// one (of equal radii the later slot), else the one with j in its forward half shell (by the cell
// offsets along z, y, x, then by slot).  Antisymmetric, so both blocks of a pair agree.
__device__ __forceinline__ bool list_forward(const DevParams &P, const BoxParams &G, const double icw[3],
                                             const double4 &Xi, const double4 &Xj, int i, int j)
{
    if (P.sized) return Xj.w < Xi.w || (Xj.w == Xi.w && j < i);
    const int dz = cell_diff((int)(Xi.z * icw[2]), (int)(Xj.z * icw[2]), G.nc[2]);
    if (dz) return dz > 0;
    const int dy = cell_diff((int)(Xi.y * icw[1]), (int)(Xj.y * icw[1]), G.nc[1]);
    if (dy) return dy > 0;
    const int dx = cell_diff((int)(Xi.x * icw[0]), (int)(Xj.x * icw[0]), G.nc[0]);
    return dx ? dx > 0 : j > i;
}

// The cell rows around a particle: rows (cz + z0 .. , cy + y0 ..), ny x nz of them.  Where the reach
// spans more rows than the box has (small boxes), every row is taken once and along its whole
// length (whole).
struct ListRows {
    int ny, nz, y0, z0;
    bool whole;
};

__device__ __forceinline__ ListRows list_rows(const BoxParams &G, double reach)
{
    const int Ry = (int)ceil(reach / G.cw[1]), Rz = (int)ceil(reach / G.cw[2]);
    ListRows R;
    R.whole = 2 * Ry + 1 > G.nc[1] || 2 * Rz + 1 > G.nc[2] || 2.0 * reach + 2.0 * G.cw[0] > G.L[0];
    R.ny = R.whole ? G.nc[1] : 2 * Ry + 1;
    R.nz = R.whole ? G.nc[2] : 2 * Rz + 1;
    R.y0 = -Ry;
    R.z0 = -Rz;
    return R;
}

// A run of candidates of one particle of the block: slots jb .. jb + n, all with the same image
// (cross: y-face crossing, w: box lengths along x, z: box lengths along z; without `whole`).
// A run of kTaskMax slots or more is not searched: the lists are given up.
struct ListTask {
    int jb, code;
};
constexpr int kTaskMax = 0xffff;
__device__ __forceinline__ ListTask list_task(int jb, int n, int il, int cross, int w, int z)
{
    return {jb, min(n, kTaskMax) | (il << 16) | ((cross + 1) << 24) | ((z + 1) << 26) | ((w + 4) << 28)};
}

// Candidates of row (qy, qz) of the rows R around particle il at Xi: at most two runs.  A row
// farther than reach in y-z has none; a row reached across a y face is searched around the x
// shifted by the Lees-Edwards offset.  icw: 1 / cell widths; cell0: first cell of the lattice (of a
// size class).
template <typename Push>
__device__ __forceinline__ void list_row(const BoxParams &G, const double icw[3], double delta,
                                         const int *__restrict__ cell_start, const ListRows &R, int cell0,
                                         int il, const double4 &Xi, double reach, int qy, int qz, Push &&push)
{
    const int nxc = G.nc[0], nyc = G.nc[1], nzc = G.nc[2];
    if (R.whole) {
        const int base = cell0 + (qz * nyc + qy) * nxc;
        const int jb = cell_start[base], n = cell_start[base + nxc] - jb;
        if (n > 0) push(list_task(jb, n, il, 0, 0, 0));
        return;
    }
    // the margin of the window covers the rounding of these cell numbers too
    const int zu = (int)(Xi.z * icw[2]) + qz + R.z0, yu = (int)(Xi.y * icw[1]) + qy + R.y0;
    const double zlo = (double)zu * G.cw[2], ylo = (double)yu * G.cw[1];
    const double ez = fmax(0.0, fmax(zlo - Xi.z, Xi.z - (zlo + G.cw[2])));
    const double ey = fmax(0.0, fmax(ylo - Xi.y, Xi.y - (ylo + G.cw[1])));
    const double h2 = reach * reach - (ey * ey + ez * ez);
    if (h2 <= 0.0) return;
    const int cross = yu >= nyc ? 1 : (yu < 0 ? -1 : 0), cz = zu >= nzc ? 1 : (zu < 0 ? -1 : 0);
    // the window in x, wider by what FP32 rounds off the root
    const double xs = Xi.x - (cross > 0 ? delta : (cross < 0 ? -delta : 0.0));
    const double hw = (double)__builtin_sqrtf((float)h2) * (1.0 + 1e-6) + 1e-9 * G.L[0];
    int xl = (int)floor((xs - hw) * icw[0]);
    int span = (int)floor((xs + hw) * icw[0]) - xl + 1, w = 0;
    for (; xl < 0; xl += nxc) --w;
    for (; xl >= nxc; xl -= nxc) ++w;
    const int base = cell0 + ((zu - cz * nzc) * nyc + yu - cross * nyc) * nxc;
    const int len = min(span, nxc - xl);
    const int jb = cell_start[base + xl], n = cell_start[base + xl + len] - jb;
    if (n > 0) push(list_task(jb, n, il, cross, w, cz));
    if (span > len) {
        const int j2 = cell_start[base], n2 = cell_start[base + span - len] - j2;
        if (n2 > 0) push(list_task(j2, n2, il, cross, w + 1, cz));
    }
}

// Whether the workgroup of block K leaves a search: the window has stopped (err: the clock's word, that of
// the first lane decides), or a particle of the block is outside the box (a velocity of more than a box
// length per step, or none that is a number), whose cell numbers would be anything: the lists are
// given up.  A barrier.
__device__ __forceinline__ bool list_leave(const BoxParams &G, const ListBlock &K, const double4 *__restrict__ pa,
                                           unsigned err, DevClock *__restrict__ clk)
{
    const int t = threadIdx.x;
    bool out = false;
    if (t < K.n) {  // K.n <= kListOwnMax <= kBeginBlock
        const double4 X = pa[K.start + t];
        out = !(X.x >= 0.0 && X.x <= G.L[0] && X.y >= 0.0 && X.y <= G.L[1] && X.z >= 0.0 && X.z <= G.L[2]);
        if (out) atomicOr(&clk->err, kErrListFull);
    }
    return __syncthreads_or(out || (t == 0 && (err & kErrListMask)));
}

// The candidates of a block's particles among the cells from cell0 on (the box's, or a size
// class's), partners of radius up to amax: push(il, j, a_i, a_j) for every one inside its cutoff (Far:
// the electro-chemical ranges) plus the margin.  In batches of kBeginRows (particle, cell row) pairs the lanes write the candidate
// runs of their rows into LDS, then take the runs (so every lane has one, although most rows are
// out of reach): kBeginLanes lanes one run together (their loads are contiguous), kBeginRuns at a
// time (their loads are in flight together).  (One particle per eight lanes, each walking its
// share of the rows, took 73 us at N = 100k, k_list_begin takes 53 so.)
struct ListTasks {
    ListTask task[2 * kBeginRows];
    int n;
};

template <bool Far = false, typename Push>
__device__ __forceinline__ void list_collect(const DevParams &P, const BoxParams &G, double delta,
                                             const int *__restrict__ cell_start, const double4 *__restrict__ pa,
                                             const ListBlock &K, double own_amax, double amax, int cell0, ListTasks &T,
                                             DevClock *__restrict__ clk, Push &&push)
{
    const int t = threadIdx.x;
    // radius of the search for a pair of radius sum s
    auto reach = [&](double s) { return (Far ? s + P.rext : pair_cutoff(P, s)) + G.skin; };
    const ListRows R = list_rows(G, reach(own_amax + amax));
    const double icw[3] = {1.0 / G.cw[0], 1.0 / G.cw[1], 1.0 / G.cw[2]};
    // (particle, row) pairs numbered with a power of two of rows per particle
    int sh = 0;
    while ((1 << sh) < R.ny * R.nz) ++sh;
    const int all = K.n << sh;
    for (int k0 = 0; k0 < all; k0 += kBeginRows) {
        if (t == 0) T.n = 0;
        __syncthreads();
        for (int k = k0 + t; k < min(k0 + kBeginRows, all); k += kBeginBlock) {
            const int il = k >> sh, q = k & ((1 << sh) - 1), qz = q / R.ny, qy = q - qz * R.ny;
            if (qz >= R.nz) continue;
            const double4 Xi = pa[K.start + il];
            list_row(G, icw, delta, cell_start, R, cell0, il, Xi, reach(Xi.w + amax), qy, qz,
                     [&](const ListTask &a) { T.task[atomicAdd(&T.n, 1)] = a; });
        }
        __syncthreads();
        const int nt = T.n;
        const int sub = t & (kBeginLanes - 1);
        for (int k = t / kBeginLanes; k < nt; k += kBeginRuns * kBeginBlock / kBeginLanes) {
            int jb[kBeginRuns], n[kBeginRuns], il[kBeginRuns], most = 0;
            double sx[kBeginRuns], sy[kBeginRuns], sz[kBeginRuns], ai[kBeginRuns];
            double4 Y[kBeginRuns];
#pragma unroll
            for (int r = 0; r < kBeginRuns; ++r) {
                const int m = k + r * (kBeginBlock / kBeginLanes);
                const ListTask a = T.task[min(m, nt - 1)];
                const int cross = ((a.code >> 24) & 3) - 1, z = ((a.code >> 26) & 3) - 1, w = ((a.code >> 28) & 7) - 4;
                jb[r] = a.jb;
                n[r] = m < nt ? a.code & kTaskMax : 0;
                if (n[r] == kTaskMax) {
                    atomicOr(&clk->err, kErrListFull);
                    n[r] = 0;
                }
                il[r] = (a.code >> 16) & 0xff;
                const double4 X = pa[K.start + il[r]];
                sx[r] = X.x - ((double)cross * delta + (double)w * G.L[0]);
                sy[r] = X.y - (double)cross * G.L[1];
                sz[r] = X.z - (double)z * G.L[2];
                ai[r] = X.w;
                most = max(most, n[r]);
            }
            for (int j0 = sub; j0 < most; j0 += kBeginLanes) {
#pragma unroll
                for (int r = 0; r < kBeginRuns; ++r) Y[r] = pa[jb[r] + (j0 < n[r] ? j0 : 0)];
#pragma unroll
                for (int r = 0; r < kBeginRuns; ++r) {
                    double dx = Y[r].x - sx[r], dy = Y[r].y - sy[r], dz = Y[r].z - sz[r];
                    if (R.whole) min_image(G, delta, sx[r], sy[r], sz[r], Y[r].x, Y[r].y, Y[r].z, dx, dy, dz);
                    const double rl = reach(ai[r] + Y[r].w);
                    if (j0 < n[r] && jb[r] + j0 != K.start + il[r] && dx * dx + dy * dy + dz * dz < rl * rl)
                        push(il[r], jb[r] + j0, ai[r], Y[r].w);
                }
            }
        }
        __syncthreads();
    }
}

// ----------------------------------------------------------------------------------
// k_list_search (size-class stencils): the candidate pairs of one block, found by the pair's first
// member (the larger one, which scans the classes up to its own), appended as (partner, own index)
// to the lists of both members' blocks.  L.n counts them (zero at the window's start).
// ----------------------------------------------------------------------------------
__global__ void __launch_bounds__(kBeginBlock) k_list_search(DevParams P, const BoxParams *__restrict__ boxes,
                                                              const int *__restrict__ cell_start,
                                                              const double4 *__restrict__ pa, ListView L,
                                                              DevClock *__restrict__ clk)
{
    __shared__ ListTasks T;
    // the blocks of the largest particles, which scan most, first
    const ListBlock K = L.blocks[gridDim.x - 1 - blockIdx.x];
    const DevClock c0 = *clk;
    const BoxParams G = boxes[K.box];
    if (list_leave(G, K, pa, c0.err, clk)) return;
    const double delta = le_offset(P, G, c0.step);
    // largest radius of a class (with a margin for the rounding of its number)
    auto top = [&](int k) { return k == P.ncls - 1 ? G.amax : fmin(G.amax, (k + 1 - P.cls_add) / P.cls_mul * (1.0 + 1e-12)); };
    for (int k = 0; k <= K.cls; ++k)
        list_collect(P, G, delta, cell_start, pa, K, top(K.cls), top(k), k * (G.nc[0] * G.nc[1] * G.nc[2]), T, clk,
                     [&](int il, int j, double ai, double aj) {
                         const int i = K.start + il;
                         if (!(aj < ai || (aj == ai && j < i))) return;
                         const int bi = L.of[i], bj = L.of[j];
                         const int e = atomicAdd(&L.n[bi], 1);
                         if (e < K.cap) L.ent[K.e0 + e] = make_int2(j, il);
                         if (bj == bi) return;
                         const ListBlock Kj = L.blocks[bj];
                         const int f = atomicAdd(&L.n[bj], 1);
                         if (f < Kj.cap) L.ent[Kj.e0 + f] = make_int2(i, j - Kj.start);
                     });
}

// ----------------------------------------------------------------------------------
// k_list_begin: the lists of one block at the committed state, and the first kick and drift of
// the block's particles into the window's records.  The candidates (searched here, or with
// size-class stencils found by k_list_search) are queued in LDS; then all lanes take the queued
// ones: the pair's orientation and class (contacts, listed pairs, candidates of the margin, stored
// in this order, so that a wavefront of k_list holds one kind), a pair inside the block from its
// first member only, and the stored stretch from the committed history rows.
// ----------------------------------------------------------------------------------
template <bool Roll>
__global__ void __launch_bounds__(kBeginBlock) k_list_begin(DevParams P, const BoxParams *__restrict__ boxes,
                                                             const int *__restrict__ cell_start, CommittedView C,
                                                             HistView H, ListView L, ListRec *__restrict__ out,
                                                             int vel_is_half, DevClock *__restrict__ clk)
{
    extern __shared__ int2 q_lds[];
    __shared__ ListTasks T;
    __shared__ int qn, cnt[kClasses + 1], pos[kClasses];
    const int t = threadIdx.x;
    const int blk = xcd_row(blockIdx.x, gridDim.x);
    const ListBlock K = L.blocks[blk];
    const DevClock c0 = *clk;
    const BoxParams G = boxes[K.box];
    const int cap = K.cap;
    const double skin = G.skin;
    if (t <= kClasses) cnt[t] = 0;
    if (t == 0) qn = P.sized ? L.n[blk] : 0;
    const double delta = le_offset(P, G, c0.step);
    const double icw[3] = {1.0 / G.cw[0], 1.0 / G.cw[1], 1.0 / G.cw[2]};
    if (list_leave(G, K, C.pa, c0.err, clk)) return;
    if (P.sized) {
        for (int k = t; k < min(qn, cap); k += kBeginBlock) q_lds[k] = L.ent[K.e0 + k];
    } else {
        list_collect(P, G, delta, cell_start, C.pa, K, G.amax, G.amax, G.cell_off, T, clk,
                     [&](int il, int j, double, double) {
                         const int e = atomicAdd(&qn, 1);
                         if (e < cap) q_lds[e] = make_int2(j, il);
                     });
    }
    if (t < K.n) {
        const int i = K.start + t;
        double4 X = C.pa[i], V = C.vel[i], W = C.omg[i];
        double f[6];
        total_ft(C.B, i, f, c0.deferred || P.ec_split);
        int cross = 0;
        const double d = sqrt(advance_particle(P, G, X, V, W, f, vel_is_half != 0, clk->step + 1, cross));
        out[i].p = X;
        out[i].v = V;
        out[i].w = W;
        L.cross[i] = cross;
        L.dsum[i] = d;
        if (!(d <= list_budget(P, G, skin, 1))) atomicOr(&clk->err, kErrListStop);
    }
    __syncthreads();
    const int total = qn;
    if (total > cap) {
        if (t == 0) atomicOr(&clk->err, kErrListFull);
        return;
    }
    for (int k = t; k < total; k += kBeginBlock) {
        int2 e = q_lds[k];
        const int i = K.start + e.y, j = e.x, jl = j - K.start;
        const double4 Xi = C.pa[i], Xj = C.pa[j];
        double dx, dy, dz;
        min_image(G, delta, Xi.x, Xi.y, Xi.z, Xj.x, Xj.y, Xj.z, dx, dy, dz);
        const double r2 = dx * dx + dy * dy + dz * dz, s = Xi.w + Xj.w, rc = pair_cutoff(P, s);
        const bool fwd = list_forward(P, G, icw, Xi, Xj, i, j), in = jl >= 0 && jl < K.n;
        const int cls = in && !fwd ? kClasses : (r2 < s * s * (1.0 + 1e-9) ? (in ? 0 : 1) : (r2 < rc * rc ? (in ? 3 : 2) : 4));
        atomicAdd(&cnt[cls], 1);
        q_lds[k] = make_int2(j | (fwd ? 0 : kEntSwap),
                             e.y | (in ? (jl << kEntIdxBits) | kEntIn : 0) | (cls << (2 * kEntIdxBits)));
    }
    __syncthreads();
    if (t == 0) {
        int n = 0;
        for (int c = 0; c < kClasses; ++c) {
            pos[c] = n;
            n += cnt[c];
        }
        L.n[blk] = n;
    }
    __syncthreads();
    for (int k = t; k < total; k += kBeginBlock) {
        int2 e = q_lds[k];
        const int cls = (e.y >> (2 * kEntIdxBits)) & 7;
        if (cls == kClasses) continue;
        const int slot = K.e0 + atomicAdd(&pos[cls], 1);
        e.y &= ~(7 << (2 * kEntIdxBits));
        const int i = K.start + (e.y & kEntIdx), j = e.x & kEntSlot;
        const int a = (e.x & kEntSwap) ? j : i, b = (e.x & kEntSwap) ? i : j;
        const int ida = (int)C.omg[a].w, idb = (int)C.omg[b].w;
        double x[3], y[3] = {0.0, 0.0, 0.0};
        // only a pair in contact at the committed state has a stored stretch (the host does not begin
        // a window when the offset was changed after that step); the class is by r^2, the rows
        // hold those with sqrt(r^2) - a_i - a_j < 0
        if (cls < 2 && (row_find(H.key_old, H.xi_old, H.cnt_old, P.M, a, idb, x, Roll ? H.xr_old : nullptr, y) ||
            row_find(H.key_old, H.xi_old, H.cnt_old, P.M, b, ida, x, Roll ? H.xr_old : nullptr, y))) {
            const double sg = ida > idb ? -1.0 : 1.0;  // stored from the smaller id to the larger
            e.x |= kEntHas;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                L.xi[3LL * slot + c] = sg * x[c];
                if constexpr (Roll) L.xr[3LL * slot + c] = y[c];
            }
        }
        L.ent[slot] = e;
    }
}

// ----------------------------------------------------------------------------------
// k_list_far_begin: with the electro-chemical far pairs on a pass of their own (ec_split), the
// partners of each particle of a block within their ranges plus the margin (the lubrication list's
// among them: the step's test tells).
// ----------------------------------------------------------------------------------
__global__ void __launch_bounds__(kBeginBlock) k_list_far_begin(DevParams P, const BoxParams *__restrict__ boxes,
                                                                 const int *__restrict__ cell_start,
                                                                 const double4 *__restrict__ pa, ListView L,
                                                                 DevClock *__restrict__ clk)
{
    __shared__ ListTasks T;
    __shared__ int cnt[kListOwnMax];
    const int t = threadIdx.x;
    const ListBlock K = L.blocks[xcd_row(blockIdx.x, gridDim.x)];
    const DevClock c0 = *clk;
    const BoxParams G = boxes[K.box];
    if (t < kListOwnMax) cnt[t] = 0;
    if (list_leave(G, K, pa, c0.err, clk)) return;
    list_collect<true>(P, G, le_offset(P, G, c0.step), cell_start, pa, K, G.amax, G.amax, G.cell_off, T, clk,
                       [&](int il, int j, double, double) {
                           const int e = atomicAdd(&cnt[il], 1);
                           if (e < L.far_cap) L.far[(long long)(K.start + il) * L.far_cap + e] = j;
                       });
    if (t < K.n) {
        L.far_n[K.start + t] = min(cnt[t], L.far_cap);
        if (cnt[t] > L.far_cap) atomicOr(&clk->err, kErrListFull);
    }
}

// ----------------------------------------------------------------------------------
// k_list_far: the force of the electro-chemical far pairs on every particle at step n of a window,
// as k_pairs_ec takes it (the same FP64 distance and ranges, gathered from both sides, no atomics)
// over the far lists: kEcLanes lanes share a particle, kEcChunk partners of a lane in flight.
// The search of k_pairs_ec tests about 500 candidates per particle, a list holds about 100: 315 us
// per step at N = 100k with attraction, 68 us so, plus 145 us per window for the lists.
// ----------------------------------------------------------------------------------
template <bool Sum>
__global__ void __launch_bounds__(kBlock) k_list_far(DevParams P, BoxParams G, ListView L,
                                                      const ListRec *__restrict__ in, int n,
                                                      const DevClock *__restrict__ clk, double *__restrict__ partials,
                                                      int pstride, int rec0)
{
    __shared__ double red[kBlock / 64][12];
    const int t = threadIdx.x;
    const int sub = t & (kEcLanes - 1);
    const int i = (xcd_row(blockIdx.x, gridDim.x) * kBlock + t) / kEcLanes;
    const DevClock c0 = *clk;
    if (c0.err & kErrListMask) return;
    const bool on = i < P.N;
    const int nf = on ? L.far_n[i] : 0;
    const double4 Xi = in[on ? i : 0].p;
    const double delta = le_offset(P, G, c0.step + n);
    PairTally tally;
#pragma unroll
    for (int k = 0; k < 9; ++k) tally.S[k] = 0.0;
    tally.npair = tally.ncont = 0;
    tally.fill = 0;
    double f[3] = {0.0, 0.0, 0.0};
    const int *const list = L.far + (long long)(on ? i : 0) * L.far_cap;
    for (int e0 = sub; e0 < nf; e0 += kEcLanes * kEcChunk) {
        int j[kEcChunk];
        double4 X[kEcChunk];
#pragma unroll
        for (int u = 0; u < kEcChunk; ++u) j[u] = list[e0 + u * kEcLanes < nf ? e0 + u * kEcLanes : sub];
#pragma unroll
        for (int u = 0; u < kEcChunk; ++u) X[u] = in[j[u]].p;
#pragma unroll
        for (int u = 0; u < kEcChunk; ++u) {
            double dx, dy, dz, r2, rl, re;
            min_image(G, delta, Xi.x, Xi.y, Xi.z, X[u].x, X[u].y, X[u].z, dx, dy, dz);
            const double s = Xi.w + X[u].w;
            {
#pragma clang fp contract(off)
                r2 = (dx * dx + dy * dy) + dz * dz;
                rl = P.cf * s;
                re = s + P.rext;
            }
            if (!(e0 + u * kEcLanes < nf) || r2 < rl * rl || !(r2 < re * re)) continue;
            const double dist = sqrt(r2);
            const double g = ec_far_force(P, dist, Xi.w, X[u].w) * rcp_nr(dist);
            const double F[3] = {g * dx, g * dy, g * dz};
#pragma unroll
            for (int c = 0; c < 3; ++c) f[c] += F[c];
            if constexpr (Sum) {
                const double r[3] = {dx, dy, dz};
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int c = 0; c < 3; ++c) tally.S[3 * a + c] += 0.5 * r[a] * F[c];
                if (i < j[u]) ++tally.npair;
            }
        }
    }
#pragma unroll
    for (int o = 1; o < kEcLanes; o <<= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) f[c] += __shfl_xor(f[c], o, 64);
    if (on && sub < 3) L.far_f[3LL * i + sub] = sub == 0 ? f[0] : (sub == 1 ? f[1] : f[2]);
    if constexpr (Sum) reduce_tally(tally, red, partials, pstride, rec0 + blockIdx.x);
}

// ----------------------------------------------------------------------------------
// k_list: time step n of the window (1 .. length) of one block: the listed pairs at the records
// `in` (the physics and history of the pair kernels), the Stokes terms, then the finishing kick
// and the next step's kick, drift and wrap into `out`; with Last, instead, the state, the force
// record and the sorted history rows of the step go to the buffers that the sort reads.  Sum: the block's stress and
// counters go to its partial record.
// Bound by FP64 issue and by the latency of the partner gathers: three wavefronts per workgroup
// and four workgroups per CU keep twelve wavefronts per CU in flight (the register file's limit
// at 168 VGPRs; sixteen, at 128, take 24.9 us instead of 23.1 at N = 100k and 112 instead of 96 at
// N = 500k by events, and partners loaded straight into LDS a round ahead 26.2).
// ----------------------------------------------------------------------------------
template <typename Real, bool Roll, bool Sum, bool Last>
__global__ void __launch_bounds__(kListBlock, 3) k_list(DevParams P, const BoxParams *__restrict__ boxes,
                                                         BoxParams G0, ListView L, const ListRec *__restrict__ in,
                                                         ListRec *__restrict__ out, int n, CommittedView C, HistView H,
                                                         DevClock *__restrict__ clk, double *__restrict__ partials,
                                                         int pstride)
{
    extern __shared__ double4 list_lds[];
    // the block's records, 6 accumulators per particle, contact counts
    ListRec *const rec = reinterpret_cast<ListRec *>(list_lds);
    double *const acc = reinterpret_cast<double *>(rec + L.own_cap);
    int *const cnt = reinterpret_cast<int *>(acc + 6 * L.own_cap);
    __shared__ double red[kListBlock / 64][12];
    __shared__ unsigned stop;  // with Last
    const int t = threadIdx.x;
    const int blk = xcd_row(blockIdx.x, gridDim.x);
    // everything the block's number leads to is requested before the first use
    const ListBlock K = L.blocks[blk];
    const int ne = L.n[blk];
    const DevClock c0 = *clk;
    // by wavefronts: another workgroup may set the flag meanwhile, and what is left of this one then
    // works on records and counts that nobody has set.  Without Last its indices all come from the lists,
    // and what it writes belongs to a window that is given up (decided by the workgroup behind
    // the barrier below, the N = 100k step took 1.4 % more); with Last the counts are indices.
    if constexpr (Last) {
        if (t == 0) stop = c0.err & kErrListMask;
    } else {
        if (c0.err & kErrListMask) return;
    }
    const BoxParams G = P.nbox > 1 ? boxes[K.box] : G0;
    {
        const double2 *const src = reinterpret_cast<const double2 *>(in + K.start);
        double2 *const dst = reinterpret_cast<double2 *>(rec);
        for (int k = t; k < 6 * K.n; k += kListBlock) {
            dst[k] = src[k];
            acc[k] = 0.0;
        }
        for (int k = t; k < K.n; k += kListBlock) cnt[k] = 0;
    }
    const double delta = le_offset(P, G, c0.step + n);
    PairTally tally;
#pragma unroll
    for (int k = 0; k < 9; ++k) tally.S[k] = 0.0;
    tally.npair = tally.ncont = 0;
    tally.fill = 0;
    bool bad = false;
    __syncthreads();
    if constexpr (Last) {
        if (stop) return;
    }
    // the entry of the lane's next round is requested a round ahead, and the stretch with the
    // records: one memory latency per round instead of three
    int2 next = t < ne ? L.ent[K.e0 + t] : make_int2(0, 0);
    for (int k = t; k < ne; k += kListBlock) {
        const int2 e = next;
        if (k + kListBlock < ne) next = L.ent[K.e0 + k + kListBlock];
        const int il = e.y & kEntIdx, jl = (e.y >> kEntIdxBits) & kEntIdx;
        const bool swap = (e.x & kEntSwap) != 0, has = (e.x & kEntHas) != 0, inside = (e.y & kEntIn) != 0;
        const int own = K.start + il;
        ListRec A, B = rec[il];
        if (inside)
            A = rec[jl];
        else
            A = in[e.x & kEntSlot];
        const double4 Xi = swap ? A.p : B.p, Xj = swap ? B.p : A.p;
        const double4 Vi = swap ? A.v : B.v, Vj = swap ? B.v : A.v;
        const double4 Wi = swap ? A.w : B.w, Wj = swap ? B.w : A.w;
        double xo[3] = {0.0, 0.0, 0.0}, xro[3] = {0.0, 0.0, 0.0};
        double *const xs = L.xi + 3LL * (K.e0 + k);
        if (has) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                xo[c] = xs[c];
                if constexpr (Roll) xro[c] = L.xr[3LL * (K.e0 + k) + c];
            }
        }
        double dx, dy, dz, r2;
        min_image(G, delta, Xi.x, Xi.y, Xi.z, Xj.x, Xj.y, Xj.z, dx, dy, dz);
        const bool on = listed(P, dx, dy, dz, Xi.w, Xj.w, r2);
        const double dist = sqrt(r2);
        const bool touch = on && dist - Xi.w - Xj.w < 0.0;
        if (has != touch) L.ent[K.e0 + k].x = e.x ^ kEntHas;  // the stretch is dropped, or begins at zero
        if (!on) continue;
        PairOut o;
        double S[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        pair_physics<Real, Roll, false, true>(P, G.gd, G.wk, dx, dy, dz, dist, Xi.w, Xj.w, Xi.y, Xj.y, Vi, Vj, Wi, Wj,
                                              xo, xro, S, o, P.sized && size_class(P, Xi.w) >= P.wave_cls);
        double *const a = acc + 6 * il;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            atomicAdd(a + c, swap ? -o.Fi[c] : o.Fi[c]);
            atomicAdd(a + 3 + c, swap ? o.Tj[c] : o.Ti[c]);
        }
        if (inside) {
            double *const b = acc + 6 * jl;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                atomicAdd(b + c, -o.Fi[c]);
                atomicAdd(b + 3 + c, o.Tj[c]);
            }
        }
        if (!swap) {
            // the pair's first member counts it, holds its history row entry and its stress
            ++tally.npair;
            if constexpr (Sum) {
#pragma unroll
                for (int c = 0; c < 9; ++c) tally.S[c] += S[c];
            }
        }
        if (o.contact) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                xs[c] = o.xi[c];
                if constexpr (Roll) L.xr[3LL * (K.e0 + k) + c] = o.xr[c];
            }
            if (!swap) {
                ++tally.ncont;
                const int slot = atomicAdd(&cnt[il], 1);
                bad = bad || slot >= P.M;  // the row would overflow: a full step reports it, if it does there
                if constexpr (Last)
                    if (slot < P.M) store_history<Roll>(H, P.M, own, slot, (int)Wi.w, (int)Wj.w, o, clk);
            }
        }
    }
    if constexpr (Sum) reduce_sums(tally, red, partials, pstride, blk);
    __syncthreads();
    for (int il = t; il < K.n; il += kListBlock) {
        const int i = K.start + il;
        double4 X = rec[il].p, V = rec[il].v, W = rec[il].w;
        double f[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) f[c] = acc[6 * il + c];
        stokes_terms<false>(P, G, X, V, W, f, nullptr);
        if (P.ec_split) {
#pragma unroll
            for (int c = 0; c < 3; ++c) f[c] += L.far_f[3LL * i + c];
        }
        tally.fill = max(tally.fill, cnt[il]);
        if constexpr (Last) {
            C.pa_end[i] = X;
            C.vel_end[i] = V;
            C.omg_end[i] = W;
            store_ft(C.own_end + 6LL * i, f);
            if (!finite6(f)) atomicOr(&clk->err, kErrNonFinite);
            finish_row<Roll>(H, P.M, i, cnt[il], (int)W.w);
        } else {
            int cross = 0;
            const double d = L.dsum[i] + sqrt(advance_particle(P, G, X, V, W, f, true, c0.step + n + 1, cross));
            bad = bad || !finite6(f) || !(d <= list_budget(P, G, G.skin, n + 1));
            L.dsum[i] = d;
            if (cross) L.cross[i] += cross;
            out[i].p = X;
            out[i].v = V;
            out[i].w = W;
        }
    }
    if constexpr (Sum) reduce_fill(tally.fill, red, partials, pstride, blk);
    if (bad) atomicOr(&clk->err, kErrListStop);
    if constexpr (Last) {
        if (t == 0) {
            L.n[blk] = 0;  // of the next window's search (every lane has read its count)
            if (blk == 0) *L.x_used = c0.deferred || P.ec_split ? 1 : 0;
        }
    }
}

}  // namespace dss
