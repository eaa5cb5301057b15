// On-device observables of Sec. 3 (the quantities behind the paper's figures of the
// rheology and microstructure):
//   - shear-wise diffusivity, eq. (diffY): D_y = <[y(t) - y(t0)]^2> / (2 (t - t0) a0^2 gdot),
//     with y unwrapped across the sheared y faces (the wrap in k_predict counts the crossings
//     of each particle);
//   - autocorrelation of the shear-wise velocity fluctuations, eq. (corrV):
//     C_v = <v'(t) v'(t0)> / <v'(t)^2>, v' = u_y (the ambient shear has no y component);
//   - local volume fraction along y by size group (Fig. localPhi): the volume of every sphere
//     inside each slab [k dy, (k+1) dy) of the periodic y axis, over the slab volume;
//   - clusters of contacting particles (Fig. histo): connected components of the graph of the
//     committed contacts (d_ij < 0), as a histogram of cluster sizes.
#pragma once

#include "dss_kernels.hpp"

namespace dss {

// Reference of the diffusivity and the velocity correlation: unwrapped y and v' by id.
__global__ void __launch_bounds__(kBlock) k_obs_ref(int N, double Ly, const double *__restrict__ x,
                                                     const double *__restrict__ u, const int *__restrict__ img,
                                                     double *__restrict__ y0, double *__restrict__ v0)
{
#pragma clang fp contract(off)
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= N) return;
    y0[id] = x[3 * id + 1] + (double)img[id] * Ly;
    v0[id] = u[3 * id + 1];
}

// Per-workgroup sums of [y_unwrapped(t) - y0]^2, v'(t) v'(t0), v'(t)^2 (3 x gridDim records).
__global__ void __launch_bounds__(kBlock) k_obs_sums(int N, double Ly, const double *__restrict__ x,
                                                      const double *__restrict__ u, const int *__restrict__ img,
                                                      const double *__restrict__ y0, const double *__restrict__ v0,
                                                      double *__restrict__ part)
{
#pragma clang fp contract(off)
    __shared__ double red[kBlock / 64][3];
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    if (id < N) {
        const double dy = (x[3 * id + 1] + (double)img[id] * Ly) - y0[id];
        const double v = u[3 * id + 1];
        s[0] = dy * dy;
        s[1] = v * v0[id];
        s[2] = v * v;
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double t = warp_sum(s[k]);
        if (lane == 0) red[wid][k] = t;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t += red[w][threadIdx.x];
        part[3 * blockIdx.x + threadIdx.x] = t;
    }
}

// Volume of the sphere of radius a centred at 0 between heights z1 < z2 (a slab of the sphere):
// pi [a^2 z - z^3 / 3] over [max(z1, -a), min(z2, a)].
__device__ __forceinline__ double sphere_slab(double a, double z1, double z2)
{
    const double lo = fmax(z1, -a), hi = fmin(z2, a);
    if (!(hi > lo)) return 0.0;
    return kPi * ((a * a * hi - hi * hi * hi / 3.0) - (a * a * lo - lo * lo * lo / 3.0));
}

// Local volume fraction along y: per-workgroup partial profiles (group 0: a <= a_split,
// group 1: a > a_split), nb bins each, accumulated in LDS; part[blockIdx][2 nb].  The
// workgroups stride over the particles (one particle per lane when the grid covers N).
__global__ void __launch_bounds__(kBlock) k_phi_profile(int N, double Ly, int nb, double a_split,
                                                         const double4 *__restrict__ pa, double *__restrict__ part)
{
    extern __shared__ double hist[];  // 2 nb
    for (int k = threadIdx.x; k < 2 * nb; k += kBlock) hist[k] = 0.0;
    __syncthreads();
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < N; p += gridDim.x * blockDim.x) {
        const double4 X = pa[p];
        const double dy = Ly / (double)nb;
        const int g = X.w > a_split ? 1 : 0;
        // in no slab: a height that no slab number holds (the loop would not end)
        if (fabs(X.y) > 1.0e5 * Ly) continue;
        // slabs touched by [y - a, y + a), unwrapped bin indices, periodic in y
        const int b0 = (int)floor((X.y - X.w) / dy), b1 = (int)floor((X.y + X.w) / dy);
        for (int b = b0; b <= b1; ++b) {
            const double v = sphere_slab(X.w, (double)b * dy - X.y, (double)(b + 1) * dy - X.y);
            const int bw = ((b % nb) + nb) % nb;
            atomicAdd(&hist[g * nb + bw], v);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < 2 * nb; k += kBlock) part[(long long)blockIdx.x * 2 * nb + k] = hist[k];
}

// Sum of the nw partial profiles of k_phi_profile: out[k] = sum_b part[b][k], k < m = 2 nb, one
// wavefront per k, its lanes over the workgroups, in a fixed order (one lane per k, adding 391
// partials one after the other, took 94 us at N = 100k; 4.6 us so).
__global__ void __launch_bounds__(kBlock) k_phi_reduce(const double *__restrict__ part, int nw, int m,
                                                        double *__restrict__ out)
{
    const int k = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (k >= m) return;
    double t = 0.0;
    for (int b = lane; b < nw; b += 64) t += part[(long long)b * m + k];
    t = warp_sum(t);
    if (lane == 0) out[k] = t;
}

// Connected components of the contact graph by lock-free union-find over particle ids.
// parent[v] <= v at all times (a root is hooked under a smaller root only), so every find
// walks a strictly decreasing chain and ends.  The find splits the path it walks: each
// visited node is pointed at its grandparent, which is still an ancestor no larger than it,
// and only non-roots are written (hooks change roots only, by compare-and-swap), so the
// invariant holds under concurrent finds and hooks while chains stay short.
// The loads and stores of a find are of workgroup scope, from the XCD's own L2 (at system scope
// each went to memory: k_cc_hook alone 632 us at N = 100k, 270 us so): a parent read late is an
// older ancestor, which serves as well, and a root read late fails the compare-and-swap, whose
// answer is where the next find begins.
__device__ __forceinline__ int cc_find(int *parent, int v)
{
    int cur = __hip_atomic_load(&parent[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (cur == v) return v;
    int prev = v;
    for (;;) {
        const int next = __hip_atomic_load(&parent[cur], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (next == cur) return cur;
        __hip_atomic_store(&parent[prev], next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        prev = cur;
        cur = next;
    }
}

// base[idx] += the number of active lanes of the wavefront with that idx, one atomic per
// distinct idx.
template <typename T>
__device__ __forceinline__ void cc_add_grouped(T *base, long long idx, bool active)
{
    const int lane = threadIdx.x & 63;
    unsigned long long todo = __ballot(active);
    while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const long long v = __shfl(idx, leader, 64);
        const unsigned long long same = __ballot(active && idx == v);
        if (lane == leader) atomicAdd(&base[v], (T)__popcll(same));
        todo &= ~same;
    }
}

__global__ void __launch_bounds__(kBlock) k_cc_init(int N, int *__restrict__ parent, int *__restrict__ size)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    parent[v] = v;
    size[v] = 0;
}

// The larger of the parents of every contact's particles goes under the smaller, by a plain store:
// of several stores to one parent any may stay, since each is a smaller member of the same
// cluster, and the links that were lost are made by the next pass or by k_cc_hook, which joins
// the particles of every contact.  With k_cc_flatten after each, kLowerPasses passes leave
// k_cc_hook little to join (random spheres of mean coordination 4.5: 82 000, 33 000, 16 000, 7 500
// and 0 of 225 000 contacts are left between trees after 1 .. 5 passes), and so none of its
// compare-and-swaps of many lanes on the root of the largest cluster: 53 us of passes and 8 us of
// k_cc_hook at N = 100k, where k_cc_hook alone took 270 us (the passes by atomicMin: 118 us).
constexpr int kLowerPasses = 5;

__global__ void __launch_bounds__(kBlock) k_cc_lower(int N, int M, const int *__restrict__ own,
                                                      const int *__restrict__ key, const int *__restrict__ cnt,
                                                      int *parent)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int a = own[p];
    const int n = cnt[p];
    const int ra = __hip_atomic_load(&parent[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (int k = 0; k < n; ++k) {
        const int b = key[(long long)p * M + k] & kKeyMask;
        const int rb = __hip_atomic_load(&parent[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int lo = ra < rb ? ra : rb, hi = ra < rb ? rb : ra;
        if (lo != hi && __hip_atomic_load(&parent[hi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > lo)
            __hip_atomic_store(&parent[hi], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Every particle under its root.
__global__ void __launch_bounds__(kBlock) k_cc_flatten(int N, int *parent)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const int root = cc_find(parent, v);
    __hip_atomic_store(&parent[v], root, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Every committed contact (row owner own[p], partner key) joins its two particles.
__global__ void __launch_bounds__(kBlock) k_cc_hook(int N, int M, const int *__restrict__ own,
                                                     const int *__restrict__ key, const int *__restrict__ cnt,
                                                     int *parent)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int a = own[p];
    const int n = cnt[p];
    for (int k = 0; k < n; ++k) {
        const int b = key[(long long)p * M + k] & kKeyMask;
        int ra = cc_find(parent, a), rb = cc_find(parent, b);
        while (ra != rb) {
            const int lo = ra < rb ? ra : rb, hi = ra < rb ? rb : ra;
            const int was = atomicCAS(&parent[hi], hi, lo);
            if (was == hi) break;
            ra = cc_find(parent, lo);
            rb = cc_find(parent, was);  // was < hi
        }
    }
}

// Cluster sizes: size[root] = particles under root.  A cluster that spans the box holds most
// lanes of every workgroup: the lanes under the first lane's root are counted by the workgroup (one
// atomic for all), the others by their wavefront (one atomic per lane on one word: 1023 us at
// N = 100k with a cluster of 95 000, 7 us so).
__global__ void __launch_bounds__(kBlock) k_cc_count(int N, int *parent, int *__restrict__ size)
{
    __shared__ int first;
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    const bool on = v < N;
    const int root = on ? cc_find(parent, v) : -1;
    if (threadIdx.x == 0) first = root;
    __syncthreads();
    const int f = first;
    const int n = __syncthreads_count(root == f);
    if (threadIdx.x == 0) atomicAdd(&size[f], n);
    cc_add_grouped(size, root, on && root != f);
}

// Histogram of cluster sizes: hist[s - 1] += 1 for every root of size s (s > cap counts in
// hist[cap - 1]).
__global__ void __launch_bounds__(kBlock) k_cc_hist(int N, const int *parent, const int *__restrict__ size,
                                                     long long cap, unsigned long long *__restrict__ hist)
{
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    const bool root = v < N && parent[v] == v;
    const long long s = root ? size[v] : 1;
    const int ones = __syncthreads_count(root && s == 1);  // one atomic of the workgroup for these
    if (threadIdx.x == 0 && ones) atomicAdd(&hist[0], (unsigned long long)ones);
    cc_add_grouped(hist, (s < cap ? s : cap) - 1, root && s != 1);
}

}  // namespace dss
