// Soft-sphere compression packing of the sample (Simulations section: the
// active medium fills the voids of a granular packing of spheres obtained by
// molecular dynamics).  Read as a compression run of soft spheres in a closed
// box in the dissipative (overdamped) limit of granular dynamics:
//
//   at scale s the spheres have diameters s d_i and the energy is
//     U_s = 1/2 sum_{i<j} (s (d_i + d_j)/2 - |x_i - x_j|)_+^2
//         + 1/2 sum_i sum_a [(s d_i/2 - x_ia)_+^2 + (x_ia + s d_i/2 - L_a)_+^2];
//   one step moves every centre along its force at once, x_i += eta F_i with
//   F_i = -grad_i U_s; s grows from s0 to 1 in `stages` equal steps with
//   `iters` steps at each scale below 1 and `final_iters` steps at s = 1.
//
// Only spheres closer than the largest diameter interact, so the box is cut
// into cells at least that wide and a sphere looks at the 27 cells around its
// own.  The centres sit in per-cell lists (one atomic slot each, at most
// kPackCap per cell, in no order).  A step gives each sphere 32 lanes of a wave,
// one per neighbour cell: a lane adds the forces of its cell's spheres in
// sphere order, the lanes' sums are combined by a butterfly of fixed shape, and
// the first lane adds the walls, writes the new centre and bins it into the
// next cell table.  Every run of the same input therefore gives the same bits.
// A step is one launch: the lists of 320^3's 7200 spheres hold one or two
// centres, so a lane orders them itself as it reads them, where a launch of its
// own to sort them took 4.9 us of a step's 13.8; and the counts rotate through
// three buffers, one read, one filled, one cleared for the step after.  Every
// thread clears a count while there are no more of them; in a box of more cells
// (32 a sphere) a step clears those of the centres of two steps ago, whose
// records it is about to overwrite (8 spheres in 160^3 cells: 407 us a step when
// every count was cleared, 3 now; 7200 in 25^3: 8.6 by threads, 8.8 by
// centres).  What
// bounds a step then is the chain centre - count and list - neighbours - sum -
// new list entry, so the counts and the first eight entries are read together
// and their centres together (9.4 us before, 8.5 now).  Centres and diameters travel together
// as one 32-byte record (x, y, z, d), ping-ponged between two buffers.  FP64
// throughout.
#pragma once

#include "mbf_kernels.hpp"

namespace mbf {

constexpr int kPackCap = 32;        // centres one cell may hold
constexpr int kPackLanes = 32;      // lanes per sphere in the step (27 neighbour cells)
constexpr int kPackThreads = 256;   // 8 spheres per workgroup of the step
constexpr int kPackMaxCells = 1 << 24;

struct PackGrid {
    int g[3];          // cells per axis
    double w[3];       // cell widths, each at least the largest diameter
    double box[3];     // box edges L_a
    int ncell;
};

// Cell of one coordinate: floor(x / w) clamped to [0, g-1] (NaN -> 0).  The
// clamp keeps two centres closer than w at most one cell apart, so centres
// pushed slightly through a wall still find all their contacts.
__device__ __forceinline__ int pack_axis(double x, double w, int g) {
    const double q = x / w;
    if (!(q >= 1.0)) return 0;
    return (int)fmin(q, (double)(g - 1));
}

__device__ __forceinline__ int pack_cell(const PackGrid& gr, double4 p, int& cx, int& cy, int& cz) {
    cx = pack_axis(p.x, gr.w[0], gr.g[0]);
    cy = pack_axis(p.y, gr.w[1], gr.g[1]);
    cz = pack_axis(p.z, gr.w[2], gr.g[2]);
    return (cz * gr.g[1] + cy) * gr.g[0] + cx;
}

// Initial records from the caller's centres (n x 3) and diameters; all counts
// cleared.
__global__ void __launch_bounds__(256) k_pack_load(const double* __restrict__ x, const double* __restrict__ d, int n,
                                                   double4* __restrict__ P, int* __restrict__ cnts, int ncnts) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    for (int c = i; c < ncnts; c += gridDim.x * 256) cnts[c] = 0;
    if (i >= n) return;
    P[i] = make_double4(x[3 * i], x[3 * i + 1], x[3 * i + 2], d[i]);
}

__global__ void __launch_bounds__(64) k_pack_clear_flag(int* __restrict__ flag) {
    if (threadIdx.x == 0) flag[0] = 0;
}

__global__ void __launch_bounds__(256) k_pack_store(const double4* __restrict__ P, int n, double* __restrict__ x) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double4 p = P[i];
    x[3 * i] = p.x;
    x[3 * i + 1] = p.y;
    x[3 * i + 2] = p.z;
}

// One slot per sphere in its cell; a cell that would hold more than kPackCap
// centres raises *flag (sticky) and drops the extra ones.
__global__ void __launch_bounds__(256) k_pack_bin(const double4* __restrict__ P, int n, PackGrid gr,
                                                  int* __restrict__ cnt, int* __restrict__ lst, int* __restrict__ flag) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    int cx, cy, cz;
    const int c = pack_cell(gr, P[i], cx, cy, cz);
    const int slot = atomicAdd(cnt + c, 1);
    if (slot < kPackCap) lst[c * kPackCap + slot] = i;
    else atomicOr(flag, 1);
}

// Each cell's list in ascending sphere order (a sorting network in
// registers), for the final measurement.
__global__ void __launch_bounds__(256) k_pack_sort(const int* __restrict__ cnt, int* __restrict__ lst, int ncell) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= ncell) return;
    const int k = min(cnt[c], kPackCap);
    if (k < 2) return;
    int* L = lst + c * kPackCap;
    int v[kPackCap];
#pragma unroll
    for (int t = 0; t < kPackCap; ++t) v[t] = t < k ? L[t] : 0x7fffffff;
    // odd-even transposition sort: kPackCap rounds of compare-exchange over
    // fixed register indices (no dynamic indexing, so nothing spills)
#pragma unroll
    for (int r = 0; r < kPackCap; ++r) {
#pragma unroll
        for (int t = r & 1; t + 1 < kPackCap; t += 2) {
            const int a = min(v[t], v[t + 1]), b = max(v[t], v[t + 1]);
            v[t] = a;
            v[t + 1] = b;
        }
    }
#pragma unroll
    for (int t = 0; t < kPackCap; ++t)
        if (t < k) L[t] = v[t];
}

// Pair force on sphere p from sphere q at scale s, added to f.
__device__ __forceinline__ void pack_pair(double4 p, double4 q, double s, double& fx, double& fy, double& fz) {
    const double rx = p.x - q.x, ry = p.y - q.y, rz = p.z - q.z;
    const double r2 = rx * rx + ry * ry + rz * rz;
    const double sig = s * (0.5 * (p.w + q.w));
    if (r2 > 0.0 && r2 < sig * sig) {
        const double r = sqrt(r2);
        const double k = (sig - r) / r;
        fx += k * rx;
        fy += k * ry;
        fz += k * rz;
    }
}

// Wall forces on one coordinate added to f: the x = 0 wall, then x = L.
__device__ __forceinline__ double pack_wall(double f, double x, double r, double L) {
    const double lo = r - x, hi = x + r - L;
    if (lo > 0.0) f += lo;
    if (hi > 0.0) f -= hi;
    return f;
}

// One step at scale s: Q_i = P_i + eta F_i, binned into (cnt_out, lst_out),
// whose counts start at zero; clears the counts of `clear`.  ALL: all of them, at
// most one a thread; else those of the centres that Q still holds (nullptr: it
// holds none yet).  Lane l < 27 of a sphere's 32 takes the neighbour cell (l / 9 - 1, l / 3 % 3 - 1, l % 3 - 1) in (z, y, x).
template <bool ALL>
__global__ void __launch_bounds__(kPackThreads) k_pack_step(const double4* __restrict__ P, double4* __restrict__ Q,
                                                            int n, PackGrid gr, const int* __restrict__ cnt,
                                                            const int* __restrict__ lst, double s, double eta,
                                                            int* __restrict__ cnt_out, int* __restrict__ lst_out,
                                                            int* __restrict__ clear, int* __restrict__ flag) {
    const int lane = (int)threadIdx.x & (kPackLanes - 1);
    const int i = (int)blockIdx.x * (kPackThreads / kPackLanes) + (int)threadIdx.x / kPackLanes;
    const bool act = i < n;
    if constexpr (ALL) {
        const int c = (int)(blockIdx.x * kPackThreads + threadIdx.x);
        if (c < gr.ncell) clear[c] = 0;
    }
    // else lane 1 takes the old centre from Q[i] and writes the new one there
    [[maybe_unused]] double4 old = make_double4(0.0, 0.0, 0.0, 0.0);
    if constexpr (!ALL)
        if (act && lane == 1 && clear != nullptr) old = Q[i];
    double fx = 0.0, fy = 0.0, fz = 0.0;
    double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
    if (act) {
        p = P[i];
        int cx, cy, cz;
        pack_cell(gr, p, cx, cy, cz);
        const int z = cz + lane / 9 - 1, y = cy + (lane / 3) % 3 - 1, x = cx + lane % 3 - 1;
        if (lane < 27 && z >= 0 && z < gr.g[2] && y >= 0 && y < gr.g[1] && x >= 0 && x < gr.g[0]) {
            const int c = (z * gr.g[1] + y) * gr.g[0] + x;
            const int* L = lst + c * kPackCap;
            const int4 qa = *(const int4*)L, qb = *(const int4*)(L + 4);   // entries past the count: not used
            const int k = min(cnt[c], kPackCap);
            if (k <= 8) {
                // ascending; a place past the count holds the sphere itself,
                // which is left out below wherever it lands
                int a[8] = {qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, qb.z, qb.w};
#pragma unroll
                for (int t = 0; t < 8; ++t) a[t] = t < k ? a[t] : i;
                // Batcher's odd-even merge sort of eight
                constexpr int net[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6}, {5, 7}, {1, 2}, {5, 6},
                                            {0, 4}, {1, 5}, {2, 6}, {3, 7}, {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
                for (int t = 0; t < 19; ++t) {
                    const int lo = min(a[net[t][0]], a[net[t][1]]), hi = max(a[net[t][0]], a[net[t][1]]);
                    a[net[t][0]] = lo;
                    a[net[t][1]] = hi;
                }
                double4 q[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    q[t] = p;
                    if (a[t] != i) q[t] = P[a[t]];
                }
#pragma unroll
                for (int t = 0; t < 8; ++t) pack_pair(p, q[t], s, fx, fy, fz);
            } else {
                for (int t = 0, last = -1; t < k; ++t) {   // the next larger index each time
                    int j = 0x7fffffff;
                    for (int u = 0; u < k; ++u) j = L[u] > last ? min(j, L[u]) : j;
                    if (j != i) pack_pair(p, P[j], s, fx, fy, fz);
                    last = j;
                }
            }
        }
    }
    // butterfly over the sphere's 32 lanes: every lane ends with the same sum
#pragma unroll
    for (int o = kPackLanes / 2; o > 0; o >>= 1) {
        fx += __shfl_xor(fx, o, kPackLanes);
        fy += __shfl_xor(fy, o, kPackLanes);
        fz += __shfl_xor(fz, o, kPackLanes);
    }
    if (!act || lane > (ALL ? 0 : 1)) return;
    const double r = s * (0.5 * p.w);
    fx = pack_wall(fx, p.x, r, gr.box[0]);
    fy = pack_wall(fy, p.y, r, gr.box[1]);
    fz = pack_wall(fz, p.z, r, gr.box[2]);
    const double4 q = make_double4(p.x + eta * fx, p.y + eta * fy, p.z + eta * fz, p.w);
    int cx, cy, cz, c, slot;
    if constexpr (ALL) {
        Q[i] = q;
        c = pack_cell(gr, q, cx, cy, cz);
        slot = atomicAdd(cnt_out + c, 1);
    } else {
        // the new centre's cell and the old one's, side by side
        c = pack_cell(gr, lane == 0 ? q : old, cx, cy, cz);
        if (lane == 1) {
            Q[i] = q;
            if (clear != nullptr) clear[c] = 0;
            return;
        }
        slot = atomicAdd(cnt_out + c, 1);
    }
    if (slot < kPackCap) lst_out[c * kPackCap + slot] = i;
    else atomicOr(flag, 1);
}

// Per sphere: its share of U_1 (pairs with higher-indexed neighbours, its
// walls) and its largest overlap, into e[i], m[i].
__global__ void __launch_bounds__(256) k_pack_measure(const double4* __restrict__ P, int n, PackGrid gr,
                                                      const int* __restrict__ cnt, const int* __restrict__ lst,
                                                      double* __restrict__ e, double* __restrict__ m) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double4 p = P[i];
    if (!(fabs(p.x) + fabs(p.y) + fabs(p.z) < INFINITY)) {   // a diverged run: NaN reaches the sum
        e[i] = NAN;
        m[i] = NAN;
        return;
    }
    int cx, cy, cz;
    pack_cell(gr, p, cx, cy, cz);
    double u = 0.0, mx = 0.0;
    for (int z = max(cz - 1, 0); z <= min(cz + 1, gr.g[2] - 1); ++z)
        for (int y = max(cy - 1, 0); y <= min(cy + 1, gr.g[1] - 1); ++y)
            for (int x = max(cx - 1, 0); x <= min(cx + 1, gr.g[0] - 1); ++x) {
                const int c = (z * gr.g[1] + y) * gr.g[0] + x;
                const int k = min(cnt[c], kPackCap);
                for (int t = 0; t < k; ++t) {
                    const int j = lst[c * kPackCap + t];
                    if (j <= i) continue;
                    const double4 q = P[j];
                    const double rx = p.x - q.x, ry = p.y - q.y, rz = p.z - q.z;
                    const double ov = 0.5 * (p.w + q.w) - sqrt(rx * rx + ry * ry + rz * rz);
                    if (ov > 0.0) {
                        u += 0.5 * ov * ov;
                        mx = fmax(mx, ov);
                    }
                }
            }
    const double r = 0.5 * p.w;
    const double xs[3] = {p.x, p.y, p.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double lo = r - xs[a], hi = xs[a] + r - gr.box[a];
        if (lo > 0.0) {
            u += 0.5 * lo * lo;
            mx = fmax(mx, lo);
        }
        if (hi > 0.0) {
            u += 0.5 * hi * hi;
            mx = fmax(mx, hi);
        }
    }
    e[i] = u;
    m[i] = mx;
}

// out[0] = sum e (each thread adds a strided share in order, then the shares
// are added in thread order), out[1] = max m; one workgroup of 256 threads.
__global__ void __launch_bounds__(256) k_pack_reduce(const double* __restrict__ e, const double* __restrict__ m, int n,
                                                     double* __restrict__ out) {
    __shared__ double su[256], sm[256];
    const int t = (int)threadIdx.x;
    double u = 0.0, mx = 0.0;
    for (int i = t; i < n; i += 256) {
        u += e[i];
        mx = fmax(mx, m[i]);
    }
    su[t] = u;
    sm[t] = mx;
    __syncthreads();
    if (t == 0) {
        double a = 0.0, b = 0.0;
        for (int k = 0; k < 256; ++k) {
            a += su[k];
            b = fmax(b, sm[k]);
        }
        out[0] = a;
        out[1] = b;
    }
}

}  // namespace mbf
