// Problem build: raw points (or raw-sum clusters) -> centred point clusters
// (Eq. 2) -> static plan of the iteration.  Runs once per problem.
//
// Paper Sec. IV-A groups points by (voxel, pose) with sort_by_key and
// reduce_by_key and builds two index mappers, M_v (cluster -> voxel) and M_s
// (voxel-sorted -> pose-sorted order), consumed every iteration (Alg. 2).
// Here the same grouping runs as a stable device radix sort plus one
// wavefront per cluster, and the mappers are materialised once as two
// physical copies of the clusters:
//   * a voxel-major, wave-interleaved copy: voxels of equal cluster count m
//     are packed 64 to a wave group, cluster k of lane l at cbase + 64 k + l,
//     so the residual pass reads fully coalesced with no divergence;
//   * a pose-major copy cut into chunks of one pose, so the derivative pass
//     reduces per pose in registers without scatter or atomics;
// both in tiles of 64 clusters (Tile<T>).  The plan is formed on the device.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <vector>

#include "ba.h"
#include "ba_device.hpp"
#include "ba_internal.hpp"
#include "ba_host.hpp"

namespace ba {

// ---------------------------------------------------------------- kernels
static inline unsigned nblk(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// Sort keys (voxel << sbits | scan) and what the input's own order lacks:
// order[0] is set where a scan falls below its predecessor's, order[1] where a
// key does.  Points in scan order (a log) need a stable sort by voxel alone,
// and clusters in (voxel, scan) order (a voxel map's export) none.  The blocks
// walk the list, so that a block stores its findings once: with one atomic per
// wave on the flag word the 3.99M keys of a city took 171 us instead of 16.
static constexpr unsigned KEY_BLOCKS = 8192;

struct KeyOrder {
    bool scans = false, keys = false;
};

__device__ __forceinline__ void make_key(int64_t i, const int32_t *__restrict__ scan,
                                         const int32_t *__restrict__ voxel, int sbits, uint64_t *__restrict__ keys,
                                         KeyOrder &o) {
    const int32_t sc = scan[i], vx = voxel[i];
    const uint64_t k = (uint64_t)vx << sbits | (uint64_t)sc;
    keys[i] = k;
    if (i > 0) {
        const int32_t ps = scan[i - 1], pv = voxel[i - 1];
        o.scans |= sc < ps;
        o.keys |= k < ((uint64_t)pv << sbits | (uint64_t)ps);
    }
}

__device__ __forceinline__ void store_order(const KeyOrder &o, int32_t *__restrict__ order) {
    const int s = __syncthreads_or(o.scans), k = __syncthreads_or(o.keys);
    if (threadIdx.x == 0) {
        if (s) order[0] = 1;
        if (k) order[1] = 1;
    }
}

// Checks and sort key of every point.
__global__ __launch_bounds__(256) void k_point_keys(int64_t n, const double *__restrict__ x,
                                                    const double *__restrict__ y, const double *__restrict__ z,
                                                    const int32_t *__restrict__ scan,
                                                    const int32_t *__restrict__ voxel, int32_t n_scans,
                                                    int32_t n_voxels, int sbits, uint64_t *__restrict__ keys,
                                                    int32_t *__restrict__ err) {
    KeyOrder o;
    int bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (!(isfinite(x[i]) && isfinite(y[i]) && isfinite(z[i]))) bad |= 1;
        if (scan[i] < 0 || scan[i] >= n_scans) bad |= 2;
        if (voxel[i] < 0 || voxel[i] >= n_voxels) bad |= 4;
        make_key(i, scan, voxel, sbits, keys, o);
    }
    if (bad) atomicOr(err, bad);
    store_order(o, err + 1);
}

__global__ __launch_bounds__(256) void k_sum_keys(int64_t n, const int32_t *__restrict__ scan,
                                                  const int32_t *__restrict__ voxel, int sbits,
                                                  uint64_t *__restrict__ keys, int32_t *__restrict__ order) {
    KeyOrder o;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        make_key(i, scan, voxel, sbits, keys, o);
    store_order(o, order);
}

// Sort of the keys by what their order lacks (see make_key).
static hipError_t sort_keys(SortBuf &b, int64_t n, int vbits, int sbits, const int32_t order[2], hipStream_t s) {
    if (!order[1]) return radix_sort_pairs(b, n, 0, 0, true, s);
    if (!order[0]) return radix_sort_pairs(b, n, sbits, vbits, true, s);
    return radix_sort_pairs(b, n, 0, vbits + sbits, true, s);
}

__device__ __forceinline__ double dd_div_int(double hi, double lo, double n) {
    double q = hi / n;
    double r = fma(-q, n, hi) + lo;
    return q + r / n;
}

// One wavefront per cluster: compensated centroid, then centred scatter.  Lane
// l takes the cluster's points l, l + 64, ... through the sorted index and
// keeps the first STATS_KEEP of them in registers for the second pass, so a
// cluster of up to 64 STATS_KEEP points is read once.  Bound by the latency of
// start -> index -> point with the waves that fit.  199k clusters of 29.6M
// points: 363 us; 421 us keeping 8 points a lane (5 waves per SIMD instead of
// 6), 469 us with 16 lanes per cluster, 632 us with a gathered copy of the
// points in between, read by both passes.
// Clusters of more than STATS_LONG points are only listed (see k_long_stats).
static constexpr int STATS_KEEP = 4;
static constexpr int64_t STATS_LONG = 32768;

struct PointSums {
    double hx = 0, lx = 0, hy = 0, ly = 0, hz = 0, lz = 0;
    __device__ __forceinline__ void add(double x, double y, double z) {
        dd_add(hx, lx, x);
        dd_add(hy, ly, y);
        dd_add(hz, lz, z);
    }
    // the wave's centroid of n points
    __device__ __forceinline__ void mean(double n, double (&m)[3]) {
        wave_dd_sum(hx, lx);
        wave_dd_sum(hy, ly);
        wave_dd_sum(hz, lz);
        m[0] = dd_div_int(hx, lx, n);
        m[1] = dd_div_int(hy, ly, n);
        m[2] = dd_div_int(hz, lz, n);
    }
};

struct PointScatter {
    double xx = 0, xy = 0, xz = 0, yy = 0, yz = 0, zz = 0;
    __device__ __forceinline__ void add(const double (&m)[3], double qx, double qy, double qz) {
        const double dx = qx - m[0], dy = qy - m[1], dz = qz - m[2];
        xx = fma(dx, dx, xx); xy = fma(dx, dy, xy); xz = fma(dx, dz, xz);
        yy = fma(dy, dy, yy); yz = fma(dy, dz, yz); zz = fma(dz, dz, zz);
    }
    // the wave's record of cluster c
    __device__ __forceinline__ void store(int64_t c, int lane, double n, const double (&m)[3],
                                          double *__restrict__ crec) {
        xx = wave_sum(xx); xy = wave_sum(xy); xz = wave_sum(xz);
        yy = wave_sum(yy); yz = wave_sum(yz); zz = wave_sum(zz);
        if (lane != 0) return;
        double2 *o = reinterpret_cast<double2 *>(crec + CREC * c);
        o[0] = {n, m[0]};
        o[1] = {m[1], m[2]};
        o[2] = {xx, xy};
        o[3] = {xz, yy};
        o[4] = {yz, zz};
    }
};

__global__ __launch_bounds__(256) void k_cluster_stats(int64_t C, const int64_t *__restrict__ starts,
                                                       const uint32_t *__restrict__ idx,
                                                       const double *__restrict__ x, const double *__restrict__ y,
                                                       const double *__restrict__ z,
                                                       const uint64_t *__restrict__ skeys, int sbits,
                                                       double *__restrict__ crec, int32_t *__restrict__ cvox,
                                                       int32_t *__restrict__ cscan, int64_t c_first,
                                                       unsigned long long *__restrict__ n_long,
                                                       uint32_t *__restrict__ longs) {
    int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    int lane = threadIdx.x & 63;
    if (c >= C) return;
    int64_t a = starts[c], b = starts[c + 1];
    const uint64_t key = skeys[a];
    if (lane == 0) {
        cvox[c] = (int32_t)(key >> sbits);
        cscan[c] = (int32_t)(key & (((uint64_t)1 << sbits) - 1));
    }
    if (b - a > STATS_LONG) {
        if (lane == 0) longs[atomicAdd(n_long, 1ull)] = (uint32_t)(c_first + c);
        return;
    }
    double px[STATS_KEEP], py[STATS_KEEP], pz[STATS_KEEP];
#pragma unroll
    for (int k = 0; k < STATS_KEEP; k++) {
        const int64_t i = a + 64 * k + lane;
        if (i < b) {
            const uint32_t j = idx[i];
            px[k] = x[j];
            py[k] = y[j];
            pz[k] = z[j];
        }
    }
    PointSums sum;
#pragma unroll
    for (int k = 0; k < STATS_KEEP; k++)
        if (a + 64 * k + lane < b) sum.add(px[k], py[k], pz[k]);
    for (int64_t i = a + 64 * STATS_KEEP + lane; i < b; i += 64) {
        const uint32_t j = idx[i];
        sum.add(x[j], y[j], z[j]);
    }
    const double n = (double)(b - a);
    double m[3];
    sum.mean(n, m);
    PointScatter sc;
#pragma unroll
    for (int k = 0; k < STATS_KEEP; k++)
        if (a + 64 * k + lane < b) sc.add(m, px[k], py[k], pz[k]);
    for (int64_t i = a + 64 * STATS_KEEP + lane; i < b; i += 64) {
        const uint32_t j = idx[i];
        sc.add(m, x[j], y[j], z[j]);
    }
    sc.store(c, lane, n, m, crec);
}

// The listed long clusters, one wave each in the same order of sums, with
// LONG_ROWS of its rows of 64 points in flight: alone on a chip a wave is bound
// by the two dependent loads of every row.  10M points in one cluster: a build
// of 90 ms against 247 in the kernel above and 132 with the points gathered
// first; in eight 12.8 against 34 and 22.
static constexpr int LONG_ROWS = 8;

template <class Take>
__device__ __forceinline__ void long_points(int64_t a, int64_t b, int lane, const uint32_t *__restrict__ idx,
                                            const double *__restrict__ x, const double *__restrict__ y,
                                            const double *__restrict__ z, Take take) {
    for (int64_t i = a + lane; i < b; i += 64 * LONG_ROWS) {
        uint32_t j[LONG_ROWS];
        double px[LONG_ROWS], py[LONG_ROWS], pz[LONG_ROWS];
#pragma unroll
        for (int r = 0; r < LONG_ROWS; r++) j[r] = idx[min(i + 64 * r, b - 1)];
#pragma unroll
        for (int r = 0; r < LONG_ROWS; r++) {
            px[r] = x[j[r]];
            py[r] = y[j[r]];
            pz[r] = z[j[r]];
        }
#pragma unroll
        for (int r = 0; r < LONG_ROWS; r++)
            if (i + 64 * r < b) take(px[r], py[r], pz[r]);
    }
}

__global__ __launch_bounds__(64) void k_long_stats(int64_t n_long, const uint32_t *__restrict__ longs,
                                                   const int64_t *__restrict__ starts,
                                                   const uint32_t *__restrict__ idx, const double *__restrict__ x,
                                                   const double *__restrict__ y, const double *__restrict__ z,
                                                   double *__restrict__ crec) {
    const int lane = threadIdx.x;
    for (int64_t e = blockIdx.x; e < n_long; e += gridDim.x) {
        const int64_t c = longs[e], a = starts[c], b = starts[c + 1];
        PointSums sum;
        long_points(a, b, lane, idx, x, y, z, [&](double qx, double qy, double qz) { sum.add(qx, qy, qz); });
        const double n = (double)(b - a);
        double m[3];
        sum.mean(n, m);
        PointScatter sc;
        long_points(a, b, lane, idx, x, y, z, [&](double qx, double qy, double qz) { sc.add(m, qx, qy, qz); });
        sc.store(c, lane, n, m, crec);
    }
}

__global__ void k_validate_sums(int64_t n, const int32_t *__restrict__ voxel, const int32_t *__restrict__ scan,
                                const int64_t *__restrict__ count, const double *__restrict__ s1,
                                const double *__restrict__ s2, int32_t n_scans, int32_t n_voxels,
                                int32_t *__restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int bad = 0;
    if (scan[i] < 0 || scan[i] >= n_scans) bad |= 2;
    if (voxel[i] < 0 || voxel[i] >= n_voxels) bad |= 4;
    if (count[i] < 1) bad |= 8;
    for (int k = 0; k < 3; k++) if (!isfinite(s1[3 * i + k])) bad |= 1;
    for (int k = 0; k < 6; k++) if (!isfinite(s2[6 * i + k])) bad |= 1;
    if (bad) atomicOr(err, bad);
}

__global__ void k_dup_keys(int64_t n, const uint64_t *__restrict__ keys, int32_t *__restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || i == 0) return;
    if (keys[i] == keys[i - 1]) atomicOr(err, 16);
}

// Centre raw sums once in double-double: mu = s / N, S = Q - s s^T / N.
__device__ __forceinline__ double centre_entry(double q, double sa, double sb, double n) {
    double ph = sa * sb;
    double pl = fma(sa, sb, -ph);
    double qh = ph / n;
    double rem = fma(-qh, n, ph) + pl;
    double ql = rem / n;
    double s, e;
    two_sum(q, -qh, s, e);
    return s + (e - ql);
}

// A block centres 256 clusters: their sums come and their records go through
// LDS in whole lines (thread by thread, the 24- and 48-byte rows in and the
// 80-byte records out took 192 us for 3.99M clusters; so: 135).
__global__ __launch_bounds__(256) void k_center_sums(int64_t C, const uint32_t *__restrict__ order,
                                                     const uint64_t *__restrict__ skeys,
                                                     const int64_t *__restrict__ count,
                                                     const double *__restrict__ s1, const double *__restrict__ s2,
                                                     int sbits, double *__restrict__ crec,
                                                     int32_t *__restrict__ cvox, int32_t *__restrict__ cscan) {
    __shared__ __attribute__((aligned(16))) double row[256 * CREC];
    __shared__ uint32_t from[256];
    const int64_t c_first = (int64_t)blockIdx.x * 256;
    const int t = threadIdx.x, nb = (int)min((int64_t)256, C - c_first);
    if (t < nb) from[t] = order[c_first + t];
    __syncthreads();
    for (int e = t; e < 3 * nb; e += 256) row[CREC * (e / 3) + 1 + e % 3] = s1[3 * (int64_t)from[e / 3] + e % 3];
    for (int e = t; e < 6 * nb; e += 256) row[CREC * (e / 6) + 4 + e % 6] = s2[6 * (int64_t)from[e / 6] + e % 6];
    __syncthreads();
    if (t < nb) {
        const int64_t c = c_first + t;
        double *v = row + CREC * t;
        const double n = (double)count[from[t]];
        const double s[3] = {v[1], v[2], v[3]};
        const double Q[6] = {v[4], v[5], v[6], v[7], v[8], v[9]};
        v[0] = n;
        for (int k = 0; k < 3; k++) {
            double q = s[k] / n;
            double r = fma(-q, n, s[k]);
            v[1 + k] = q + r / n;
        }
        v[4] = centre_entry(Q[0], s[0], s[0], n);
        v[5] = centre_entry(Q[1], s[0], s[1], n);
        v[6] = centre_entry(Q[2], s[0], s[2], n);
        v[7] = centre_entry(Q[3], s[1], s[1], n);
        v[8] = centre_entry(Q[4], s[1], s[2], n);
        v[9] = centre_entry(Q[5], s[2], s[2], n);
        const uint64_t key = skeys[c];
        cvox[c] = (int32_t)(key >> sbits);
        cscan[c] = (int32_t)(key & (((uint64_t)1 << sbits) - 1));
    }
    __syncthreads();
    double2 *o = reinterpret_cast<double2 *>(crec + CREC * c_first);
    const double2 *r2 = reinterpret_cast<const double2 *>(row);
    for (int e = t; e < CREC / 2 * nb; e += 256) o[e] = r2[e];
}

// Row e of the tile that holds cluster i (ten component rows), and its id.
template <class T>
__device__ __forceinline__ T *tile_at(char *tiles, int64_t i) {
    return reinterpret_cast<T *>(tiles + (i >> 6) * Tile<T>::BYTES) + (i & 63);
}
template <class T>
__device__ __forceinline__ int32_t *tile_id(char *tiles, int64_t i) {
    return reinterpret_cast<int32_t *>(tiles + (i >> 6) * Tile<T>::BYTES + Tile<T>::IDS) + (i & 63);
}

__device__ __forceinline__ void load_record(const double *__restrict__ crec, int64_t c, double (&v)[CREC]) {
    const double2 *p = reinterpret_cast<const double2 *>(crec + CREC * c);
#pragma unroll
    for (int k = 0; k < CREC / 2; k++) {
        const double2 d = p[k];
        v[2 * k] = d.x;
        v[2 * k + 1] = d.y;
    }
}

// Voxel-major copy, one thread per slot: the voxel's clusters lie together in
// the centred records, so a thread reads its records in turn and the 64 lanes
// of a group write whole tile rows.  Padding lanes hold zeros.  Bound by the
// record loads, 64 lines an instruction: five of 16 bytes a record, where ten
// loads from three arrays took 59 us for 199k clusters (now 32) and, in the
// FP32 form with two passes over them, 618 us for 3.99M (now 237).  A thread
// takes at most FILL_RUN clusters: of longer voxels a second launch fills the
// rest, a wave per FILL_RUN more (parts), so that one voxel of very many scans
// is no serial chain (200,000 scans beside 80,000 ordinary clusters: a build of
// 72 ms, now 2.4).
static constexpr int FILL_RUN = 64;
struct FillPart {
    int32_t group, k0;
};
__global__ __launch_bounds__(256) void k_fill_vox(int64_t n, const FillPart *__restrict__ parts,
                                                  const GroupDesc *__restrict__ groups,
                                                  const int64_t *__restrict__ slot_start,
                                                  const double *__restrict__ crec, const int32_t *__restrict__ cscan,
                                                  char *__restrict__ tiles) {
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (wave >= n) return;
    const int lane = (int)(threadIdx.x & 63);
    const FillPart part = parts ? parts[wave] : FillPart{(int32_t)wave, 0};
    const GroupDesc g = groups[part.group];
    const bool used = lane < g.nvox;
    const int64_t c0 = slot_start[64LL * part.group + lane];
    const int k1 = min(g.m, part.k0 + FILL_RUN);
#pragma unroll 2
    for (int k = part.k0; k < k1; k++) {
        const int64_t d = g.cbase + 64LL * k + lane;
        double v[CREC];
#pragma unroll
        for (int e = 0; e < CREC; e++) v[e] = 0.0;
        int32_t j = 0;
        if (used) {
            load_record(crec, c0 + k, v);
            j = cscan[c0 + k];
        }
        double *o = tile_at<double>(tiles, d);
#pragma unroll
        for (int e = 0; e < CREC; e++) o[64 * e] = v[e];
        *tile_id<double>(tiles, d) = j;
    }
}

// Gather centred clusters into the pose-major layout.
__global__ void k_gather_pose(int64_t C, const uint32_t *__restrict__ order, const int32_t *__restrict__ slot_of,
                              const double *__restrict__ crec, char *__restrict__ tiles,
                              int32_t *__restrict__ cidx) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= C) return;
    int64_t c = order[q];
    cidx[q] = (int32_t)c;
    double v[CREC];
    load_record(crec, c, v);
    double *o = tile_at<double>(tiles, q);
#pragma unroll
    for (int e = 0; e < CREC; e++) o[64 * e] = v[e];
    *tile_id<double>(tiles, q) = slot_of[c];
}

__global__ void k_export_records(int64_t C, const double *__restrict__ crec, double *__restrict__ count,
                                 double *__restrict__ mu, double *__restrict__ S) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < CREC * C;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = t / CREC;
        const int e = (int)(t - CREC * c);
        const double v = crec[t];
        if (e == 0) {
            if (count) count[c] = v;
        } else if (e < 4) {
            if (mu) mu[3 * c + e - 1] = v;
        } else if (S) {
            S[6 * c + e - 4] = v;
        }
    }
}

hipError_t export_records(const Problem *P, double *count, double *mu, double *S, hipStream_t s) {
    const int64_t C = P->n_clusters;
    hipLaunchKernelGGL(k_export_records, dim3(stride_blocks(CREC * C)), dim3(256), 0, s, C, P->c_rec, count, mu, S);
    return hipGetLastError();
}

// ---------------------------------------------------------------- precision form
// Reference point of each voxel slot: the FP64 centroid c_i of the voxel's
// clusters placed by the reference poses T0.  Each cluster is then stored in
// FP32 in the world frame of its scan's reference pose, relative to c_i:
//   mu' = R0 mu + t0 - c_i,   S' = R0 S R0^T,
// so that at poses T the iteration only applies the pose change
// G = R R0^T = I + E (small) to small, voxel-centred quantities.
__device__ __forceinline__ void ref_frame_f32(const Pose &P0, const double *c, const double *mu, const double *S,
                                              float *mu32, float *S32) {
    double y[3], St[6];
    rot(P0.r, mu, y);
#pragma unroll
    for (int k = 0; k < 3; k++) mu32[k] = (float)((y[k] + P0.t[k]) - c[k]);
    rot_sym(P0.r, S, St);
#pragma unroll
    for (int k = 0; k < 6; k++) S32[k] = (float)St[k];
}

// One thread per slot, as k_fill_vox: the voxel's reference point, then its
// clusters in the reference frame.  Padding slots get a zero reference and
// zero clusters.  err: 1 = non-finite reference, 2 = a count >= 2^24.
// A wave's group observes a short run of scans, whose reference poses it stages
// in LDS when they are at most FILL_STAGE (they would be half of the loads).
static constexpr int FILL_STAGE = 32, FILL_KEEP = 8;
__global__ __launch_bounds__(256) void k_fill_vox_f32(
    int32_t n_groups, const GroupDesc *__restrict__ groups, const int64_t *__restrict__ slot_start,
    const double *__restrict__ crec, const int32_t *__restrict__ cscan, const double *__restrict__ ref_poses,
    double *__restrict__ vref, char *__restrict__ tiles, int32_t *__restrict__ err) {
    __shared__ double rows[4][FILL_STAGE * 12];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int32_t gi = (int32_t)(blockIdx.x * 4 + w);
    const bool has = gi < n_groups;
    const GroupDesc g = groups[has ? gi : 0];
    const bool staged = g.nscan <= FILL_STAGE;
    if (staged)
        for (int e = lane; e < 12 * g.nscan; e += 64) rows[w][e] = ref_poses[12LL * g.scan0 + e];
    __syncthreads();
    if (!has) return;
    const int64_t sl = 64LL * gi + lane;
    double *ref = vref + 4 * sl;
    if (lane >= g.nvox) {
        ref[0] = ref[1] = ref[2] = ref[3] = 0.0;
        for (int k = 0; k < g.m; k++) {
            const int64_t idx = g.cbase + 64LL * k + lane;
            float *o = tile_at<float>(tiles, idx);
#pragma unroll
            for (int e = 0; e < CREC; e++) o[64 * e] = 0.0f;
            *tile_id<float>(tiles, idx) = 0;
        }
        return;
    }
    const int64_t c0 = slot_start[sl];
    auto pose_of = [&](int32_t j, Pose &P0) {
        if (staged) {
            const double *q = rows[w] + 12 * (j - g.scan0);
#pragma unroll
            for (int e = 0; e < 9; e++) P0.r[e] = q[e];
#pragma unroll
            for (int e = 0; e < 3; e++) P0.t[e] = q[9 + e];
        } else {
            load_pose(ref_poses, j, P0);
        }
    };
    // one pass over the records: the reference point needs every cluster's
    // placed centroid first, so the first FILL_KEEP of them wait in registers
    // and only longer voxels read theirs again
    double n = 0.0, c[3] = {0.0, 0.0, 0.0}, held[FILL_KEEP][3];
    int bad = 0;
    auto first = [&](int k, double *p) {
        const int64_t idx = g.cbase + 64LL * k + lane;
        const int32_t j = cscan[c0 + k];
        double v[CREC];
        load_record(crec, c0 + k, v);
        Pose P0;
        pose_of(j, P0);
        double y[3], St[6];
        rot(P0.r, v + 1, y);
        n += v[0];
#pragma unroll
        for (int q = 0; q < 3; q++) {
            p[q] = y[q] + P0.t[q];
            c[q] = fma(v[0], p[q], c[q]);
        }
        rot_sym(P0.r, v + 4, St);
        float *o = tile_at<float>(tiles, idx);
        if (v[0] >= 16777216.0) bad |= 2;
        o[0] = (float)v[0];
#pragma unroll
        for (int e = 0; e < 6; e++) o[64 * (4 + e)] = (float)St[e];
        *tile_id<float>(tiles, idx) = j;
    };
#pragma unroll
    for (int k = 0; k < FILL_KEEP; k++)
        if (k < g.m) first(k, held[k]);
    for (int k = FILL_KEEP; k < g.m; k++) {
        double p[3];
        first(k, p);
    }
#pragma unroll
    for (int q = 0; q < 3; q++) c[q] /= n;
    if (!(isfinite(c[0]) && isfinite(c[1]) && isfinite(c[2]))) bad |= 1;
    ref[0] = c[0]; ref[1] = c[1]; ref[2] = c[2]; ref[3] = 0.0;
    auto second = [&](int k, const double *p) {
        float *o = tile_at<float>(tiles, g.cbase + 64LL * k + lane);
#pragma unroll
        for (int e = 0; e < 3; e++) o[64 * (1 + e)] = (float)(p[e] - c[e]);
    };
#pragma unroll
    for (int k = 0; k < FILL_KEEP; k++)
        if (k < g.m) second(k, held[k]);
    for (int k = FILL_KEEP; k < g.m; k++) {
        const double2 *p = reinterpret_cast<const double2 *>(crec + CREC * (c0 + k));
        const double2 p0 = p[0], p1 = p[1];
        const double mu[3] = {p0.y, p1.x, p1.y};
        Pose P0;
        pose_of(cscan[c0 + k], P0);
        double y[3];
        rot(P0.r, mu, y);
        const double q[3] = {y[0] + P0.t[0], y[1] + P0.t[1], y[2] + P0.t[2]};
        second(k, q);
    }
    if (bad) atomicOr(err, bad);
}

// Pose-major FP32 copy in the same reference frames.
__global__ void k_gather_pose_f32(int64_t C, const uint32_t *__restrict__ order, const uint64_t *__restrict__ scan_of,
                                  const int32_t *__restrict__ slot_of, const double *__restrict__ crec,
                                  const double *__restrict__ vref, const double *__restrict__ ref_poses,
                                  char *__restrict__ tiles, int32_t *__restrict__ cidx) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= C) return;
    const int64_t c = order[q];
    cidx[q] = (int32_t)c;
    const int32_t sl = slot_of[c];
    double v[CREC];
    load_record(crec, c, v);
    Pose P0;
    load_pose(ref_poses, (int)scan_of[q], P0);
    const double2 *rp = reinterpret_cast<const double2 *>(vref + 4LL * sl);
    const double2 r0 = rp[0], r1 = rp[1];
    const double ref[3] = {r0.x, r0.y, r1.x};
    float m32[3], S32[6];
    ref_frame_f32(P0, ref, v + 1, v + 4, m32, S32);
    float *o = tile_at<float>(tiles, q);
#pragma unroll
    for (int k = 0; k < 3; k++) o[64 * (1 + k)] = m32[k];
#pragma unroll
    for (int k = 0; k < 6; k++) o[64 * (4 + k)] = S32[k];
    o[0] = (float)v[0];
    *tile_id<float>(tiles, q) = sl;
}

__global__ void k_validate_poses(int64_t n, const double *__restrict__ poses, int32_t *__restrict__ err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && !isfinite(poses[i])) atomicOr(err, 1);
}


static ba_status read_count(int64_t *dst, const int64_t *src, hipStream_t s) {
    BA_HIP(hipMemcpyAsync(dst, src, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    return BA_OK;
}

// What a build reads back, in one allocation cleared by one fill: error flags
// and the order's two; then, where the plan first waits for the device, a count
// of the caller's, the number of voxels, an error of the reference poses, and
// what k_plan_check finds.
struct BuildHead {
    int32_t err, order[2], bad_poses;
    int64_t pending, total;
    int32_t max_m, bad_voxel;
};

static int bit_length(uint64_t v) {
    int b = 0;
    while (v) { b++; v >>= 1; }
    return b;
}

// ---------------------------------------------------------------- pose chunks
// One thread per pose: its chunks, from chunk_ptr[j] on.
__global__ void k_chunks(int32_t N, const int64_t *__restrict__ start, const int32_t *__restrict__ chunk_ptr,
                         int32_t chunk_len, ChunkDesc *__restrict__ chunks) {
    const int32_t j = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (j >= N) return;
    int32_t o = chunk_ptr[j];
    const int64_t b = start[j + 1];
    for (int64_t s0 = start[j]; s0 < b; s0 += chunk_len) {
        ChunkDesc ch;
        ch.start = s0;
        ch.count = (int32_t)min((int64_t)chunk_len, b - s0);
        ch.pose = j;
        chunks[o++] = ch;
    }
}

// Cuts every pose's range of the pose-major layout into chunks of at most
// chunk_len clusters and fills the chunk tables (synchronous).
ba_status replan_chunks(Problem *P, int32_t chunk_len, hipStream_t s) {
    if (chunk_len < MIN_CHUNK || chunk_len > MAX_CHUNK) {
        set_error("chunk_len %d out of range [%d, %d]", chunk_len, MIN_CHUNK, MAX_CHUNK);
        return BA_E_ARG;
    }
    const int32_t N = P->n_poses;
    std::vector<int32_t> chunk_ptr(N + 1, 0);
    int64_t n = 0;
    bool one = true;
    for (int32_t j = 0; j < N; j++) {
        chunk_ptr[j] = (int32_t)n;
        n += (P->h_pose_start[j + 1] - P->h_pose_start[j] + chunk_len - 1) / chunk_len;
        one = one && n == j + 1;
    }
    chunk_ptr[N] = (int32_t)n;
    if (n > P->chunk_cap) {
        set_error("internal: %lld chunks exceed the table capacity %lld", (long long)n, (long long)P->chunk_cap);
        return BA_E_ARG;
    }
    BA_HIP(hipMemcpyAsync(P->chunk_ptr, chunk_ptr.data(), sizeof(int32_t) * (N + 1), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_chunks, dim3(nblk(N)), dim3(256), 0, s, N, P->pose_start, P->chunk_ptr, chunk_len,
                       P->chunks);
    BA_HIP(hipGetLastError());
    BA_HIP(hipStreamSynchronize(s));
    P->n_chunks = (int32_t)n;
    P->one_chunk = one && N > 0;
    P->chunk_len = chunk_len;
    P->tune.chunk_len = chunk_len;
    return BA_OK;
}

// ---------------------------------------------------------------- plan
// The static tables of the iteration, formed on the device from the cluster
// labels (in (voxel, scan) order).  The host sees only counts, the runs of
// voxels that share a window and a cluster count, and the poses' ranges.  (As
// counting passes on one host core, with the labels copied down and four
// tables up, the plan took 104 ms of a 107 ms build of 4M clusters, which now
// takes 1.55 ms.)

// The largest cluster count of a voxel (one atomic per block: blocks walk the
// voxels), and the first voxel that is observed from more than one window
// (kept as INT32_MAX less the voxel, so that zero means none).
__global__ __launch_bounds__(256) void k_plan_check(const int64_t *__restrict__ n_vox,
                                                    const int64_t *__restrict__ vstart,
                                                    const int32_t *__restrict__ cscan,
                                                    const int32_t *__restrict__ pose_window, int32_t W,
                                                    int32_t *__restrict__ max_m, int32_t *__restrict__ err) {
    const int64_t V = *n_vox;
    int32_t m = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t a = vstart[v], b = vstart[v + 1];
        m = max(m, (int32_t)(b - a));
        // the scans rise, and so do their windows
        if (W > 1 && pose_window[cscan[b - 1]] != pose_window[cscan[a]]) atomicMax(err, INT32_MAX - (int32_t)v);
    }
    __shared__ int red[4];
    m = -block_min_i<4>(-m, red);
    if (threadIdx.x == 0) atomicMax(max_m, m);
}

// Sort key (window, m, first observing scan) of every voxel.  Where these take
// more than 64 bits the voxels are sorted by the scan (k_plan_scans) and then,
// stably, by (window, m) (k_plan_windows).
__global__ void k_plan_keys(int32_t V, const int64_t *__restrict__ vstart, const int32_t *__restrict__ cscan,
                            const int32_t *__restrict__ pose_window, int mbits, int sbits,
                            uint64_t *__restrict__ keys) {
    const int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (v >= V) return;
    const int64_t a = vstart[v];
    const uint64_t m = (uint64_t)(vstart[v + 1] - a), j = (uint64_t)cscan[a];
    keys[v] = (((uint64_t)pose_window[j] << mbits | m) << sbits) | j;
}

__global__ void k_plan_scans(int32_t V, const int64_t *__restrict__ vstart, const int32_t *__restrict__ cscan,
                             uint64_t *__restrict__ keys) {
    const int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (v < V) keys[v] = (uint64_t)cscan[vstart[v]];
}

__global__ void k_plan_windows(int32_t V, const uint32_t *__restrict__ order, const int64_t *__restrict__ vstart,
                               const int32_t *__restrict__ pose_window, int mbits, uint64_t *__restrict__ keys) {
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= V) return;
    const int64_t v = order[i];
    const uint64_t m = (uint64_t)(vstart[v + 1] - vstart[v]);
    keys[i] = (uint64_t)pose_window[keys[i]] << mbits | m;   // the key is the first scan
}

// First position and (window, m) of every run, behind the number of runs: the
// host takes the first RUNS_AHEAD with their number, and the rest by itself.
struct RunHead {
    int64_t first;
    uint64_t key;
};
static constexpr int64_t RUNS_AHEAD = 2048;
__global__ void k_run_list(const int64_t *__restrict__ n_runs, const int64_t *__restrict__ starts,
                           const uint64_t *__restrict__ keys, int shift, RunHead *__restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t R = *n_runs;
    if (r == 0) out[0] = RunHead{R, 0};
    if (r < R) out[1 + r] = RunHead{starts[r], keys[starts[r]] >> shift};
}

// A run of voxels (in plan order) of one window and one cluster count m.
struct PlanRun {
    int64_t first, len;   // positions in the sorted voxel order
    int64_t cbase;        // first cluster of its first group, padded
    int64_t ubase;        // the same, unpadded
    int32_t gbase;        // first group
    int32_t m, window, pad;
};

// One window's groups by split class, ascending (k_vox_mixed).
struct PlanMix {
    int32_t base, g0, n1, n2, n4, pad;   // first block, first group, groups per class
};

static __host__ __device__ int split_of(int32_t m) { return m <= 4 ? 1 : (m <= 8 ? 2 : 4); }

// One wave per group, one lane per voxel slot: the group's descriptor, its
// residual-pass block (the largest cluster counts first within a window, so
// that the longest blocks start earliest), the slots' voxels, and the
// clusters' slots; every cluster is listed under its scan, in slot order.
__global__ __launch_bounds__(256) void k_plan_groups(int32_t G, int32_t R, const PlanRun *__restrict__ runs,
                                                     const uint32_t *__restrict__ order,
                                                     const int64_t *__restrict__ vstart,
                                                     const int32_t *__restrict__ cvox,
                                                     const int32_t *__restrict__ cscan,
                                                     const int32_t *__restrict__ win_group_ptr,
                                                     GroupDesc *__restrict__ groups, VoxBlock *__restrict__ vblocks,
                                                     int32_t *__restrict__ slot_vox, int64_t *__restrict__ slot_start,
                                                     int32_t *__restrict__ c_slot, uint64_t *__restrict__ keys,
                                                     uint32_t *__restrict__ vals) {
    const int32_t gi = (int32_t)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (gi >= G) return;
    int32_t lo = 0, hi = R;   // the last run with gbase <= gi
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (runs[mid].gbase <= gi) lo = mid;
        else hi = mid;
    }
    const PlanRun r = runs[lo];
    const int64_t v0 = 64LL * (gi - r.gbase);
    const int32_t nvox = (int32_t)min((int64_t)64, r.len - v0);
    const int64_t sl = 64LL * gi + lane;
    int32_t s0 = INT32_MAX, s1 = INT32_MAX;   // lowest scan, minus the highest
    int64_t a = 0;
    if (lane < nvox) {
        a = vstart[order[r.first + v0 + lane]];
        s0 = cscan[a];
        s1 = -cscan[a + r.m - 1];
        slot_vox[sl] = cvox[a];
        slot_start[sl] = a;
    } else {
        slot_vox[sl] = -1;
        slot_start[sl] = 0;
    }
    // the group's clusters voxel by voxel, 64 at a time: the list is written in
    // whole lines and the clusters are read in runs of m
    const int64_t u = r.ubase + r.m * v0;
    for (int32_t e0 = 0; e0 < nvox * r.m; e0 += 64) {
        const int32_t e = e0 + lane, l = min(e / r.m, 63);
        const int64_t c = __shfl(a, l, BA_WAVE) + (e - l * r.m);
        if (e < nvox * r.m) {
            c_slot[c] = 64 * gi + l;
            keys[u + e] = (uint64_t)cscan[c];
            vals[u + e] = (uint32_t)c;
        }
    }
    s0 = wave_min_i(s0);
    s1 = -wave_min_i(s1);
    if (lane == 0) {
        GroupDesc g;
        g.cbase = r.cbase + r.m * v0;
        g.m = r.m;
        g.nvox = nvox;
        g.window = r.window;
        g.scan0 = s0;
        g.nscan = s1 - s0 + 1;
        g.pad = 0;
        groups[gi] = g;
        const int32_t a = win_group_ptr[r.window], b = win_group_ptr[r.window + 1];
        vblocks[a + (b - 1 - gi)] = VoxBlock{gi, 1, 4, r.window};
    }
}

// One thread per block of the per-group split: one wave per group up to 4
// clusters per voxel, two up to 8, four beyond, so that no wave walks more
// than about five clusters; a 256-thread block takes four one-wave, two
// two-wave or one four-wave group of one window, largest counts first.
__global__ void k_plan_mix(int32_t n, int32_t W, const PlanMix *__restrict__ mix, VoxBlock *__restrict__ out) {
    const int32_t b = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (b >= n) return;
    int32_t lo = 0, hi = W;   // the last window with base <= b (windows without groups have no block)
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (mix[mid].base <= b) lo = mid;
        else hi = mid;
    }
    const PlanMix w = mix[lo];
    int32_t i = b - w.base;
    if (i < w.n4) {
        out[b] = VoxBlock{w.g0 + w.n1 + w.n2 + w.n4 - 1 - i, 1, 4, lo};
        return;
    }
    i -= w.n4;
    const int32_t p2 = (w.n2 + 1) / 2;
    if (i < p2) {
        const int32_t ng = min(2, w.n2 - 2 * i);
        out[b] = VoxBlock{w.g0 + w.n1 + w.n2 - 2 * i - ng, ng, 2, lo};
        return;
    }
    i -= p2;
    const int32_t ng = min(4, w.n1 - 4 * i);
    out[b] = VoxBlock{w.g0 + w.n1 - 4 * i - ng, ng, 1, lo};
}

// First position of every scan in the sorted list (start[N] = C): a binary
// search per scan, so that scans without clusters cost what the others do.  A
// build of 100,000 clusters with 4M scans, 1000 of them observed, takes 19.4 ms
// and took 115 with a thread per cluster that also wrote the scans before it;
// 3.99M clusters of 2000 scans 1.62 ms either way.
__global__ void k_pose_starts(int64_t C, int32_t N, const uint64_t *__restrict__ keys, int64_t *__restrict__ start) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j > N) return;
    int64_t lo = 0, hi = C;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < (uint64_t)j) lo = mid + 1;
        else hi = mid;
    }
    start[j] = lo;
}

// seen(count) is called with head->pending where the plan first waits for the
// device, ahead of its kernels that read the centred clusters.
using Seen = std::function<ba_status(int64_t)>;

static ba_status make_plan(Problem *P, const std::vector<int32_t> &scan_window, SortBuf &bw, DevArena &keep,
                           BuildHead *head, const Seen &seen, hipStream_t s) {
    const int64_t C = P->n_clusters;
    const int32_t N = P->n_poses;
    const int32_t W = P->n_windows;
    DevArena tmp;
    // windows of the poses
    std::vector<int32_t> win_pose_ptr(W + 1, 0);
    for (int32_t j = 0; j < N; j++) win_pose_ptr[scan_window[j] + 1] = j + 1;
    for (int32_t w = 0; w < W; w++) win_pose_ptr[w + 1] = std::max(win_pose_ptr[w + 1], win_pose_ptr[w]);
    BA_TRY(keep.alloc(&P->win_pose_ptr, W + 1));
    BA_TRY(keep.alloc(&P->pose_window, N));
    BA_HIP(hipMemcpyAsync(P->win_pose_ptr, win_pose_ptr.data(), sizeof(int32_t) * (W + 1), hipMemcpyHostToDevice, s));
    BA_HIP(hipMemcpyAsync(P->pose_window, scan_window.data(), sizeof(int32_t) * N, hipMemcpyHostToDevice, s));
    P->h_win_pose_ptr = new int32_t[W + 1];
    std::memcpy(P->h_win_pose_ptr, win_pose_ptr.data(), sizeof(int32_t) * (W + 1));

    // voxels (their number stays on the device until they have been checked)
    const int64_t v_max = std::min<int64_t>(C, P->n_voxels_in);
    int64_t *vstart;
    BA_TRY(tmp.alloc(&vstart, v_max + 1));
    BA_HIP(segments(P->c_vox, C, 0, bw.total, vstart, bw.ws, s));
    hipLaunchKernelGGL(k_plan_check, dim3(std::min(nblk(v_max), 512u)), dim3(256), 0, s, bw.total, vstart, P->c_scan,
                       P->pose_window, W, &head->max_m, &head->bad_voxel);
    BA_HIP(hipGetLastError());
    BuildHead h;
    BA_HIP(hipMemcpyAsync(&h, head, sizeof(h), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    BA_TRY(seen(h.pending));
    if (h.bad_poses) {
        set_error("ref_poses holds non-finite values");
        return BA_E_ARG;
    }
    if (h.bad_voxel) {
        int64_t a = 0;
        int32_t id = 0;
        BA_TRY(read_count(&a, vstart + (INT32_MAX - h.bad_voxel), s));
        BA_HIP(hipMemcpyAsync(&id, P->c_vox + a, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        BA_HIP(hipStreamSynchronize(s));
        set_error("voxel %d is observed by scans of different windows", id);
        return BA_E_ARG;
    }
    const int32_t V = (int32_t)h.total;
    P->n_vox = V;
    P->max_m = h.max_m;

    // voxel order: (window, m, first observing scan, voxel id), a stable sort;
    // then its runs of one window and one m
    const int sbits = bit_length((uint64_t)(N - 1)), mbits = bit_length((uint64_t)P->max_m);
    const int wbits = bit_length((uint64_t)(W - 1));
    const bool one_key = wbits + mbits + sbits <= 64;
    const int shift = one_key ? sbits : 0;   // of a key's (window, m)
    if (one_key) {
        hipLaunchKernelGGL(k_plan_keys, dim3(nblk(V)), dim3(256), 0, s, V, vstart, P->c_scan, P->pose_window, mbits,
                           sbits, bw.keys);
        BA_HIP(radix_sort_pairs(bw, V, 0, sbits + mbits + wbits, true, s));
    } else {
        hipLaunchKernelGGL(k_plan_scans, dim3(nblk(V)), dim3(256), 0, s, V, vstart, P->c_scan, bw.keys);
        BA_HIP(radix_sort_pairs(bw, V, 0, sbits, true, s));
        hipLaunchKernelGGL(k_plan_windows, dim3(nblk(V)), dim3(256), 0, s, V, bw.vals, vstart, P->pose_window, mbits,
                           bw.keys);
        BA_HIP(radix_sort_pairs(bw, V, 0, mbits + wbits, false, s));
    }
    int64_t *d_rs;
    RunHead *d_rl;
    PlanRun *d_runs;
    BA_TRY(tmp.alloc(&d_rs, (int64_t)V + 1));
    BA_TRY(tmp.alloc(&d_rl, (int64_t)V + 1));
    BA_HIP(segments((const uint64_t *)bw.keys, (int64_t)V, shift, bw.total, d_rs, bw.ws, s));
    hipLaunchKernelGGL(k_run_list, dim3(nblk(V)), dim3(256), 0, s, bw.total, d_rs, bw.keys, shift, d_rl);
    BA_HIP(hipGetLastError());
    std::vector<RunHead> rl(1 + std::min<int64_t>(V, RUNS_AHEAD));
    BA_HIP(hipMemcpyAsync(rl.data(), d_rl, sizeof(RunHead) * rl.size(), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    const int64_t R = rl[0].first, ahead = (int64_t)rl.size();
    rl.resize(R + 2);
    if (R >= ahead) {
        BA_HIP(hipMemcpyAsync(rl.data() + ahead, d_rl + ahead, sizeof(RunHead) * (R + 1 - ahead),
                              hipMemcpyDeviceToHost, s));
        BA_HIP(hipStreamSynchronize(s));
    }
    rl[R + 1].first = V;
    BA_TRY(tmp.alloc(&d_runs, R));
    std::vector<PlanRun> runs(R);
    std::vector<int32_t> win_group_ptr(W + 1, 0);
    std::vector<PlanMix> mix(W);
    std::vector<FillPart> parts;   // of voxels of more than FILL_RUN clusters (FP64 form)
    int64_t cbase = 0, ubase = 0, G = 0;
    for (int64_t r = 0; r < R; r++) {
        PlanRun &q = runs[r];
        q.first = rl[1 + r].first;
        q.len = rl[2 + r].first - q.first;
        q.m = (int32_t)(rl[1 + r].key & (((uint64_t)1 << mbits) - 1));
        q.window = (int32_t)(rl[1 + r].key >> mbits);
        q.gbase = (int32_t)G;
        q.cbase = cbase;
        q.ubase = ubase;
        q.pad = 0;
        const int64_t ng = tiles_of(q.len);
        G += ng;
        cbase += 64LL * q.m * ng;
        ubase += (int64_t)q.m * q.len;
        win_group_ptr[q.window + 1] = (int32_t)G;
        PlanMix &x = mix[q.window];
        if (P->prec == BA_PREC_F64)
            for (int32_t gi = q.gbase; gi < (int32_t)G; gi++)
                for (int64_t k = FILL_RUN; k < q.m; k += FILL_RUN) parts.push_back({gi, (int32_t)k});
        const int sp = split_of(q.m);
        (sp == 1 ? x.n1 : sp == 2 ? x.n2 : x.n4) += (int32_t)ng;
    }
    for (int32_t w = 0; w < W; w++) win_group_ptr[w + 1] = std::max(win_group_ptr[w + 1], win_group_ptr[w]);
    P->n_groups = (int32_t)G;
    P->c_pad = cbase;
    P->n_vblocks = (int32_t)G;
    int32_t n_mix = 0;
    for (int32_t w = 0; w < W; w++) {
        mix[w].base = n_mix;
        mix[w].g0 = win_group_ptr[w];
        n_mix += mix[w].n4 + (mix[w].n2 + 1) / 2 + (mix[w].n1 + 3) / 4;
    }
    P->n_vblocks_mix = n_mix;
    P->chunk_cap = C / MIN_CHUNK + N + 1;

    // device allocations owned by the problem
    const int64_t CP = P->c_pad;
    const int64_t NS = (int64_t)P->n_groups * 64;
    const bool f32 = P->prec == BA_PREC_F32;
    const int64_t tile_bytes = f32 ? Tile<float>::BYTES : Tile<double>::BYTES;
    BA_TRY(keep.alloc(&P->v_tiles, tiles_of(CP) * tile_bytes));
    BA_TRY(keep.alloc(&P->p_tiles, tiles_of(C) * tile_bytes));
    BA_TRY(keep.alloc(&P->groups, std::max<int64_t>(P->n_groups, 1)));
    BA_TRY(keep.alloc(&P->vblocks, std::max<int64_t>(P->n_vblocks, 1)));
    BA_TRY(keep.alloc(&P->vblocks_mix, std::max<int64_t>(P->n_vblocks_mix, 1)));
    BA_TRY(keep.alloc(&P->slot_vox, std::max<int64_t>(NS, 1)));
    BA_TRY(keep.alloc(&P->vstate, 2 * std::max<int64_t>(NS, 1) * VSTATE));
    BA_TRY(keep.alloc(&P->wave_cost, std::max<int64_t>(P->n_groups, 1)));
    if (f32) {
        BA_TRY(keep.alloc(&P->v_ref, 4 * std::max<int64_t>(NS, 1)));
        BA_TRY(keep.alloc(&P->pdelta, 16LL * N));
    }
    BA_TRY(keep.alloc(&P->p_cidx, C));
    BA_TRY(keep.alloc(&P->c_slot, C));
    BA_TRY(keep.alloc(&P->chunks, P->chunk_cap));
    BA_TRY(keep.alloc(&P->chunk_ptr, N + 1));
    BA_TRY(keep.alloc(&P->pose_start, N + 1));
    BA_TRY(keep.alloc(&P->partials, P->chunk_cap * NPART));
    BA_TRY(keep.alloc(&P->win_group_ptr, W + 1));
    BA_TRY(keep.alloc(&P->g, 6LL * N));
    BA_TRY(keep.alloc(&P->H, 36LL * N));
    BA_TRY(keep.alloc(&P->dx, 6LL * N));
    BA_TRY(keep.alloc(&P->poses_trial, 12LL * N));
    BA_TRY(keep.alloc(&P->pose_q, N));
    BA_TRY(keep.alloc(&P->pose_info, N));
    BA_TRY(keep.alloc(&P->lm, W));

    // groups, blocks and the clusters listed by slot under their scans
    int64_t *slot_start;
    PlanMix *d_mix;
    int32_t *d_err;
    BA_TRY(tmp.alloc(&slot_start, NS));
    BA_TRY(tmp.alloc(&d_mix, W));
    BA_TRY(tmp.alloc(&d_err, 1));
    BA_HIP(hipMemcpyAsync(P->win_group_ptr, win_group_ptr.data(), sizeof(int32_t) * (W + 1), hipMemcpyHostToDevice, s));
    BA_HIP(hipMemcpyAsync(d_runs, runs.data(), sizeof(PlanRun) * R, hipMemcpyHostToDevice, s));
    BA_HIP(hipMemcpyAsync(d_mix, mix.data(), sizeof(PlanMix) * W, hipMemcpyHostToDevice, s));
    BA_HIP(hipMemsetAsync(P->vstate, 0, sizeof(double) * 2 * std::max<int64_t>(NS, 1) * VSTATE, s));
    hipLaunchKernelGGL(k_plan_groups, dim3(nblk(NS)), dim3(256), 0, s, P->n_groups, (int32_t)R, d_runs, bw.vals,
                       vstart, P->c_vox, P->c_scan, P->win_group_ptr, P->groups, P->vblocks, P->slot_vox, slot_start,
                       P->c_slot, bw.keys2, bw.vals2);
    std::swap(bw.keys, bw.keys2);
    std::swap(bw.vals, bw.vals2);
    hipLaunchKernelGGL(k_plan_mix, dim3(nblk(n_mix)), dim3(256), 0, s, n_mix, W, d_mix, P->vblocks_mix);
    // pose-major order (scan, slot): a stable sort by scan of that list (a
    // voxel's clusters have distinct scans)
    BA_HIP(radix_sort_pairs(bw, C, 0, sbits, false, s));
    hipLaunchKernelGGL(k_pose_starts, dim3(nblk((int64_t)N + 1)), dim3(256), 0, s, C, N, bw.keys, P->pose_start);
    BA_HIP(hipGetLastError());
    P->h_pose_start.resize(N + 1);
    BA_HIP(hipMemcpyAsync(P->h_pose_start.data(), P->pose_start, sizeof(int64_t) * (N + 1), hipMemcpyDeviceToHost, s));
    // the two copies of the clusters
    if (!f32) {
        hipLaunchKernelGGL(k_fill_vox, dim3(nblk(NS)), dim3(256), 0, s, (int64_t)P->n_groups,
                           (const FillPart *)nullptr, P->groups, slot_start, P->c_rec, P->c_scan, P->v_tiles);
        if (!parts.empty()) {
            FillPart *d_parts;
            BA_TRY(tmp.alloc(&d_parts, (int64_t)parts.size()));
            BA_HIP(hipMemcpyAsync(d_parts, parts.data(), sizeof(FillPart) * parts.size(), hipMemcpyHostToDevice, s));
            hipLaunchKernelGGL(k_fill_vox, dim3(nblk(64 * (int64_t)parts.size())), dim3(256), 0, s,
                               (int64_t)parts.size(), d_parts, P->groups, slot_start, P->c_rec, P->c_scan, P->v_tiles);
        }
        hipLaunchKernelGGL(k_gather_pose, dim3(nblk(C)), dim3(256), 0, s, C, bw.vals, P->c_slot, P->c_rec,
                           P->p_tiles, P->p_cidx);
        BA_HIP(hipGetLastError());
        BA_HIP(hipStreamSynchronize(s));
        BA_TRY(replan_chunks(P, P->chunk_len, s));
        tmp.drained = true;
        return BA_OK;
    }
    BA_HIP(hipMemsetAsync(d_err, 0, sizeof(int32_t), s));
    hipLaunchKernelGGL(k_fill_vox_f32, dim3(nblk(NS)), dim3(256), 0, s, P->n_groups, P->groups, slot_start, P->c_rec,
                       P->c_scan, P->ref_poses, P->v_ref, P->v_tiles, d_err);
    hipLaunchKernelGGL(k_gather_pose_f32, dim3(nblk(C)), dim3(256), 0, s, C, bw.vals, bw.keys, P->c_slot, P->c_rec,
                       P->v_ref, P->ref_poses, P->p_tiles, P->p_cidx);
    BA_HIP(hipGetLastError());
    int32_t herr = 0;
    BA_HIP(hipMemcpyAsync(&herr, d_err, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    BA_TRY(replan_chunks(P, P->chunk_len, s));
    tmp.drained = true;
    if (herr & 2) {
        set_error("precision form: a cluster holds 2^24 points or more (its count is not exact in FP32)");
        return BA_E_UNSUPPORTED;
    }
    if (herr & 1) {
        set_error("precision form: non-finite voxel reference point (check ref_poses)");
        return BA_E_ARG;
    }
    return BA_OK;
}

static ba_status finish_build(Problem *P, DevArena &keep, const ba_build_options *opt, SortBuf &bw,
                              BuildHead *head, const Seen &seen, hipStream_t s) {
    std::vector<int32_t> scan_window(P->n_poses, 0);
    int32_t W = 1;
    if (opt && opt->n_windows > 1) {
        if (!opt->scan_window) {
            set_error("n_windows > 1 needs scan_window");
            return BA_E_ARG;
        }
        W = opt->n_windows;
        for (int32_t j = 0; j < P->n_poses; j++) {
            int32_t w = opt->scan_window[j];
            if (w < 0 || w >= W || (j > 0 && w < scan_window[j - 1])) {
                set_error("scan_window must be non-decreasing in [0, n_windows)");
                return BA_E_ARG;
            }
            scan_window[j] = w;
        }
    }
    P->n_windows = W;
    P->prec = opt ? opt->precision : BA_PREC_F64;
    if (P->prec != BA_PREC_F64 && P->prec != BA_PREC_F32) {
        set_error("unknown precision %d", P->prec);
        return BA_E_ARG;
    }
    if (P->prec == BA_PREC_F32) {
        if (!opt->ref_poses) {
            set_error("the precision form needs ref_poses");
            return BA_E_ARG;
        }
        const int64_t np = 12LL * P->n_poses;
        BA_TRY(keep.alloc(&P->ref_poses, np));
        BA_HIP(hipMemcpyAsync(P->ref_poses, opt->ref_poses, sizeof(double) * np, hipMemcpyDeviceToDevice, s));
        hipLaunchKernelGGL(k_validate_poses, dim3(nblk(np)), dim3(256), 0, s, np, P->ref_poses, &head->bad_poses);
        BA_HIP(hipGetLastError());
    }
    return make_plan(P, scan_window, bw, keep, head, seen, s);
}

ba_status build_from_points(const ba_points *pts, const ba_build_options *opt, Problem *P, DevArena &keep,
                            hipStream_t s) {
    const int64_t n = pts->n;
    if (n < 1 || n > (int64_t)0xFFFFFFFF) {
        set_error("point count %lld out of range [1, 2^32)", (long long)n);
        return BA_E_ARG;
    }
    if (!pts->x || !pts->y || !pts->z || !pts->scan || !pts->voxel || pts->n_scans < 1 || pts->n_voxels < 1) {
        set_error("null point array or empty label range");
        return BA_E_ARG;
    }
    P->n_poses = pts->n_scans;
    P->n_voxels_in = pts->n_voxels;
    P->chunk_len = (opt && opt->chunk_len > 0) ? opt->chunk_len : 256;
    DevArena tmp;
    BuildHead *head;
    SortBuf b;
    BA_TRY(tmp.alloc(&head, 1));
    BA_TRY(b.alloc(tmp, n));
    b.total = &head->total;
    BA_HIP(hipMemsetAsync(head, 0, sizeof(BuildHead), s));
    const int sbits = bit_length((uint64_t)(pts->n_scans - 1)), vbits = bit_length((uint64_t)(pts->n_voxels - 1));
    hipLaunchKernelGGL(k_point_keys, dim3(std::min(nblk(n), KEY_BLOCKS)), dim3(256), 0, s, n, pts->x, pts->y, pts->z, pts->scan, pts->voxel,
                       pts->n_scans, pts->n_voxels, sbits, b.keys, &head->err);
    BA_HIP(hipGetLastError());
    int32_t flags[3] = {0, 0, 0};
    BA_HIP(hipMemcpyAsync(flags, &head->err, sizeof(flags), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    if (flags[0]) {
        set_error("invalid points (flags 0x%x: 1 non-finite, 2 scan out of range, 4 voxel out of range)", flags[0]);
        return BA_E_ARG;
    }
    BA_HIP(sort_keys(b, n, vbits, sbits, flags + 1, s));
    int64_t C = 0;
    BA_HIP(segment_count((const uint64_t *)b.keys, n, 0, b.total, b.ws, s));
    BA_TRY(read_count(&C, b.total, s));
    P->n_clusters = C;
    int64_t *starts;
    uint32_t *longs;
    BA_TRY(tmp.alloc(&starts, C + 1));
    BA_TRY(tmp.alloc(&longs, n / STATS_LONG + 1));
    BA_HIP(segment_write((const uint64_t *)b.keys, n, 0, b.total, starts, b.ws, s));
    BA_TRY(keep.alloc(&P->c_rec, CREC * C));
    BA_TRY(keep.alloc(&P->c_vox, C));
    BA_TRY(keep.alloc(&P->c_scan, C));
    for (int64_t c = 0, k; c < C; c += k) {
        k = std::min(C - c, launch_items(64));
        hipLaunchKernelGGL(k_cluster_stats, dim3(nblk(k * 64)), dim3(256), 0, s, k, starts + c, b.vals, pts->x, pts->y,
                           pts->z, b.keys, sbits, P->c_rec + CREC * c, P->c_vox + c, P->c_scan + c, c,
                           (unsigned long long *)&head->pending, longs);
        BA_HIP(hipGetLastError());
    }
    BA_TRY(finish_build(P, keep, opt, b, head, [&](int64_t n_long) -> ba_status {
        if (n_long > 0)
            hipLaunchKernelGGL(k_long_stats, dim3((unsigned)std::min<int64_t>(n_long, 1 << 20)), dim3(64), 0, s, n_long,
                               longs, starts, b.vals, pts->x, pts->y, pts->z, P->c_rec);
        BA_HIP(hipGetLastError());
        return BA_OK;
    }, s));
    tmp.drained = true;   // the plan's last step waits for the stream
    return BA_OK;
}

ba_status build_from_sums(const ba_cluster_sums *cs, const ba_build_options *opt, Problem *P, DevArena &keep,
                          hipStream_t s) {
    const int64_t n = cs->n;
    if (n < 1 || n > (int64_t)0xFFFFFFFF) {
        set_error("cluster count %lld out of range [1, 2^32)", (long long)n);
        return BA_E_ARG;
    }
    if (!cs->voxel || !cs->scan || !cs->count || !cs->sum || !cs->sumsq || cs->n_scans < 1 || cs->n_voxels < 1) {
        set_error("null cluster array or empty label range");
        return BA_E_ARG;
    }
    P->n_poses = cs->n_scans;
    P->n_voxels_in = cs->n_voxels;
    P->chunk_len = (opt && opt->chunk_len > 0) ? opt->chunk_len : 256;
    DevArena tmp;
    BuildHead *head;
    SortBuf b;
    BA_TRY(tmp.alloc(&head, 1));
    BA_TRY(b.alloc(tmp, n));
    b.total = &head->total;
    BA_HIP(hipMemsetAsync(head, 0, sizeof(BuildHead), s));
    int32_t *err = &head->err;
    const int sbits = bit_length((uint64_t)(cs->n_scans - 1)), vbits = bit_length((uint64_t)(cs->n_voxels - 1));
    hipLaunchKernelGGL(k_validate_sums, dim3(nblk(n)), dim3(256), 0, s, n, cs->voxel, cs->scan, cs->count, cs->sum,
                       cs->sumsq, cs->n_scans, cs->n_voxels, err);
    hipLaunchKernelGGL(k_sum_keys, dim3(std::min(nblk(n), KEY_BLOCKS)), dim3(256), 0, s, n, cs->scan, cs->voxel, sbits, b.keys, err + 1);
    BA_HIP(hipGetLastError());
    int32_t flags[3] = {0, 0, 0};
    BA_HIP(hipMemcpyAsync(flags, err, sizeof(flags), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    BA_HIP(sort_keys(b, n, vbits, sbits, flags + 1, s));
    // duplicates are known where the plan first waits, or here if the input is invalid anyway
    hipLaunchKernelGGL(k_dup_keys, dim3(nblk(n)), dim3(256), 0, s, n, b.keys, (int32_t *)&head->pending);
    BA_HIP(hipGetLastError());
    auto refuse = [](int32_t e) {
        set_error("invalid clusters (flags 0x%x: 1 non-finite, 2 scan, 4 voxel, 8 count < 1, 16 duplicate pair)", e);
        return BA_E_ARG;
    };
    if (flags[0]) {
        int64_t dup = 0;
        BA_TRY(read_count(&dup, &head->pending, s));
        return refuse(flags[0] | (int32_t)dup);
    }
    P->n_clusters = n;
    BA_TRY(keep.alloc(&P->c_rec, CREC * n));
    BA_TRY(keep.alloc(&P->c_vox, n));
    BA_TRY(keep.alloc(&P->c_scan, n));
    hipLaunchKernelGGL(k_center_sums, dim3(nblk(n)), dim3(256), 0, s, n, b.vals, b.keys, cs->count, cs->sum, cs->sumsq,
                       sbits, P->c_rec, P->c_vox, P->c_scan);
    BA_HIP(hipGetLastError());
    BA_TRY(finish_build(P, keep, opt, b, head,
                        [&](int64_t dup) -> ba_status { return dup ? refuse((int32_t)dup) : BA_OK; }, s));
    tmp.drained = true;   // the plan's last step waits for the stream
    return BA_OK;
}

}  // namespace ba
