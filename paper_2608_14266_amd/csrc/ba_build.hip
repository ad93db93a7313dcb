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
//     reduces per pose in registers without scatter or atomics.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "ba.h"
#include "ba_device.hpp"
#include "ba_internal.hpp"
#include "ba_host.hpp"

namespace ba {

// ---------------------------------------------------------------- kernels
__global__ void k_validate_points(int64_t n, const double *__restrict__ x, const double *__restrict__ y,
                                  const double *__restrict__ z, const int32_t *__restrict__ scan,
                                  const int32_t *__restrict__ voxel, int32_t n_scans, int32_t n_voxels,
                                  int32_t *__restrict__ err) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int bad = 0;
    if (!(isfinite(x[i]) && isfinite(y[i]) && isfinite(z[i]))) bad |= 1;
    if (scan[i] < 0 || scan[i] >= n_scans) bad |= 2;
    if (voxel[i] < 0 || voxel[i] >= n_voxels) bad |= 4;
    if (bad) atomicOr(err, bad);
}

__global__ void k_make_keys(int64_t n, const int32_t *__restrict__ scan, const int32_t *__restrict__ voxel,
                            int32_t n_scans, uint64_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = (uint64_t)voxel[i] * (uint64_t)n_scans + (uint64_t)scan[i];
    vals[i] = (uint32_t)i;
}

__global__ void k_head_flags(int64_t n, const uint64_t *__restrict__ keys, int64_t *__restrict__ flags) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    flags[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
}

// after an exclusive scan of the head flags: starts[cid] = i for every head
__global__ void k_segment_starts(int64_t n, const uint64_t *__restrict__ keys, const int64_t *__restrict__ excl,
                                 int64_t *__restrict__ starts, int64_t n_seg) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (i == 0 || keys[i] != keys[i - 1]) starts[excl[i]] = i;
    if (i == 0) starts[n_seg] = n;
}

__global__ void k_gather_xyz(int64_t n, const uint32_t *__restrict__ idx, const double *__restrict__ x,
                             const double *__restrict__ y, const double *__restrict__ z, double *__restrict__ xs,
                             double *__restrict__ ys, double *__restrict__ zs) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t j = idx[i];
    xs[i] = x[j];
    ys[i] = y[j];
    zs[i] = z[j];
}

__device__ __forceinline__ double dd_div_int(double hi, double lo, double n) {
    double q = hi / n;
    double r = fma(-q, n, hi) + lo;
    return q + r / n;
}

// One wavefront per cluster: compensated centroid, then centred scatter.
__global__ __launch_bounds__(256) void k_cluster_stats(int64_t C, const int64_t *__restrict__ starts,
                                                       const double *__restrict__ xs, const double *__restrict__ ys,
                                                       const double *__restrict__ zs,
                                                       const uint64_t *__restrict__ skeys, int32_t n_scans,
                                                       double *__restrict__ cN, double *__restrict__ cmu,
                                                       double *__restrict__ cS, int32_t *__restrict__ cvox,
                                                       int32_t *__restrict__ cscan) {
    int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    int lane = threadIdx.x & 63;
    if (c >= C) return;
    int64_t a = starts[c], b = starts[c + 1];
    double hx = 0, lx = 0, hy = 0, ly = 0, hz = 0, lz = 0;
    for (int64_t i = a + lane; i < b; i += 64) {
        dd_add(hx, lx, xs[i]);
        dd_add(hy, ly, ys[i]);
        dd_add(hz, lz, zs[i]);
    }
    wave_dd_sum(hx, lx);
    wave_dd_sum(hy, ly);
    wave_dd_sum(hz, lz);
    double n = (double)(b - a);
    double mx = dd_div_int(hx, lx, n), my = dd_div_int(hy, ly, n), mz = dd_div_int(hz, lz, n);
    double sxx = 0, sxy = 0, sxz = 0, syy = 0, syz = 0, szz = 0;
    for (int64_t i = a + lane; i < b; i += 64) {
        double dx = xs[i] - mx, dy = ys[i] - my, dz = zs[i] - mz;
        sxx = fma(dx, dx, sxx); sxy = fma(dx, dy, sxy); sxz = fma(dx, dz, sxz);
        syy = fma(dy, dy, syy); syz = fma(dy, dz, syz); szz = fma(dz, dz, szz);
    }
    sxx = wave_sum(sxx); sxy = wave_sum(sxy); sxz = wave_sum(sxz);
    syy = wave_sum(syy); syz = wave_sum(syz); szz = wave_sum(szz);
    if (lane == 0) {
        uint64_t key = skeys[a];
        cN[c] = n;
        cmu[3 * c + 0] = mx; cmu[3 * c + 1] = my; cmu[3 * c + 2] = mz;
        cS[6 * c + 0] = sxx; cS[6 * c + 1] = sxy; cS[6 * c + 2] = sxz;
        cS[6 * c + 3] = syy; cS[6 * c + 4] = syz; cS[6 * c + 5] = szz;
        cvox[c] = (int32_t)(key / (uint64_t)n_scans);
        cscan[c] = (int32_t)(key % (uint64_t)n_scans);
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

__global__ void k_center_sums(int64_t C, const uint32_t *__restrict__ order, const uint64_t *__restrict__ skeys,
                              const int64_t *__restrict__ count, const double *__restrict__ s1,
                              const double *__restrict__ s2, int32_t n_scans, double *__restrict__ cN,
                              double *__restrict__ cmu, double *__restrict__ cS, int32_t *__restrict__ cvox,
                              int32_t *__restrict__ cscan) {
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    uint32_t j = order[c];
    double n = (double)count[j];
    double s[3] = {s1[3 * (int64_t)j], s1[3 * (int64_t)j + 1], s1[3 * (int64_t)j + 2]};
    for (int k = 0; k < 3; k++) {
        double q = s[k] / n;
        double r = fma(-q, n, s[k]);
        cmu[3 * c + k] = q + r / n;
    }
    const double *Q = s2 + 6 * (int64_t)j;
    cS[6 * c + 0] = centre_entry(Q[0], s[0], s[0], n);
    cS[6 * c + 1] = centre_entry(Q[1], s[0], s[1], n);
    cS[6 * c + 2] = centre_entry(Q[2], s[0], s[2], n);
    cS[6 * c + 3] = centre_entry(Q[3], s[1], s[1], n);
    cS[6 * c + 4] = centre_entry(Q[4], s[1], s[2], n);
    cS[6 * c + 5] = centre_entry(Q[5], s[2], s[2], n);
    cN[c] = n;
    uint64_t key = skeys[c];
    cvox[c] = (int32_t)(key / (uint64_t)n_scans);
    cscan[c] = (int32_t)(key % (uint64_t)n_scans);
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

// Voxel-major copy, one thread per slot: the voxel's clusters lie together in
// the centred arrays, so a thread reads its rows in turn and the 64 lanes of a
// group write whole tile rows.  Padding lanes hold zeros.
__global__ __launch_bounds__(256) void k_fill_vox(int64_t n_slots, const GroupDesc *__restrict__ groups,
                                                  const int64_t *__restrict__ slot_start,
                                                  const double *__restrict__ cN, const double *__restrict__ cmu,
                                                  const double *__restrict__ cS, const int32_t *__restrict__ cscan,
                                                  char *__restrict__ tiles) {
    const int64_t sl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= n_slots) return;
    const GroupDesc g = groups[sl >> 6];
    const int lane = (int)(sl & 63);
    const bool used = lane < g.nvox;
    const int64_t c0 = used ? slot_start[sl] : 0;
    for (int k = 0; k < g.m; k++) {
        const int64_t d = g.cbase + 64LL * k + lane, c = c0 + k;
        double *o = tile_at<double>(tiles, d);
        o[0] = used ? cN[c] : 0.0;
        *tile_id<double>(tiles, d) = used ? cscan[c] : 0;
#pragma unroll
        for (int e = 0; e < 3; e++) o[64 * (1 + e)] = used ? cmu[3 * c + e] : 0.0;
#pragma unroll
        for (int e = 0; e < 6; e++) o[64 * (4 + e)] = used ? cS[6 * c + e] : 0.0;
    }
}

// Gather centred clusters into the pose-major layout.
__global__ void k_gather_pose(int64_t C, const uint32_t *__restrict__ order, const int32_t *__restrict__ slot_of,
                              const double *__restrict__ cN, const double *__restrict__ cmu,
                              const double *__restrict__ cS, char *__restrict__ tiles, int32_t *__restrict__ cidx) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= C) return;
    int64_t c = order[q];
    cidx[q] = (int32_t)c;
    double *o = tile_at<double>(tiles, q);
    o[0] = cN[c];
    *tile_id<double>(tiles, q) = slot_of[c];
#pragma unroll
    for (int k = 0; k < 3; k++) o[64 * (1 + k)] = cmu[3 * c + k];
#pragma unroll
    for (int k = 0; k < 6; k++) o[64 * (4 + k)] = cS[6 * c + k];
}

static inline unsigned nblk(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

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
__global__ __launch_bounds__(256) void k_fill_vox_f32(
    int64_t n_slots, const GroupDesc *__restrict__ groups, const int64_t *__restrict__ slot_start,
    const double *__restrict__ cN, const double *__restrict__ cmu, const double *__restrict__ cS,
    const int32_t *__restrict__ cscan, const double *__restrict__ ref_poses, double *__restrict__ vref,
    char *__restrict__ tiles, int32_t *__restrict__ err) {
    const int64_t sl = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sl >= n_slots) return;
    const GroupDesc g = groups[sl >> 6];
    const int lane = (int)(sl & 63);
    double *ref = vref + 4 * sl;
    if (lane >= g.nvox) {
        ref[0] = ref[1] = ref[2] = ref[3] = 0.0;
        for (int k = 0; k < g.m; k++) {
            const int64_t idx = g.cbase + 64LL * k + lane;
            float *o = tile_at<float>(tiles, idx);
#pragma unroll
            for (int e = 0; e < 10; e++) o[64 * e] = 0.0f;
            *tile_id<float>(tiles, idx) = 0;
        }
        return;
    }
    const int64_t c0 = slot_start[sl];
    double n = 0.0, c[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < g.m; k++) {
        Pose P0;
        load_pose(ref_poses, cscan[c0 + k], P0);
        double y[3];
        rot(P0.r, cmu + 3 * (c0 + k), y);
        const double nk = cN[c0 + k];
        n += nk;
#pragma unroll
        for (int q = 0; q < 3; q++) c[q] = fma(nk, y[q] + P0.t[q], c[q]);
    }
#pragma unroll
    for (int q = 0; q < 3; q++) c[q] /= n;
    int bad = 0;
    if (!(isfinite(c[0]) && isfinite(c[1]) && isfinite(c[2]))) bad |= 1;
    ref[0] = c[0]; ref[1] = c[1]; ref[2] = c[2]; ref[3] = 0.0;
    for (int k = 0; k < g.m; k++) {
        const int64_t idx = g.cbase + 64LL * k + lane;
        const int32_t j = cscan[c0 + k];
        Pose P0;
        load_pose(ref_poses, j, P0);
        float m32[3], S32[6];
        ref_frame_f32(P0, c, cmu + 3 * (c0 + k), cS + 6 * (c0 + k), m32, S32);
        float *o = tile_at<float>(tiles, idx);
#pragma unroll
        for (int e = 0; e < 3; e++) o[64 * (1 + e)] = m32[e];
#pragma unroll
        for (int e = 0; e < 6; e++) o[64 * (4 + e)] = S32[e];
        const double nk = cN[c0 + k];
        if (nk >= 16777216.0) bad |= 2;
        o[0] = (float)nk;
        *tile_id<float>(tiles, idx) = j;
    }
    if (bad) atomicOr(err, bad);
}

// Pose-major FP32 copy in the same reference frames.
__global__ void k_gather_pose_f32(int64_t C, const uint32_t *__restrict__ order, const int32_t *__restrict__ slot_of,
                                  const int32_t *__restrict__ cscan, const double *__restrict__ cN,
                                  const double *__restrict__ cmu, const double *__restrict__ cS,
                                  const double *__restrict__ vref, const double *__restrict__ ref_poses,
                                  char *__restrict__ tiles, int32_t *__restrict__ cidx) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= C) return;
    const int64_t c = order[q];
    cidx[q] = (int32_t)c;
    const int32_t sl = slot_of[c];
    Pose P0;
    load_pose(ref_poses, cscan[c], P0);
    const double mu[3] = {cmu[3 * c], cmu[3 * c + 1], cmu[3 * c + 2]};
    double S[6];
#pragma unroll
    for (int k = 0; k < 6; k++) S[k] = cS[6 * c + k];
    float m32[3], S32[6];
    ref_frame_f32(P0, vref + 4LL * sl, mu, S, m32, S32);
    float *o = tile_at<float>(tiles, q);
#pragma unroll
    for (int k = 0; k < 3; k++) o[64 * (1 + k)] = m32[k];
#pragma unroll
    for (int k = 0; k < 6; k++) o[64 * (4 + k)] = S32[k];
    o[0] = (float)cN[c];
    *tile_id<float>(tiles, q) = sl;
}

__global__ void k_validate_poses(int64_t n, const double *__restrict__ poses, int32_t *__restrict__ err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && !isfinite(poses[i])) atomicOr(err, 1);
}


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
    for (int32_t j = 0; j < N; j++) {
        chunk_ptr[j] = (int32_t)n;
        n += (P->h_pose_start[j + 1] - P->h_pose_start[j] + chunk_len - 1) / chunk_len;
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
// takes 2.7 ms.)

// One thread per voxel: the largest cluster count, and the first voxel that
// is observed from more than one window (err, or INT32_MAX).
__global__ __launch_bounds__(256) void k_plan_check(int32_t V, const int64_t *__restrict__ vstart,
                                                    const int32_t *__restrict__ cscan,
                                                    const int32_t *__restrict__ pose_window, int32_t W,
                                                    int32_t *__restrict__ max_m, int32_t *__restrict__ err) {
    const int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    int32_t m = 0;
    if (v < V) {
        const int64_t a = vstart[v], b = vstart[v + 1];
        m = (int32_t)(b - a);
        // the scans rise, and so do their windows
        if (W > 1 && pose_window[cscan[b - 1]] != pose_window[cscan[a]]) atomicMin(err, v);
    }
    m = -wave_min_i(-m);
    if ((threadIdx.x & 63) == 0) atomicMax(max_m, m);
}

// Sort key (window, m, first observing scan) of every voxel.
__global__ void k_plan_keys(int32_t V, const int64_t *__restrict__ vstart, const int32_t *__restrict__ cscan,
                            const int32_t *__restrict__ pose_window, int mbits, int sbits,
                            uint64_t *__restrict__ keys, uint32_t *__restrict__ vals) {
    const int32_t v = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (v >= V) return;
    const int64_t a = vstart[v];
    const uint64_t m = (uint64_t)(vstart[v + 1] - a), j = (uint64_t)cscan[a];
    keys[v] = (((uint64_t)pose_window[j] << mbits | m) << sbits) | j;
    vals[v] = (uint32_t)v;
}

__global__ void k_run_keys(int64_t R, const int64_t *__restrict__ starts, const uint64_t *__restrict__ keys,
                           int shift, uint64_t *__restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < R) out[r] = keys[starts[r]] >> shift;
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
    if (lane < nvox) {
        const int64_t a = vstart[order[r.first + v0 + lane]];
        s0 = cscan[a];
        s1 = -cscan[a + r.m - 1];
        slot_vox[sl] = cvox[a];
        slot_start[sl] = a;
        const int64_t u = r.ubase + r.m * (v0 + lane);
        for (int32_t k = 0; k < r.m; k++) {
            c_slot[a + k] = (int32_t)sl;
            keys[u + k] = (uint64_t)cscan[a + k];
            vals[u + k] = (uint32_t)(a + k);
        }
    } else {
        slot_vox[sl] = -1;
        slot_start[sl] = 0;
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

// First position of every scan in the sorted list (start[N] = C).
__global__ void k_pose_starts(int64_t C, int32_t N, const uint64_t *__restrict__ keys, int64_t *__restrict__ start) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= C) return;
    const int64_t j = (int64_t)keys[q];
    for (int64_t t = q ? (int64_t)keys[q - 1] + 1 : 0; t <= j; t++) start[t] = q;
    if (q == C - 1)
        for (int64_t t = j + 1; t <= N; t++) start[t] = C;
}

// Sort buffers of the build, at least as long as the cluster list.
struct BuildWork {
    uint64_t *keys;
    uint32_t *vals;
    char *ws;
    int64_t *total;   // device: one count
};

static ba_status read_count(int64_t *dst, const int64_t *src, hipStream_t s) {
    BA_HIP(hipMemcpyAsync(dst, src, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    return BA_OK;
}

static ba_status make_plan(Problem *P, const std::vector<int32_t> &scan_window, const BuildWork &bw, DevArena &keep,
                           hipStream_t s) {
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

    // voxels
    int64_t V64 = 0;
    BA_HIP(segment_count(P->c_vox, C, 0, bw.total, bw.ws, s));
    BA_TRY(read_count(&V64, bw.total, s));
    const int32_t V = (int32_t)V64;
    P->n_vox = V;
    int64_t *vstart;
    int32_t *d_chk;
    BA_TRY(tmp.alloc(&vstart, (int64_t)V + 1));
    BA_TRY(tmp.alloc(&d_chk, 2));
    BA_HIP(segment_write(P->c_vox, C, 0, (int64_t)V, vstart, (int32_t *)nullptr, bw.ws, s));
    int32_t chk[2] = {0, INT32_MAX};   // largest m, first offending voxel
    BA_HIP(hipMemcpyAsync(d_chk, chk, sizeof(chk), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_plan_check, dim3(nblk(V)), dim3(256), 0, s, V, vstart, P->c_scan, P->pose_window, W, d_chk,
                       d_chk + 1);
    BA_HIP(hipGetLastError());
    BA_HIP(hipMemcpyAsync(chk, d_chk, sizeof(chk), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    if (chk[1] != INT32_MAX) {
        int64_t a = 0;
        int32_t id = 0;
        BA_TRY(read_count(&a, vstart + chk[1], s));
        BA_HIP(hipMemcpyAsync(&id, P->c_vox + a, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        BA_HIP(hipStreamSynchronize(s));
        set_error("voxel %d is observed by scans of different windows", id);
        return BA_E_ARG;
    }
    P->max_m = chk[0];

    // voxel order: (window, m, first observing scan, voxel id), a stable sort;
    // then its runs of one window and one m
    const int sbits = bit_length((uint64_t)(N - 1)), mbits = bit_length((uint64_t)P->max_m);
    hipLaunchKernelGGL(k_plan_keys, dim3(nblk(V)), dim3(256), 0, s, V, vstart, P->c_scan, P->pose_window, mbits,
                       sbits, bw.keys, bw.vals);
    BA_HIP(radix_sort_pairs(bw.keys, bw.vals, V, sbits + mbits + bit_length((uint64_t)(W - 1)), bw.ws, s));
    int64_t R = 0;
    BA_HIP(segment_count((const uint64_t *)bw.keys, (int64_t)V, sbits, bw.total, bw.ws, s));
    BA_TRY(read_count(&R, bw.total, s));
    int64_t *d_rs;
    uint64_t *d_rk;
    uint32_t *order;
    PlanRun *d_runs;
    BA_TRY(tmp.alloc(&d_rs, R + 1));
    BA_TRY(tmp.alloc(&d_rk, R));
    BA_TRY(tmp.alloc(&order, V));
    BA_TRY(tmp.alloc(&d_runs, R));
    BA_HIP(segment_write((const uint64_t *)bw.keys, (int64_t)V, sbits, R, d_rs, (int32_t *)nullptr, bw.ws, s));
    hipLaunchKernelGGL(k_run_keys, dim3(nblk(R)), dim3(256), 0, s, R, d_rs, bw.keys, sbits, d_rk);
    BA_HIP(hipGetLastError());
    BA_HIP(hipMemcpyAsync(order, bw.vals, sizeof(uint32_t) * V, hipMemcpyDeviceToDevice, s));
    std::vector<int64_t> rs(R + 1);
    std::vector<uint64_t> rk(R);
    BA_HIP(hipMemcpyAsync(rs.data(), d_rs, sizeof(int64_t) * (R + 1), hipMemcpyDeviceToHost, s));
    BA_HIP(hipMemcpyAsync(rk.data(), d_rk, sizeof(uint64_t) * R, hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    std::vector<PlanRun> runs(R);
    std::vector<int32_t> win_group_ptr(W + 1, 0);
    std::vector<PlanMix> mix(W);
    int64_t cbase = 0, ubase = 0, G = 0;
    for (int64_t r = 0; r < R; r++) {
        PlanRun &q = runs[r];
        q.first = rs[r];
        q.len = rs[r + 1] - rs[r];
        q.m = (int32_t)(rk[r] & (((uint64_t)1 << mbits) - 1));
        q.window = (int32_t)(rk[r] >> mbits);
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
    hipLaunchKernelGGL(k_plan_groups, dim3(nblk(NS)), dim3(256), 0, s, P->n_groups, (int32_t)R, d_runs, order, vstart,
                       P->c_vox, P->c_scan, P->win_group_ptr, P->groups, P->vblocks, P->slot_vox, slot_start,
                       P->c_slot, bw.keys, bw.vals);
    hipLaunchKernelGGL(k_plan_mix, dim3(nblk(n_mix)), dim3(256), 0, s, n_mix, W, d_mix, P->vblocks_mix);
    // pose-major order (scan, slot): a stable sort by scan of that list (a
    // voxel's clusters have distinct scans)
    BA_HIP(radix_sort_pairs(bw.keys, bw.vals, C, sbits, bw.ws, s));
    hipLaunchKernelGGL(k_pose_starts, dim3(nblk(C)), dim3(256), 0, s, C, N, bw.keys, P->pose_start);
    BA_HIP(hipGetLastError());
    P->h_pose_start.resize(N + 1);
    BA_HIP(hipMemcpyAsync(P->h_pose_start.data(), P->pose_start, sizeof(int64_t) * (N + 1), hipMemcpyDeviceToHost, s));
    // the two copies of the clusters
    if (!f32) {
        hipLaunchKernelGGL(k_fill_vox, dim3(nblk(NS)), dim3(256), 0, s, NS, P->groups, slot_start, P->c_N, P->c_mu,
                           P->c_S, P->c_scan, P->v_tiles);
        hipLaunchKernelGGL(k_gather_pose, dim3(nblk(C)), dim3(256), 0, s, C, bw.vals, P->c_slot, P->c_N, P->c_mu,
                           P->c_S, P->p_tiles, P->p_cidx);
        BA_HIP(hipGetLastError());
        BA_HIP(hipStreamSynchronize(s));
        BA_TRY(replan_chunks(P, P->chunk_len, s));
        tmp.drained = true;
        return BA_OK;
    }
    BA_HIP(hipMemsetAsync(d_err, 0, sizeof(int32_t), s));
    hipLaunchKernelGGL(k_fill_vox_f32, dim3(nblk(NS)), dim3(256), 0, s, NS, P->groups, slot_start, P->c_N, P->c_mu,
                       P->c_S, P->c_scan, P->ref_poses, P->v_ref, P->v_tiles, d_err);
    hipLaunchKernelGGL(k_gather_pose_f32, dim3(nblk(C)), dim3(256), 0, s, C, bw.vals, P->c_slot, P->c_scan, P->c_N,
                       P->c_mu, P->c_S, P->v_ref, P->ref_poses, P->p_tiles, P->p_cidx);
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

static ba_status finish_build(Problem *P, DevArena &keep, const ba_build_options *opt, const BuildWork &bw,
                              hipStream_t s) {
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
        DevArena tmp;
        int32_t *d_err;
        BA_TRY(tmp.alloc(&d_err, 1));
        BA_HIP(hipMemsetAsync(d_err, 0, sizeof(int32_t), s));
        hipLaunchKernelGGL(k_validate_poses, dim3(nblk(np)), dim3(256), 0, s, np, P->ref_poses, d_err);
        BA_HIP(hipGetLastError());
        int32_t herr = 0;
        BA_HIP(hipMemcpyAsync(&herr, d_err, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        BA_HIP(hipStreamSynchronize(s));
        tmp.drained = true;
        if (herr) {
            set_error("ref_poses holds non-finite values");
            return BA_E_ARG;
        }
    }
    return make_plan(P, scan_window, bw, keep, s);
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
    int32_t *err;
    uint64_t *keys;
    uint32_t *vals;
    int64_t *flags, *total;
    BA_TRY(tmp.alloc(&err, 1));
    BA_TRY(tmp.alloc(&keys, n));
    BA_TRY(tmp.alloc(&vals, n));
    BA_TRY(tmp.alloc(&flags, n + 1));
    BA_TRY(tmp.alloc(&total, 1));
    size_t ws_bytes = std::max(radix_sort_workspace_bytes(n), scan_workspace_bytes(n));
    char *ws;
    BA_TRY(tmp.alloc(&ws, (int64_t)ws_bytes));
    BA_HIP(hipMemsetAsync(err, 0, sizeof(int32_t), s));
    hipLaunchKernelGGL(k_validate_points, dim3(nblk(n)), dim3(256), 0, s, n, pts->x, pts->y, pts->z, pts->scan,
                       pts->voxel, pts->n_scans, pts->n_voxels, err);
    hipLaunchKernelGGL(k_make_keys, dim3(nblk(n)), dim3(256), 0, s, n, pts->scan, pts->voxel, pts->n_scans, keys,
                       vals);
    BA_HIP(hipGetLastError());
    int32_t herr = 0;
    BA_HIP(hipMemcpyAsync(&herr, err, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    if (herr) {
        set_error("invalid points (flags 0x%x: 1 non-finite, 2 scan out of range, 4 voxel out of range)", herr);
        return BA_E_ARG;
    }
    int bits = bit_length((uint64_t)pts->n_voxels * (uint64_t)pts->n_scans - 1);
    BA_HIP(radix_sort_pairs(keys, vals, n, bits, ws, s));
    hipLaunchKernelGGL(k_head_flags, dim3(nblk(n)), dim3(256), 0, s, n, keys, flags);
    BA_HIP(exclusive_scan_i64(flags, flags, n, total, ws, s));
    int64_t C = 0;
    BA_HIP(hipMemcpyAsync(&C, total, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    P->n_clusters = C;
    int64_t *starts;
    double *xs, *ys, *zs;
    BA_TRY(tmp.alloc(&starts, C + 1));
    BA_TRY(tmp.alloc(&xs, n));
    BA_TRY(tmp.alloc(&ys, n));
    BA_TRY(tmp.alloc(&zs, n));
    hipLaunchKernelGGL(k_segment_starts, dim3(nblk(n)), dim3(256), 0, s, n, keys, flags, starts, C);
    hipLaunchKernelGGL(k_gather_xyz, dim3(nblk(n)), dim3(256), 0, s, n, vals, pts->x, pts->y, pts->z, xs, ys, zs);
    BA_TRY(keep.alloc(&P->c_N, C));
    BA_TRY(keep.alloc(&P->c_mu, 3 * C));
    BA_TRY(keep.alloc(&P->c_S, 6 * C));
    BA_TRY(keep.alloc(&P->c_vox, C));
    BA_TRY(keep.alloc(&P->c_scan, C));
    hipLaunchKernelGGL(k_cluster_stats, dim3(nblk(C * 64)), dim3(256), 0, s, C, starts, xs, ys, zs, keys,
                       pts->n_scans, P->c_N, P->c_mu, P->c_S, P->c_vox, P->c_scan);
    BA_HIP(hipGetLastError());
    BA_TRY(finish_build(P, keep, opt, BuildWork{keys, vals, ws, total}, s));
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
    int32_t *err;
    uint64_t *keys;
    uint32_t *vals;
    BA_TRY(tmp.alloc(&err, 1));
    BA_TRY(tmp.alloc(&keys, n));
    BA_TRY(tmp.alloc(&vals, n));
    char *ws;
    int64_t *total;
    BA_TRY(tmp.alloc(&ws, (int64_t)std::max(radix_sort_workspace_bytes(n), scan_workspace_bytes(n))));
    BA_TRY(tmp.alloc(&total, 1));
    BA_HIP(hipMemsetAsync(err, 0, sizeof(int32_t), s));
    hipLaunchKernelGGL(k_validate_sums, dim3(nblk(n)), dim3(256), 0, s, n, cs->voxel, cs->scan, cs->count, cs->sum,
                       cs->sumsq, cs->n_scans, cs->n_voxels, err);
    hipLaunchKernelGGL(k_make_keys, dim3(nblk(n)), dim3(256), 0, s, n, cs->scan, cs->voxel, cs->n_scans, keys, vals);
    int bits = bit_length((uint64_t)cs->n_voxels * (uint64_t)cs->n_scans - 1);
    BA_HIP(radix_sort_pairs(keys, vals, n, bits, ws, s));
    hipLaunchKernelGGL(k_dup_keys, dim3(nblk(n)), dim3(256), 0, s, n, keys, err);
    BA_HIP(hipGetLastError());
    int32_t herr = 0;
    BA_HIP(hipMemcpyAsync(&herr, err, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BA_HIP(hipStreamSynchronize(s));
    if (herr) {
        set_error("invalid clusters (flags 0x%x: 1 non-finite, 2 scan, 4 voxel, 8 count < 1, 16 duplicate pair)",
                  herr);
        return BA_E_ARG;
    }
    P->n_clusters = n;
    BA_TRY(keep.alloc(&P->c_N, n));
    BA_TRY(keep.alloc(&P->c_mu, 3 * n));
    BA_TRY(keep.alloc(&P->c_S, 6 * n));
    BA_TRY(keep.alloc(&P->c_vox, n));
    BA_TRY(keep.alloc(&P->c_scan, n));
    hipLaunchKernelGGL(k_center_sums, dim3(nblk(n)), dim3(256), 0, s, n, vals, keys, cs->count, cs->sum, cs->sumsq,
                       cs->n_scans, P->c_N, P->c_mu, P->c_S, P->c_vox, P->c_scan);
    BA_HIP(hipGetLastError());
    BA_TRY(finish_build(P, keep, opt, BuildWork{keys, vals, ws, total}, s));
    tmp.drained = true;   // the plan's last step waits for the stream
    return BA_OK;
}

}  // namespace ba
