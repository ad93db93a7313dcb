// Device-wide primitives for the one-time problem build (paper Sec. IV-A,
// "Standard Primitives": sort_by_key, exclusive_scan, scatter):
//   * exclusive prefix scan of int64 (reduce-then-scan, three launches);
//   * stable LSD radix sort of (uint64 key, uint32 value) pairs with 8-bit
//     digits: per-tile digit histograms, a scan of the (digit, tile) counts
//     and a stable scatter in which every wave ranks its own keys against a
//     digit table of its own, so equal keys keep their input order;
//   * runs of equal keys (count and starts).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

#include "ba_internal.hpp"

namespace ba {

// ---------------------------------------------------------------- scan
static constexpr int SCAN_THREADS = 256;
static constexpr int SCAN_IPT = 8;
static constexpr int SCAN_TILE = SCAN_THREADS * SCAN_IPT;

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane ? ~0ull >> (64 - lane) : 0ull; }

__device__ __forceinline__ int64_t wave_incl_scan(int64_t v) {
    int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t y = __shfl_up(v, o, 64);
        if (lane >= o) v += y;
    }
    return v;
}

// exclusive scan of one value per thread across a 256-thread block
__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t *lds_waves, int64_t &total) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t inc = wave_incl_scan(v);
    if (lane == 63) lds_waves[w] = inc;
    __syncthreads();
    int64_t base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < SCAN_THREADS / 64; k++) {
        int64_t s = lds_waves[k];
        if (k < w) base += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return base + inc - v;
}

template <class T>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(const T *__restrict__ in, int64_t n,
                                                              int64_t *__restrict__ bsum) {
    __shared__ int64_t lw[SCAN_THREADS / 64];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_IPT;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_IPT; k++)
        if (base + k < n) s += in[base + k];
    int64_t tot;
    block_excl_scan(s, lw, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// single block: exclusive scan of nb block sums, writes total to *total
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_top(int64_t *__restrict__ bsum, int64_t nb,
                                                           int64_t *__restrict__ total) {
    __shared__ int64_t lw[SCAN_THREADS / 64];
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += SCAN_TILE) {
        int64_t base = c0 + (int64_t)threadIdx.x * SCAN_IPT;
        int64_t v[SCAN_IPT];
        int64_t s = 0;
#pragma unroll
        for (int k = 0; k < SCAN_IPT; k++) {
            v[k] = (base + k < nb) ? bsum[base + k] : 0;
            s += v[k];
        }
        int64_t tot;
        int64_t ex = block_excl_scan(s, lw, tot);
        int64_t run = carry + ex;
#pragma unroll
        for (int k = 0; k < SCAN_IPT; k++) {
            if (base + k < nb) bsum[base + k] = run;
            run += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

template <class T>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_down(const T *__restrict__ in, int64_t n,
                                                            const int64_t *__restrict__ boff, T *__restrict__ out) {
    __shared__ int64_t lw[SCAN_THREADS / 64];
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_IPT;
    int64_t v[SCAN_IPT];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_IPT; k++) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        s += v[k];
    }
    int64_t tot;
    int64_t run = boff[blockIdx.x] + block_excl_scan(s, lw, tot);
#pragma unroll
    for (int k = 0; k < SCAN_IPT; k++) {
        if (base + k < n) out[base + k] = (T)run;
        run += v[k];
    }
}

size_t scan_workspace_bytes(int64_t n) {
    int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    return (size_t)(nb + 1) * sizeof(int64_t);
}

// out may alias in.  total (device pointer, may be null) receives the sum.
template <class T>
hipError_t exclusive_scan(const T *in, T *out, int64_t n, int64_t *total, void *ws, hipStream_t s) {
    int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    int64_t *bsum = (int64_t *)ws;
    if (n == 0) {
        if (total) return hipMemsetAsync(total, 0, sizeof(int64_t), s);
        return hipSuccess;
    }
    hipLaunchKernelGGL(k_scan_reduce<T>, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, s, in, n, bsum);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(SCAN_THREADS), 0, s, bsum, nb, total);
    hipLaunchKernelGGL(k_scan_down<T>, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, s, in, n, bsum, out);
    return hipGetLastError();
}

hipError_t exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, int64_t *total, void *ws, hipStream_t s) {
    return exclusive_scan<int64_t>(in, out, n, total, ws, s);
}

__global__ void k_iota(int64_t n, uint32_t *__restrict__ v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = (uint32_t)i;
}

// ---------------------------------------------------------------- segments
// Runs of equal (key >> shift) in a sorted key array, without a flag array:
// the heads are counted per tile from the keys, the tile counts scanned, and
// a second pass over the keys writes every run's first position.  Two reads of
// the keys (16 bytes an element) where flags, their scan and the scatter of
// the starts moved 72: 117M keys 1.13 -> 0.45 ms.  A wave takes 8 rows of 64
// keys, so the loads are whole lines and all in flight.
static constexpr int SEG_ROWS = SCAN_TILE / SCAN_THREADS;

// Heads of the wave's rows (bit l of h[r]: key 64 r + l of the wave starts a
// run); returns their number.
template <class K>
__device__ __forceinline__ int seg_heads(const K *__restrict__ keys, int64_t w0, int64_t n, int shift,
                                         uint64_t (&h)[SEG_ROWS]) {
    const int lane = threadIdx.x & 63;
    K cur[SEG_ROWS];
#pragma unroll
    for (int r = 0; r < SEG_ROWS; r++) {
        const int64_t i = w0 + 64 * r + lane;
        cur[r] = i < n ? keys[i] : K(0);
    }
    K last = (w0 > 0 && w0 < n) ? keys[w0 - 1] : K(0);   // the key before the row
    int c = 0;
#pragma unroll
    for (int r = 0; r < SEG_ROWS; r++) {
        const int64_t i = w0 + 64 * r + lane;
        K prev = __shfl_up(cur[r], 1, 64);
        if (lane == 0) prev = last;
        h[r] = __ballot(i < n && (i == 0 || (cur[r] >> shift) != (prev >> shift)));
        c += __popcll(h[r]);
        last = __shfl(cur[r], 63, 64);
    }
    return c;
}

template <class K>
__global__ __launch_bounds__(SCAN_THREADS) void k_seg_reduce(const K *__restrict__ keys, int64_t n, int shift,
                                                             int64_t *__restrict__ bsum) {
    __shared__ int lw[SCAN_THREADS / 64];
    const int w = threadIdx.x >> 6;
    uint64_t h[SEG_ROWS];
    const int c = seg_heads(keys, (int64_t)blockIdx.x * SCAN_TILE + w * (64 * SEG_ROWS), n, shift, h);
    if ((threadIdx.x & 63) == 0) lw[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int v = 0; v < SCAN_THREADS / 64; v++) tot += lw[v];
        bsum[blockIdx.x] = tot;
    }
}

template <class K>
__global__ __launch_bounds__(SCAN_THREADS) void k_seg_write(const K *__restrict__ keys, int64_t n, int shift,
                                                            const int64_t *__restrict__ boff,
                                                            const int64_t *__restrict__ total,
                                                            int64_t *__restrict__ starts) {
    __shared__ int lw[SCAN_THREADS / 64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t w0 = (int64_t)blockIdx.x * SCAN_TILE + w * (64 * SEG_ROWS);
    uint64_t h[SEG_ROWS];
    const int c = seg_heads(keys, w0, n, shift, h);
    if (lane == 0) lw[w] = c;
    __syncthreads();
    int64_t r0 = boff[blockIdx.x];
    for (int v = 0; v < w; v++) r0 += lw[v];
    const uint64_t below = lanes_below(lane);
#pragma unroll
    for (int r = 0; r < SEG_ROWS; r++) {
        if ((h[r] >> lane) & 1) starts[r0 + __popcll(h[r] & below)] = w0 + 64 * r + lane;
        r0 += __popcll(h[r]);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) starts[*total] = n;
}

// One tile of keys in one launch: the number of runs and, with starts, their
// first positions.
template <class K>
__global__ __launch_bounds__(SCAN_THREADS) void k_seg_one(const K *__restrict__ keys, int64_t n, int shift,
                                                          int64_t *__restrict__ total, int64_t *__restrict__ starts) {
    __shared__ int lw[SCAN_THREADS / 64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t w0 = w * (64 * SEG_ROWS);
    uint64_t h[SEG_ROWS];
    const int c = seg_heads(keys, w0, n, shift, h);
    if (lane == 0) lw[w] = c;
    __syncthreads();
    int64_t r0 = 0, all = 0;
    for (int v = 0; v < SCAN_THREADS / 64; v++) {
        r0 += v < w ? lw[v] : 0;
        all += lw[v];
    }
    if (threadIdx.x == 0) {
        *total = all;
        if (starts) starts[all] = n;
    }
    if (!starts) return;
    const uint64_t below = lanes_below(lane);
#pragma unroll
    for (int r = 0; r < SEG_ROWS; r++) {
        if ((h[r] >> lane) & 1) starts[r0 + __popcll(h[r] & below)] = w0 + 64 * r + lane;
        r0 += __popcll(h[r]);
    }
}

// total (device) receives the number of runs; ws as for a scan of n values.
template <class K>
hipError_t segment_count(const K *keys, int64_t n, int shift, int64_t *total, void *ws, hipStream_t s) {
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb == 1) {
        hipLaunchKernelGGL(k_seg_one<K>, dim3(1), dim3(SCAN_THREADS), 0, s, keys, n, shift, total, (int64_t *)nullptr);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_seg_reduce<K>, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, s, keys, n, shift, (int64_t *)ws);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(SCAN_THREADS), 0, s, (int64_t *)ws, nb, total);
    return hipGetLastError();
}

// starts[0 .. *total] (after segment_count with the same arguments and ws)
template <class K>
hipError_t segment_write(const K *keys, int64_t n, int shift, int64_t *total, int64_t *starts, void *ws,
                         hipStream_t s) {
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb == 1)
        hipLaunchKernelGGL(k_seg_one<K>, dim3(1), dim3(SCAN_THREADS), 0, s, keys, n, shift, total, starts);
    else
        hipLaunchKernelGGL(k_seg_write<K>, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, s, keys, n, shift,
                           (const int64_t *)ws, total, starts);
    return hipGetLastError();
}

// Both, for starts of at least as many entries as there can be runs, and one.
template <class K>
hipError_t segments(const K *keys, int64_t n, int shift, int64_t *total, int64_t *starts, void *ws, hipStream_t s) {
    if (n > SCAN_TILE) {
        const hipError_t e = segment_count(keys, n, shift, total, ws, s);
        if (e != hipSuccess) return e;
    }
    return segment_write(keys, n, shift, total, starts, ws, s);
}

template hipError_t segment_count<uint64_t>(const uint64_t *, int64_t, int, int64_t *, void *, hipStream_t);
template hipError_t segment_write<uint64_t>(const uint64_t *, int64_t, int, int64_t *, int64_t *, void *, hipStream_t);
template hipError_t segments<uint64_t>(const uint64_t *, int64_t, int, int64_t *, int64_t *, void *, hipStream_t);
template hipError_t segments<int32_t>(const int32_t *, int64_t, int, int64_t *, int64_t *, void *, hipStream_t);

// ---------------------------------------------------------------- radix sort
static constexpr int RS_THREADS = 256;
static constexpr int RS_WAVES = RS_THREADS / 64;
static constexpr int RS_IPT = 16;
static constexpr int RS_TILE = RS_THREADS * RS_IPT;
static constexpr int RS_BITS = 8;                 // bits per pass
static constexpr int RS_BINS = 1 << RS_BITS;      // one digit per thread of a block
static_assert(RS_BINS == RS_THREADS, "a block handles one digit per thread");

__device__ __forceinline__ int digit_of(uint64_t k, int shift) { return (int)((k >> shift) & (RS_BINS - 1)); }

// Lanes of the wave holding the same digit d (d == RS_BINS marks an empty
// slot): a ballot per bit of d, RS_BITS + 1 bits.
__device__ __forceinline__ uint64_t same_digit_lanes(int d) {
    uint64_t same = ~0ull;
#pragma unroll
    for (int b = 0; b <= RS_BITS; b++) {
        const bool bit = (d >> b) & 1;
        const uint64_t bal = __ballot(bit);
        same &= bit ? bal : ~bal;
    }
    return same;
}

// Digit counts of every tile of RS_TILE keys, hist[digit][tile].
__global__ __launch_bounds__(RS_THREADS) void k_radix_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                           uint32_t *__restrict__ hist, int64_t nblocks) {
    __shared__ uint32_t cnt[RS_BINS];
    const int t = threadIdx.x;
    cnt[t] = 0;
    __syncthreads();
    const int64_t tile0 = (int64_t)blockIdx.x * RS_TILE;
    if (tile0 + RS_TILE <= n) {
        const ulonglong2 *k2 = reinterpret_cast<const ulonglong2 *>(keys + tile0) + t;   // tiles are 32 KB apart
        ulonglong2 v[RS_IPT / 2];
#pragma unroll
        for (int k = 0; k < RS_IPT / 2; k++) v[k] = k2[k * RS_THREADS];
#pragma unroll
        for (int k = 0; k < RS_IPT / 2; k++) {
            atomicAdd(&cnt[digit_of(v[k].x, shift)], 1u);
            atomicAdd(&cnt[digit_of(v[k].y, shift)], 1u);
        }
    } else {
        for (int64_t i = tile0 + t; i < n; i += RS_THREADS) atomicAdd(&cnt[digit_of(keys[i], shift)], 1u);
    }
    __syncthreads();
    hist[(int64_t)t * nblocks + blockIdx.x] = cnt[t];
}

// Stable scatter of one tile.  Every wave ranks its 1024 keys in order: within
// a row by ballots, across its rows by its own digit counters (a wave's LDS
// operations are in order, so its rows follow each other without a barrier);
// one block scan then places the waves' digit groups behind each other, the
// tile is laid out by digit in LDS and written as one contiguous run per
// digit.  Four barriers a tile; ranking row by row over the whole block took
// three a row (49 a tile): 117M keys 1.25 ms a pass against 0.59 ms.
template <bool IOTA>
__global__ __launch_bounds__(RS_THREADS) void k_radix_scatter(const uint64_t *__restrict__ keys_in,
                                                              const uint32_t *__restrict__ vals_in, int64_t n,
                                                              int shift, const uint32_t *__restrict__ gofs,
                                                              int64_t nblocks, uint64_t *__restrict__ keys_out,
                                                              uint32_t *__restrict__ vals_out) {
    __shared__ uint64_t sk[RS_TILE];
    __shared__ uint32_t sv[RS_TILE];
    __shared__ uint32_t cnt[RS_WAVES][RS_BINS];
    __shared__ uint32_t shift_to[RS_BINS];   // output place of a digit's run minus its place in the tile (mod 2^32)
    __shared__ uint32_t wsum[RS_WAVES];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t tile0 = (int64_t)blockIdx.x * RS_TILE;
    const int tile_n = (int)(n - tile0 < RS_TILE ? n - tile0 : RS_TILE);
    const uint64_t below = lanes_below(lane);
    uint64_t key[RS_IPT];
    uint32_t val[RS_IPT];
    uint32_t rank[RS_IPT];
    const int64_t w0 = tile0 + w * (RS_TILE / RS_WAVES) + lane;
#pragma unroll
    for (int k = 0; k < RS_IPT; k++) {
        const int64_t i = w0 + 64 * k;
        key[k] = i < n ? keys_in[i] : 0ull;
        val[k] = IOTA ? (uint32_t)i : (i < n ? vals_in[i] : 0u);
    }
#pragma unroll
    for (int v = 0; v < RS_WAVES; v++) cnt[v][t] = 0;
    const uint32_t gbase = gofs[(int64_t)t * nblocks + blockIdx.x];
    __syncthreads();
    volatile uint32_t *mine = cnt[w];
#pragma unroll
    for (int k = 0; k < RS_IPT; k++) {
        const int d = w0 + 64 * k < n ? digit_of(key[k], shift) : RS_BINS;   // RS_BINS marks an empty slot
        const uint64_t same = same_digit_lanes(d);
        const uint32_t rw = (uint32_t)__popcll(same & below);
        const uint32_t c = d < RS_BINS ? mine[d] : 0u;
        rank[k] = c + rw;
        __builtin_amdgcn_wave_barrier();   // every lane has read before a group's first lane writes
        if (d < RS_BINS && rw == 0) mine[d] = c + (uint32_t)__popcll(same);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread t holds digit t: the waves' counts become their first places
    {
        uint32_t c[RS_WAVES], tot = 0;
#pragma unroll
        for (int v = 0; v < RS_WAVES; v++) {
            c[v] = cnt[v][t];
            tot += c[v];
        }
        uint32_t inc = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) wsum[w] = inc;
        __syncthreads();
        uint32_t at = inc - tot;
        for (int v = 0; v < w; v++) at += wsum[v];
        shift_to[t] = gbase - at;
#pragma unroll
        for (int v = 0; v < RS_WAVES; v++) {
            cnt[v][t] = at;
            at += c[v];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RS_IPT; k++) {
        if (w0 + 64 * k < n) {
            const uint32_t p = cnt[w][digit_of(key[k], shift)] + rank[k];
            if (p < (uint32_t)RS_TILE) {
                sk[p] = key[k];
                sv[p] = val[k];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RS_IPT; k++) {
        const int j = k * RS_THREADS + t;
        if (j < tile_n) {
            const uint64_t kk = sk[j];
            const uint32_t pos = shift_to[digit_of(kk, shift)] + (uint32_t)j;
            if (pos < n) {
                keys_out[pos] = kk;
                vals_out[pos] = sv[j];
            }
        }
    }
}

// A sort of at most one tile in one launch: all passes in LDS, the waves taking
// equal shares of rows.  Five launches a pass are most of the time of a small
// problem's build: 270 voxels of four clusters 0.36 ms, and 0.22 with this and two
// waits fewer in the plan (0.30 with the plan made on the host).
template <bool IOTA>
__global__ __launch_bounds__(RS_THREADS) void k_radix_one(uint64_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                                          int n, int lo, int passes) {
    __shared__ uint64_t sk[RS_TILE];
    __shared__ uint32_t sv[RS_TILE];
    __shared__ uint32_t cnt[RS_WAVES][RS_BINS];
    __shared__ uint32_t wsum[RS_WAVES];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int rows = (n + RS_THREADS - 1) / RS_THREADS;   // of 64 keys per wave, at most RS_IPT
    const int w0 = w * rows * 64 + lane;
    const uint64_t below = lanes_below(lane);
    for (int j = t; j < n; j += RS_THREADS) {
        sk[j] = keys[j];
        sv[j] = IOTA ? (uint32_t)j : vals[j];
    }
    __syncthreads();
    volatile uint32_t *mine = cnt[w];
    for (int pass = 0; pass < passes; pass++) {
        const int shift = lo + RS_BITS * pass;
        uint64_t key[RS_IPT];
        uint32_t val[RS_IPT], rank[RS_IPT];
#pragma unroll
        for (int v = 0; v < RS_WAVES; v++) cnt[v][t] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RS_IPT; k++) {
            if (k >= rows) break;
            const bool has = w0 + 64 * k < n;
            key[k] = has ? sk[w0 + 64 * k] : 0ull;
            val[k] = has ? sv[w0 + 64 * k] : 0u;
            const int d = has ? digit_of(key[k], shift) : RS_BINS;   // RS_BINS marks an empty slot
            const uint64_t same = same_digit_lanes(d);
            const uint32_t rw = (uint32_t)__popcll(same & below);
            const uint32_t c = d < RS_BINS ? mine[d] : 0u;
            rank[k] = c + rw;
            __builtin_amdgcn_wave_barrier();   // every lane has read before a group's first lane writes
            if (d < RS_BINS && rw == 0) mine[d] = c + (uint32_t)__popcll(same);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // thread t holds digit t: the waves' counts become their first places
        uint32_t c[RS_WAVES], tot = 0;
#pragma unroll
        for (int v = 0; v < RS_WAVES; v++) {
            c[v] = cnt[v][t];
            tot += c[v];
        }
        uint32_t inc = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) wsum[w] = inc;
        __syncthreads();
        uint32_t at = inc - tot;
        for (int v = 0; v < w; v++) at += wsum[v];
#pragma unroll
        for (int v = 0; v < RS_WAVES; v++) {
            cnt[v][t] = at;
            at += c[v];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RS_IPT; k++) {
            if (k >= rows) break;
            if (w0 + 64 * k < n) {
                const uint32_t p = cnt[w][digit_of(key[k], shift)] + rank[k];
                if (p < (uint32_t)RS_TILE) {
                    sk[p] = key[k];
                    sv[p] = val[k];
                }
            }
        }
        __syncthreads();
    }
    for (int j = t; j < n; j += RS_THREADS) {
        keys[j] = sk[j];
        vals[j] = sv[j];
    }
}

size_t radix_sort_workspace_bytes(int64_t n) {
    const int64_t nb = (n + RS_TILE - 1) / RS_TILE;
    return align_up((size_t)nb * RS_BINS * sizeof(uint32_t), 256) + align_up(scan_workspace_bytes(nb * RS_BINS), 256);
}

// Sorts (keys, vals) by the `bits` bits of the keys from bit lo on (stable).  The arrays
// change places with their second halves as the passes go: the result is in
// b.keys and b.vals.  iota: vals are 0 .. n-1 and need not be filled.  Counts
// and positions are 32 bits (n < 2^32).
hipError_t radix_sort_pairs(SortBuf &b, int64_t n, int lo, int bits, bool iota, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t nb = (n + RS_TILE - 1) / RS_TILE;
    uint32_t *hist = (uint32_t *)b.ws;
    void *scan_ws = b.ws + align_up((size_t)nb * RS_BINS * sizeof(uint32_t), 256);
    const int passes = n > 1 ? (bits + RS_BITS - 1) / RS_BITS : 0;
    if (nb == 1 && passes > 0) {
        if (iota)
            hipLaunchKernelGGL(k_radix_one<true>, dim3(1), dim3(RS_THREADS), 0, s, b.keys, b.vals, (int)n, lo, passes);
        else
            hipLaunchKernelGGL(k_radix_one<false>, dim3(1), dim3(RS_THREADS), 0, s, b.keys, b.vals, (int)n, lo, passes);
        return hipGetLastError();
    }
    if (passes <= 0 && iota) hipLaunchKernelGGL(k_iota, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, b.vals);
    for (int pass = 0; pass < passes; pass++) {
        const int shift = lo + RS_BITS * pass;
        hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nb), dim3(RS_THREADS), 0, s, b.keys, n, shift, hist, nb);
        hipError_t e = exclusive_scan<uint32_t>(hist, hist, nb * RS_BINS, nullptr, scan_ws, s);
        if (e != hipSuccess) return e;
        if (iota && pass == 0)
            hipLaunchKernelGGL(k_radix_scatter<true>, dim3((unsigned)nb), dim3(RS_THREADS), 0, s, b.keys, b.vals, n,
                               shift, hist, nb, b.keys2, b.vals2);
        else
            hipLaunchKernelGGL(k_radix_scatter<false>, dim3((unsigned)nb), dim3(RS_THREADS), 0, s, b.keys, b.vals, n,
                               shift, hist, nb, b.keys2, b.vals2);
        std::swap(b.keys, b.keys2);
        std::swap(b.vals, b.vals2);
    }
    return hipGetLastError();
}

ba_status SortBuf::alloc(DevArena &a, int64_t cap) {
    BA_TRY(a.alloc(&keys, cap));
    BA_TRY(a.alloc(&vals, cap));
    BA_TRY(a.alloc(&keys2, cap));
    BA_TRY(a.alloc(&vals2, cap));
    BA_TRY(a.alloc(&ws, (int64_t)std::max(radix_sort_workspace_bytes(cap), scan_workspace_bytes(cap))));
    BA_TRY(a.alloc(&total, 1));
    return BA_OK;
}

}  // namespace ba
