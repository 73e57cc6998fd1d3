// Float32 images (Sec. 3, "Other Ranges of Gray Values"): the values are not known
// in advance; the voxels whose change is not zero (a few in a hundred) leave
// (key, change) records (ecc_change.hip), and each change is added at its key's
// rank among the distinct values; a prefix sum over them gives the curve.  The
// distinct values are found by bits (ecc_distinct.hip) or, where the keys hold
// more than 32 top bytes (or the bits find no memory), by sorting every voxel's
// key (ecc_sort.hip); here are the compaction of the sort's records, the curve
// from the sorted keys and records, the change points and the quantisation.
//
// Keys: the canonical float (-0 folded into +0) mapped to an unsigned integer
// with the same order (f32_key).

#include "ecc_internal.h"

namespace ecc {

__device__ __forceinline__ float key_to_f32(uint32_t k) {
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// Axes of extent 1 are dropped (the complex of the others times unit
// intervals has the same curve), the first of the rest is walked.
int float_job(const float *img_dev, const ecc_dims *dims, ChangeJob *job) {
    int64_t ext[4];
    int d = 0;
    int64_t total = 1;
    for (int i = 0; i < dims->ndim; ++i) {
        total *= dims->n[i];
        if (dims->n[i] > 1) ext[d++] = dims->n[i];
    }
    if (total * 4 > (int64_t)UINT32_MAX) {
        set_error("float images are limited to 2^30 elements");
        return ECC_E_UNSUPPORTED;
    }
    *job = ChangeJob{};
    if (d == 0) ext[d++] = 1;
    job->dtype = ECC_F32;
    job->nl = d <= 2 ? 0 : d - 2;
    job->nx = (int32_t)ext[d - 1];
    job->ny = d >= 3 ? (int32_t)ext[d - 2] : 1;
    job->nz = d >= 4 ? (int32_t)ext[d - 3] : 1;
    job->src.base = job->src.lo_base = (const uint8_t *)img_dev;
    job->src.plane_bytes = (int64_t)job->nx * job->ny * job->nz * 4;
    job->e0 = 0;
    job->e1 = d == 1 ? 1 : (int32_t)ext[0];
    job->lo_inf = job->hi_inf = 1;
    return ECC_OK;
}

// ----------------------------------------------------------------------------
// The non-zero change records, from the workgroups' regions to one dense
// array of 64-bit words (key << 32 | change as uint32), sorted by key.

// After the exclusive scan of nz_off (region offsets; in place, from a copy
// of the counts with one entry more): the record count, written to
// host-mapped memory (read by the host after an event, to size the record
// sort).
__global__ void nz_total_kernel(const uint32_t *nz_off, int64_t regions, int64_t *total_host) {
    *total_host = (int64_t)nz_off[regions];
}
__global__ void __launch_bounds__(256) nz_copy_kernel(const uint32_t *__restrict__ nz_cnt, int64_t regions,
                                                      uint32_t *__restrict__ nz_off) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i <= regions) nz_off[i] = i < regions ? nz_cnt[i] : 0u;
}

int launch_nz_total(const uint32_t *nz_cnt, uint32_t *nz_off, int64_t regions, uint32_t *sums, int64_t *total_host,
                    hipStream_t stream) {
    hipLaunchKernelGGL(nz_copy_kernel, dim3((unsigned)((regions + 256) / 256)), dim3(256), 0, stream, nz_cnt, regions,
                       nz_off);
    ECC_HIP(hipGetLastError());
    int rc = exclusive_scan_u32(nz_off, regions + 1, sums, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(nz_total_kernel, dim3(1), dim3(1), 0, stream, (const uint32_t *)nz_off, regions, total_host);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// (a wave per region: a region is one wave's work in the change kernel, a
// few hundred records)
__global__ void __launch_bounds__(256) nz_compact_kernel(const uint64_t *__restrict__ nz,
                                                         const uint32_t *__restrict__ nz_cnt,
                                                         const uint32_t *__restrict__ nz_off, int64_t regions,
                                                         int64_t region_slots, uint64_t *__restrict__ rec) {
    const int64_t reg = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (reg >= regions) return;
    const uint32_t c = nz_cnt[reg];
    const int64_t src = reg * region_slots, dst = nz_off[reg];
    for (uint32_t i = threadIdx.x & 63; i < c; i += 64) rec[dst + i] = nz[src + i];
}

int launch_nz_compact(const uint64_t *nz, const uint32_t *nz_cnt, const uint32_t *nz_off, int64_t regions,
                      int64_t region_slots, uint64_t *rec, hipStream_t stream) {
    hipLaunchKernelGGL(nz_compact_kernel, dim3((unsigned)((regions + 3) / 4)), dim3(256), 0, stream, nz, nz_cnt, nz_off,
                       regions, region_slots, rec);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// ----------------------------------------------------------------------------
// After both sorts: the distinct keys and the curve.  chi after a distinct
// value v is the sum of the changes of the voxels with key <= v, i.e. the
// inclusive prefix P of the sorted records' changes at the last record with
// key <= v (0 if there is none).
//  1. ukey_count_kernel: per tile of kFTile sorted keys, the number of
//     last-of-key positions (a key differing from the next one), and its
//     exclusive scan: the tile's first rank;
//  2. rec_tile_sums_kernel, fscan_tiles_kernel, rec_prefix_kernel: P over
//     the records;
//  4. slice_bounds_kernel, curve_write_kernel: each last-of-key position
//     writes its key (as float) and chi at its rank.  Tile t of the keys,
//     [i0, i1), owns the key values in [key[i0], key[i1]) (from minus
//     infinity for the first tile, to plus infinity for the last): those
//     whose last position lies in the tile.  Its records are the ones in
//     [lower_bound(key[i0]), lower_bound(key[i1])) (one binary search per
//     tile, all tiles at once); the tile's distinct keys then look only at
//     that slice, from LDS when it is short.  The last tile writes K (known
//     on the device only).

constexpr int kFThreads = 256;
constexpr int kFItems = 16;
constexpr int kFTile = kFThreads * kFItems;

template <typename T>
__device__ T block_sum(T v, T *sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    T t = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
    __syncthreads();
    return t;
}

__device__ __forceinline__ bool last_of_key(const uint32_t *key, int64_t i, int64_t n) {
    return i == n - 1 || key[i] != key[i + 1];
}

// Last-of-key positions per tile: four 16-byte loads per thread (groups of
// four keys, coalesced across the wave), the key after each group from the
// next group (a cache hit).
__global__ void __launch_bounds__(kFThreads) ukey_count_kernel(const uint32_t *__restrict__ key, int64_t n,
                                                              uint32_t *__restrict__ tile_last) {
    __shared__ uint32_t sh[4];
    const int64_t t0 = (int64_t)blockIdx.x * kFTile;
    uint32_t l = 0;
    const bool vec = (reinterpret_cast<uintptr_t>(key) & 15u) == 0;
#pragma unroll
    for (int j = 0; j < kFItems / 4; ++j) {
        const int64_t g = t0 + ((int64_t)j * kFThreads + threadIdx.x) * 4;
        if (vec && g + 4 < n) {
            const uint4 w = *reinterpret_cast<const uint4 *>(key + g);
            const uint32_t nx = key[g + 4];
            l += (w.x != w.y) + (w.y != w.z) + (w.z != w.w) + (w.w != nx);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (g + q < n) l += last_of_key(key, g + q, n);
        }
    }
    l = block_sum(l, sh);
    if (threadIdx.x == 0) tile_last[blockIdx.x] = l;
}

__device__ __forceinline__ int32_t rec_change(uint64_t r) { return (int32_t)(uint32_t)r; }
__device__ __forceinline__ uint32_t rec_key(uint64_t r) { return (uint32_t)(r >> 32); }

// Change sums of record tiles [t * kFTile, (t+1) * kFTile).
__global__ void __launch_bounds__(kFThreads) rec_tile_sums_kernel(const uint64_t *__restrict__ rec, int64_t nnz,
                                                                 int64_t *__restrict__ tsum) {
    __shared__ int64_t sh[4];
    const int64_t t0 = (int64_t)blockIdx.x * kFTile;
    int64_t s = 0;
#pragma unroll
    for (int j = 0; j < kFItems; ++j) {
        const int64_t i = t0 + (int64_t)j * kFThreads + threadIdx.x;
        if (i < nnz) s += rec_change(rec[i]);
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) tsum[blockIdx.x] = s;
}

// Exclusive scans of both tile arrays in one workgroup of 1024 threads, in
// chunks of 16384 tiles: thread t holds tiles c0 + k * 1024 + t (k < 16:
// sixteen rows, every load and store coalesced).  Each row is scanned
// across the wave with shuffles; the wave totals per row go to LDS, where
// 32 threads turn them into per-wave prefixes and row totals.  The running
// carries are the same in all threads.  total_b receives the sum of b.  b may
// be null (then only a is scanned).
__global__ void __launch_bounds__(1024) fscan_tiles_kernel(int64_t *a, int64_t *b, int64_t nt, int64_t *total_b) {
    __shared__ int64_t wsa[16][17], wsb[16][17];  // [row][wave]
    __shared__ int64_t tota[16], totb[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t ca = 0, cb = 0;
    for (int64_t c0 = 0; c0 < nt; c0 += 1024 * 16) {
        int64_t xa[16], xb[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int64_t i = c0 + k * 1024 + tid;
            xa[k] = i < nt ? a[i] : 0;
            xb[k] = b && i < nt ? b[i] : 0;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int64_t ua = __shfl_up(xa[k], off, 64), ub = __shfl_up(xb[k], off, 64);
                if (lane >= off) {
                    xa[k] += ua;
                    xb[k] += ub;
                }
            }
        }
        if (lane == 63) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                wsa[k][wave] = xa[k];
                wsb[k][wave] = xb[k];
            }
        }
        __syncthreads();
        if (tid < 32) {  // row tid & 15 of array tid >> 4: exclusive prefix over the waves, row total
            int64_t(*ws)[17] = tid < 16 ? wsa : wsb;
            const int k = tid & 15;
            int64_t run = 0;
            for (int w = 0; w < 16; ++w) {
                const int64_t x = ws[k][w];
                ws[k][w] = run;
                run += x;
            }
            (tid < 16 ? tota : totb)[k] = run;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            // exclusive within the wave: the inclusive value of the lane below
            const int64_t pa = __shfl_up(xa[k], 1, 64), pb = __shfl_up(xb[k], 1, 64);
            const int64_t i = c0 + k * 1024 + tid;
            if (i < nt) {
                a[i] = ca + wsa[k][wave] + (lane > 0 ? pa : 0);
                if (b) b[i] = cb + wsb[k][wave] + (lane > 0 ? pb : 0);
            }
            ca += tota[k];
            cb += totb[k];
        }
        __syncthreads();  // the LDS rows are rewritten by the next chunk
    }
    if (tid == 0 && b && total_b) *total_b = cb;
}

// LDS slot of tile position i: one pad word per 16 entries, so that a
// thread's run of 16 (thread t reads 17 t + j) spreads over the banks.
__device__ __forceinline__ int fpad(int i) { return i + (i >> 4); }

// Inclusive prefix of the records' changes: the tile's changes staged in LDS
// (coalesced loads), a thread's run of kFItems scanned, the runs scanned over
// the workgroup with the tile's offset added, the prefixes staged back for
// coalesced stores.
__global__ void __launch_bounds__(kFThreads) rec_prefix_kernel(const uint64_t *__restrict__ rec, int64_t nnz,
                                                              const int64_t *__restrict__ tbase,
                                                              int64_t *__restrict__ prefix) {
    __shared__ int64_t st[kFTile + kFTile / 16];
    __shared__ int64_t ws[kFThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * kFTile;
#pragma unroll
    for (int j = 0; j < kFItems; ++j) {
        const int i = j * kFThreads + tid;
        st[fpad(i)] = t0 + i < nnz ? rec_change(rec[t0 + i]) : 0;
    }
    __syncthreads();
    const int r0 = tid * kFItems;
    int64_t v[kFItems], s = 0;
#pragma unroll
    for (int j = 0; j < kFItems; ++j) {
        v[j] = st[fpad(r0 + j)];
        s += v[j];
    }
    int64_t x = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t u = __shfl_up(x, off, 64);
        if (lane >= off) x += u;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    int64_t p = tbase[blockIdx.x] + x - s;
    for (int w = 0; w < wave; ++w) p += ws[w];
#pragma unroll
    for (int j = 0; j < kFItems; ++j) {
        p += v[j];
        st[fpad(r0 + j)] = p;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kFItems; ++j) {
        const int i = j * kFThreads + tid;
        if (t0 + i < nnz) prefix[t0 + i] = st[fpad(i)];
    }
}

// First record index in [lo, hi) whose key is >= k (strict: > k), or hi.
template <bool STRICT>
__device__ __forceinline__ int64_t rec_bound(const uint64_t *rec, int64_t lo, int64_t hi, uint32_t k) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        const uint32_t x = rec_key(rec[mid]);
        if (STRICT ? x <= k : x < k) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// bound[t] = the first record whose key is >= the first key of key tile t
// (0 for t = 0; the record count for t = nt): one thread per tile, all
// searches in flight together.
__global__ void __launch_bounds__(256) slice_bounds_kernel(const uint32_t *__restrict__ key, int64_t n, int64_t nt,
                                                           const uint64_t *__restrict__ rec, int64_t nnz,
                                                           int64_t *__restrict__ bound) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > nt) return;
    bound[t] = t == 0 ? 0 : t == nt ? nnz : rec_bound<false>(rec, 0, nnz, key[t * kFTile]);
}

// Records of a tile's slice kept in LDS (keys and prefixes): short slices
// (most tiles) in a small copy that leaves room for many workgroups per CU;
// the long ones (the tiles of the lowest and highest values, where the
// critical points gather) in a second launch with a large copy.
constexpr int kShortSlice = 512;
constexpr int kLongSlice = 4096;

// Thread t takes the run of kFItems sorted keys at t * kFItems of the tile
// (16-byte loads; the key after the run from the next lane, or from memory
// for the wave's last lane) and puts its distinct keys, in rank order, into
// LDS; the workgroup then takes them one per thread at a time (a binary
// search of the slice each, coalesced stores).  LONG = false takes the tiles
// whose slice has at most kShortSlice records, LONG = true the others: up to
// kLongSlice from LDS, beyond that (images with very few distinct values) one
// binary search in memory per distinct key.
template <bool LONG>
__global__ void __launch_bounds__(kFThreads) curve_write_kernel(const uint32_t *__restrict__ key, int64_t n,
                                                               int64_t nt, const uint32_t *__restrict__ tile_base,
                                                               const int64_t *__restrict__ bound,
                                                               const uint64_t *__restrict__ rec,
                                                               const int64_t *__restrict__ prefix,
                                                               float *__restrict__ out_keys,
                                                               int64_t *__restrict__ out_chi, int64_t *kcount) {
    constexpr int CAP = LONG ? kLongSlice : kShortSlice;
    __shared__ uint32_t sl[CAP];
    __shared__ int64_t sp[CAP + 1];  // sp[i] = P at record j0 + i - 1 (0 before the first)
    __shared__ uint32_t ck[kFTile];   // the tile's distinct keys
    __shared__ uint32_t ws[kFThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * kFTile;
    const int64_t j0 = bound[blockIdx.x], j1 = bound[blockIdx.x + 1];
    const int64_t len = j1 - j0;
    if ((len > kShortSlice) != LONG) return;  // (uniform) the other launch's tile
    const bool in_lds = len <= CAP;
    const int64_t base = tile_base[blockIdx.x];
    const int64_t i0 = t0 + (int64_t)tid * kFItems;
    uint32_t k[kFItems + 1];
    static_assert(kFItems % 4 == 0, "runs of whole 16-byte groups");
    if ((reinterpret_cast<uintptr_t>(key) & 15u) == 0 && i0 + kFItems <= n) {
        const uint4 *k4 = reinterpret_cast<const uint4 *>(key + i0);
#pragma unroll
        for (int q = 0; q < kFItems / 4; ++q) {
            const uint4 w = k4[q];
            k[4 * q] = w.x;
            k[4 * q + 1] = w.y;
            k[4 * q + 2] = w.z;
            k[4 * q + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kFItems; ++j) k[j] = i0 + j < n ? key[i0 + j] : 0u;
    }
    {
        const uint32_t nx = __shfl_down(k[0], 1, 64);  // the next lane's first key
        const int64_t after = i0 + kFItems;
        k[kFItems] = lane < 63 ? nx : (after < n ? key[after] : 0u);
    }
    if (in_lds) {
        for (int i = tid; i < (int)len; i += kFThreads) {
            sl[i] = rec_key(rec[j0 + i]);
            sp[i + 1] = prefix[j0 + i];
        }
        if (tid == 0) sp[0] = j0 > 0 ? prefix[j0 - 1] : 0;
    }
    uint32_t s = 0;
    bool last[kFItems];
#pragma unroll
    for (int j = 0; j < kFItems; ++j) {
        const int64_t i = i0 + j;
        last[j] = i < n && (i == n - 1 || k[j] != k[j + 1]);
        s += last[j];
    }
    uint32_t x = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(x, off, 64);
        if (lane >= off) x += u;
    }
    if (lane == 63) ws[wave] = x;
    __syncthreads();  // (also: the slice is staged)
    int64_t r = base + x - s;
    uint32_t cnt = 0;
    for (int w = 0; w < kFThreads / 64; ++w) {
        if (w < wave) r += ws[w];
        cnt += ws[w];
    }
    if (tid == 0 && (int64_t)blockIdx.x == nt - 1) *kcount = base + cnt;
    // the tile's distinct keys in rank order, then one per thread at a time:
    // a binary search of the slice each, coalesced stores
    const uint32_t rl = (uint32_t)(r - base);
    {
        uint32_t q = rl;
#pragma unroll
        for (int j = 0; j < kFItems; ++j)
            if (last[j]) ck[q++] = k[j];
    }
    __syncthreads();
    for (uint32_t q = tid; q < cnt; q += kFThreads) {
        const uint32_t v = ck[q];
        int64_t chi;
        if (in_lds) {
            int lo = 0, hi = (int)len;  // first record above v
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (sl[mid] <= v) lo = mid + 1;
                else hi = mid;
            }
            chi = sp[lo];
        } else {
            const int64_t u = rec_bound<true>(rec, j0, j1, v);
            chi = u > 0 ? prefix[u - 1] : 0;
        }
        out_keys[base + q] = key_to_f32(v);
        out_chi[base + q] = chi;
    }
}

int launch_float_curve(const uint32_t *key, int64_t n, const uint64_t *rec, int64_t nnz, int64_t *prefix,
                       uint32_t *tile_cnt, uint32_t *sums, int64_t *tile_sum, int64_t *bound, int64_t *kcount,
                       float *out_keys, int64_t *out_chi, hipStream_t stream) {
    const int64_t nt = (n + kFTile - 1) / kFTile;
    if (nt > INT32_MAX || nnz > n) {
        set_error("float curve: too many keys");
        return ECC_E_UNSUPPORTED;
    }
    // the distinct keys' first rank per key tile
    hipLaunchKernelGGL(ukey_count_kernel, dim3((unsigned)nt), dim3(kFThreads), 0, stream, key, n, tile_cnt);
    ECC_HIP(hipGetLastError());
    int rc = exclusive_scan_u32(tile_cnt, nt, sums, stream);
    if (rc) return rc;
    // the records' prefix
    const int64_t rt = (nnz + kFTile - 1) / kFTile;
    if (rt > 0) {
        hipLaunchKernelGGL(rec_tile_sums_kernel, dim3((unsigned)rt), dim3(kFThreads), 0, stream, rec, nnz, tile_sum);
        ECC_HIP(hipGetLastError());
        hipLaunchKernelGGL(fscan_tiles_kernel, dim3(1), dim3(1024), 0, stream, tile_sum, (int64_t *)nullptr, rt,
                           (int64_t *)nullptr);
        ECC_HIP(hipGetLastError());
        hipLaunchKernelGGL(rec_prefix_kernel, dim3((unsigned)rt), dim3(kFThreads), 0, stream, rec, nnz,
                           (const int64_t *)tile_sum, prefix);
        ECC_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(slice_bounds_kernel, dim3((unsigned)((nt + 256) / 256)), dim3(256), 0, stream, key, n, nt, rec,
                       nnz, bound);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(curve_write_kernel<false>, dim3((unsigned)nt), dim3(kFThreads), 0, stream, key, n, nt,
                       (const uint32_t *)tile_cnt, (const int64_t *)bound, rec, (const int64_t *)prefix, out_keys,
                       out_chi, kcount);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(curve_write_kernel<true>, dim3((unsigned)nt), dim3(kFThreads), 0, stream, key, n, nt,
                       (const uint32_t *)tile_cnt, (const int64_t *)bound, rec, (const int64_t *)prefix, out_keys,
                       out_chi, kcount);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

int64_t float_tiles(int64_t n) { return (n + kFTile - 1) / kFTile; }

// ----------------------------------------------------------------------------
// Change points of a float curve: the keys where chi differs from the
// previous key's (chi = 0 before the first key).

__device__ __forceinline__ uint32_t is_step(const int64_t *chi, int64_t k) {
    return chi[k] != (k > 0 ? chi[k - 1] : 0) ? 1u : 0u;
}

__global__ void __launch_bounds__(256) step_flags_kernel(const int64_t *__restrict__ chi, int64_t K,
                                                         uint32_t *__restrict__ pos) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += stride) pos[k] = is_step(chi, k);
}

__global__ void __launch_bounds__(256) step_scatter_kernel(const float *__restrict__ keys,
                                                           const int64_t *__restrict__ chi,
                                                           const uint32_t *__restrict__ pos, int64_t K,
                                                           float *__restrict__ out_keys,
                                                           int64_t *__restrict__ out_chi, int64_t *count) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += stride) {
        const uint32_t f = is_step(chi, k);
        if (f) {
            out_keys[pos[k]] = keys[k];
            out_chi[pos[k]] = chi[k];
        }
        if (k == K - 1) *count = (int64_t)pos[k] + f;
    }
}

// pos: K uint32 (positions, scratch); sums: radix_scan_tiles(K) uint32.
int launch_change_points(const float *keys, const int64_t *chi, int64_t K, uint32_t *pos, uint32_t *sums,
                         float *out_keys, int64_t *out_chi, int64_t *count, hipStream_t stream) {
    if (K <= 0) return ECC_OK;
    int64_t blocks = (K + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(step_flags_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, chi, K, pos);
    ECC_HIP(hipGetLastError());
    int rc = exclusive_scan_u32(pos, K, sums, stream);
    if (rc) return rc;
    hipLaunchKernelGGL(step_scatter_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, keys, chi,
                       (const uint32_t *)pos, K, out_keys, out_chi, count);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// ----------------------------------------------------------------------------
// Quantisation of a float image to integer bins: x = (v - lo) * scale in
// float32 (each operation rounded to nearest); bin 0 below x = 0 (and -inf),
// m-1 from x = m on (and +inf), else the integer part of x.  NaN sets the
// status bit and writes bin 0.

// (four values per load and store where the image starts at one: 1537 x 2048
// to 8 bits takes 4.8 us, 3.3 of them the memory's; a buffer that starts
// between two loads goes one value at a time)
template <typename T>
__global__ void __launch_bounds__(256) quantize_kernel(const float *__restrict__ img, int64_t n, float lo,
                                                       float scale, int m, T *__restrict__ out,
                                                       uint32_t *status) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool nan = false;
    auto bin = [&](float v) -> uint32_t {
        nan |= v != v;
        const float x = __fmul_rn(__fsub_rn(v, lo), scale);
        if (!(x >= 0.0f)) return 0u;
        if (x >= (float)m) return (uint32_t)(m - 1);
        return (uint32_t)x;
    };
    const int64_t quads = (reinterpret_cast<uintptr_t>(img) & 15u) == 0 ? n / 4 : 0;
    for (int64_t i = t; i < quads; i += stride) {
        const float4 v = reinterpret_cast<const float4 *>(img)[i];
        const uint32_t a = bin(v.x), b = bin(v.y), c = bin(v.z), d = bin(v.w);
        if constexpr (sizeof(T) == 1) reinterpret_cast<uint32_t *>(out)[i] = a | b << 8 | c << 16 | d << 24;
        else reinterpret_cast<uint2 *>(out)[i] = make_uint2(a | b << 16, c | d << 16);
    }
    for (int64_t i = 4 * quads + t; i < n; i += stride) out[i] = (T)bin(img[i]);
    if (__builtin_amdgcn_ballot_w64(nan) != 0 && (threadIdx.x & 63) == 0) atomicOr(status, kStatusNaN);
}

int launch_quantize(const float *img, int64_t n, float lo, float scale, int m, int elem, void *out,
                    uint32_t *status, hipStream_t stream) {
    const int64_t blocks = std::min<int64_t>((n + 1023) / 1024, 65536);
    if (elem == 1)
        hipLaunchKernelGGL(quantize_kernel<uint8_t>, dim3((unsigned)blocks), dim3(256), 0, stream, img, n, lo, scale,
                           m, (uint8_t *)out, status);
    else
        hipLaunchKernelGGL(quantize_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, img, n, lo,
                           scale, m, (uint16_t *)out, status);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

}  // namespace ecc
