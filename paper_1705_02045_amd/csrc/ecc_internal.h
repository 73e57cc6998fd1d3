// Internal declarations of libecc (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "ecc.h"

namespace ecc {

constexpr int kWave = 64;
constexpr uint32_t kStatusRange = ECC_STATUS_RANGE_BIT;
constexpr uint32_t kStatusNaN = 2u;  // a float image holds a NaN
// Device status block (one per workspace or stream): word 0 status, word 1
// its copy taken for the scan, word 2 the copy handed to the host, word 4 the
// scan's count of workgroups (zero between launches), words 8-9 a value
// range, from byte kStatusTotalsOffset on the totals of up to 1024 blocks of
// 64 columns.
constexpr size_t kStatusTotalsOffset = 128;
constexpr size_t kStatusBytes = kStatusTotalsOffset + 1024 * 8 + 128;
constexpr size_t kStatusMinMaxOffset = 32;  // two words: minimum and maximum of a 16-bit image

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Logical index of workgroup b of a grid of G: the workgroups of one XCD
// take one contiguous range of indices (a bijection of [0, G)), so that
// neighbouring work shares an L2.
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t G) {
    const uint32_t q = G / 8, rem = G % 8, x = b % 8;
    return x * q + (x < rem ? x : rem) + b / 8;
}

void set_error(const char *fmt, ...);
void g_err_clear();
int hip_fail(hipError_t e, const char *what);

#define ECC_HIP(call)                                  \
    do {                                               \
        hipError_t _e = (call);                        \
        if (_e != hipSuccess) return hip_fail(_e, #call); \
    } while (0)

// Source of axis-0 planes for one launch.  Plane p of a launch (buffer coordinates) is read at base + p * plane_bytes
// for p >= 0 and at lo_base + p * plane_bytes for p < 0: a launch can start in
// a second buffer that holds the planes just before `base` (the carried
// planes of a stream).  lo_base = base when there is no such buffer.
struct PlaneSrc {
    const uint8_t *base;
    const uint8_t *lo_base;
    int64_t plane_bytes;
};

// Integer-path view of an image: axis 0 is the walking axis, the remaining
// axes (at most two here) are the in-plane axes; nin = number of in-plane axes.
struct IntView {
    int nin;        // 1: plane is one row of n2 values; 2: plane is n1 rows of n2 values
    int64_t n0;     // planes in the whole image
    int32_t n1, n2; // in-plane extents (n1 = 1 when nin == 1)
};

// One launch of the integer kernel over planes [e0, e1) of a buffer.
struct IntJob {
    PlaneSrc src;
    IntView view;
    int32_t e0, e1;       // emitted planes, buffer coordinates
    int32_t lo_inf;       // plane e0-1 lies outside the image
    int32_t hi_inf;       // plane e1 lies outside the image
    int dtype;            // ECC_U8 or ECC_U14
    int invert;           // values read as M-1-v (largest-value convention)
    int32_t win_shift;    // ECC_U16: the launch counts bin = clamp(v - win_shift, 0, 16383)
    // ECC_U16 in 32768-bin passes: 2 = the values in [win_shift, win_shift +
    // 32768) are counted at bin = v - win_shift, the others skipped; 0 = a
    // window as above
    int range_pass;
    uint32_t *high_flag;  // range passes: set to 1 when a value >= 32768 is loaded (may be null)
};

// Tiling of the integer kernel (chosen by choose_int_tiling in ecc_api.cpp).
struct IntTiling {
    int rows;      // rows (nin == 2) or 64-wide x segments (nin == 1) per wave
    int mode;      // update form of the four-item groups (0..3, see ecc_int.hip)
    int pd;        // planes of raw loads in flight ahead of the compared plane
    int wx, wy;    // waves per workgroup along x and along y
    int zc;        // planes per tile
    int per_wg;    // tiles walked by one workgroup into one histogram (at most)
    int tile_stride;  // 0: a workgroup walks per_wg consecutive tiles; 1: tiles strided by the grid
    int grid;      // workgroups = ceil(tiles / per_wg)
    int pair = 1;  // row-pair layout allowed (used where the shape and alignment permit)
};

// Device scratch of one (device, stream) pair.
struct Workspace {
    int device = -1;
    void *stream = nullptr;
    int32_t *partial = nullptr;  // [grid][m] per-workgroup counts
    size_t partial_bytes = 0;
    int64_t *vcec = nullptr;     // [m] changes vector
    size_t vcec_bytes = 0;
    uint32_t *status = nullptr;  // device status block (kStatusBytes)
    // A pinned, coherent host block of 16 words: word 0, the status that the
    // scan writes (read after the stream is synchronized, without a
    // device-to-host copy); word 1, the 16-bit path's high-value flag; of the
    // float path words 2-3, the sort's record count, 4-11, the mask of the keys'
    // top bytes, 12-13, the number of distinct values found by bits, and 14, the
    // status with them.  With its device-side address.
    volatile uint32_t *host_status = nullptr;
    uint32_t *host_status_dev = nullptr;
    int64_t *chi_tmp = nullptr;  // [m] curve staging for host outputs
    size_t chi_tmp_bytes = 0;
    void *img_tmp = nullptr;     // device copy of a host image
    size_t img_tmp_bytes = 0;
    void *fbuf = nullptr;        // float path: keys, record regions, sort scratch, curve staging
    size_t fbuf_bytes = 0;
    void *frec = nullptr;        // float path: the dense records (two buffers) and their prefix
    size_t frec_bytes = 0;
    void *fbits = nullptr;       // float path: the bits of the distinct values
    size_t fbits_bytes = 0;
    void *dual_buf = nullptr;    // dual complex: per-face changes vectors
    size_t dual_buf_bytes = 0;
    int64_t *vcec16 = nullptr;   // [65536] changes vector of a 16-bit image (window passes)
    size_t vcec16_bytes = 0;
    // Fixed scratch (the entry point that allocates nothing): the buffers
    // above point into memory the library does not own and never grow;
    // ws_ensure fails instead of allocating.  max_grid caps the workgroup
    // count of a launch (0: no cap) so the count rows fit.
    bool fixed = false;
    int max_grid = 0;
};

// hipMalloc / hipHostMalloc through the allocation-failure injection hook
// (ECC_FAIL_ALLOC, ecc_api.cpp); every allocation of the library uses them.
hipError_t dev_malloc(void **p, size_t bytes);
// Device memory of device dev (the current one) from the blocks that finished
// ecc_stream objects left, or new: *got bytes, which cache_free() is given
// back with once no work uses them.  A request counts as an allocation
// whether or not a block was kept.
hipError_t cache_malloc(int dev, void **p, size_t bytes, size_t *got);
void cache_free(int dev, void *p, size_t bytes);
hipError_t cache_release(int dev);
hipError_t host_malloc(void **p, size_t bytes, unsigned flags);

int get_workspace(void *stream, Workspace **out);
int ensure_bytes(void **ptr, size_t *cap, size_t need);
// ensure_bytes for a buffer of ws: grows it, or on a fixed workspace fails
// with ECC_E_NOMEM when the buffer is smaller than need.
int ws_ensure(Workspace *ws, void **ptr, size_t *cap, size_t need);
// The stream-ordered integer curve of a device image (ecc_compute_async's
// work) with the scratch of ws.
int compute_async_ws(const void *image_dev, const ecc_dims *dims, ecc_dtype dtype, int64_t *chi_dev,
                     uint32_t *status_dev, hipStream_t stream, Workspace *ws);

int64_t threshold_count(int dtype);
int device_cu_count();

IntTiling choose_int_tiling(const IntView &v, int dtype, int64_t planes, int max_grid = 0);
// The tiling of a 16-bit launch in 32768-bin passes (IntJob::range_pass).
IntTiling range_pass_tiling(const IntView &v, int64_t planes);

// Kernels (ecc_int.hip / ecc_scan.hip).  All enqueue on `stream`.
// zero_vcec: when not null, workgroup 0 clears m int64 entries there first.
int launch_int_partial(const IntJob &job, const IntTiling &tl, int32_t *partial, uint32_t *status,
                       int64_t *zero_vcec, hipStream_t stream);
int launch_zero(void *p, size_t bytes, hipStream_t stream);
// 16-bit images (m = 65536): one launch counts one window of 16384 bins,
// bin = clamp(v - shift, 0, 16383); bins [klo, khi] are values
// [shift + klo, shift + khi] (bin 0 / 16383 are guards where values lie
// below / above the window).  Windows for values [vmin, vmax], at most
// kU16MaxWindows; returns their number.
struct U16Window {
    int32_t shift;
    int klo, khi;
};
constexpr int kU16MaxWindows = 5;  // 16383 + 3 * 16382 + 16383 >= 65536
int plan_u16_windows(uint32_t vmin, uint32_t vmax, U16Window *w);
// The whole curve of a device-resident 16-bit image on stream (two 32768-bin
// passes), the status copied to status_out (may be null).
int u16_curve_async(const void *image_dev, const IntView &v, int64_t *chi_dev, uint32_t *status_out,
                    hipStream_t stream);
// Column sums of the per-workgroup rows into vcec and, with do_scan, the
// prefix sum of vcec into chi (ecc_scan.hip).  The scan copies the status
// word to status_out (when not null) and clears it.
int launch_merge(const int32_t *partial, int rows, int m, int64_t *vcec, bool accumulate, bool do_scan, int64_t *chi,
                 uint32_t *status, uint32_t *status_out, hipStream_t stream, bool reverse = false,
                 bool negate = false);
// The same in parts for 16-bit images in 32768-bin passes: the column sums of
// a pass over the lower (0) or upper (1) half of 0..65535 into that half of
// vcec16 (clear, lower half only: the upper half is zeroed), then the scan.
int launch_merge_half(const int32_t *partial, int rows, int64_t *vcec16, int half, bool clear, uint32_t *status,
                      hipStream_t stream);
int launch_scan_halves(const int64_t *vcec16, int64_t *chi, uint32_t *status, uint32_t *status_out, hipStream_t stream);

// Copies the n0 x n1 x n2 sub-array of src starting at element `base` with
// element strides s0, s1, s2 into dst (contiguous, C order).
int launch_gather(const void *src, int elem, int64_t base, int64_t s0, int64_t s1, int64_t s2, int64_t n0,
                  int64_t n1, int64_t n2, void *dst, hipStream_t stream);
// Minimum and maximum of n uint16 values into out[0], out[1].
int launch_minmax_u16(const uint16_t *img, int64_t n, uint32_t *out, hipStream_t stream);
// out[t] = sign * sum_f (-1)^((neg_mask >> f) & 1) * curves[f * m + t], t < m.
// (faces f < 128: bit f of the pair {mask[0], mask[1]})
int launch_signed_sum(const int64_t *curves, int nf, const uint64_t neg_mask[2], const uint64_t skip_mask[2],
                      int sign, int m, int64_t *out, hipStream_t stream);
// A face of the box of at most two dimensions: elements base + i * sa + j *
// sb, i < na, j < nb (na or nb 0: no such axis), added with sign (+-1).
struct BoxFace {
    int64_t base, sa, sb, na, nb;
    int32_t sign;
};
constexpr int kFacesPerLaunch = 32;  // (passed by value)
// Largest-value changes of such faces of a u8 (elem 1, m = 256) or u14 (elem 2,
// m = 16384) image as box_face_rows() count rows (max_rows: at most that many
// per launch), entries at m-1-v (ecc_scan.hip).
int box_face_rows(const BoxFace *faces, int nfaces, int max_rows);
int launch_box_faces(const void *img, int elem, const BoxFace *faces, int nfaces, int max_rows, int32_t *rows,
                     hipStream_t stream);

bool normalize_int_view(const ecc_dims *dims, IntView *v, int *err_ndim_dropped);
int check_dims(const ecc_dims *dims, int64_t *total);
size_t elem_bytes(int dtype);

// Batched integer path (ecc_int.hip, ecc_scan.hip, ecc_batch.cpp).  The
// per-image kernel parameters are opaque to the host code: kparams_bytes()
// bytes each, filled by fill_kparams().
size_t kparams_bytes();
void fill_kparams(void *dst, const IntJob &job, const IntTiling &tl, int32_t *partial, uint32_t *status);
// Table of one batched run, built on the host and copied to the device as a
// whole (offsets in bytes from the table start).  The copy also resets the
// tile kernel's work counter.
struct BatchHeader {
    int32_t njobs;
    int32_t ntiles;           // workgroup-tiles over all images
    int32_t nitems;           // (image, 1024-column group) items of the merge
    uint32_t next_tile;       // work counter of the tile kernel (0 in the copied table)
    uint32_t off_kparams;     // KParams[njobs], kparams_bytes() each
    uint32_t off_tile_begin;  // int32[njobs + 1]: prefix of the images' tiles
    uint32_t off_kind;        // int32[njobs]: (dtype == U14) * 2 + (nin == 2)
    uint32_t off_merge;       // MergeJob[njobs]
    uint32_t off_item_begin;  // int32[njobs + 1]: prefix of the images' column groups
    uint32_t pad[7];
};
// One persistent launch over the tiles of every image of the table: `grid`
// workgroups take tiles from the work counter until none are left.
int launch_int_persistent(const void *table_dev, int grid, hipStream_t stream);
struct MergeJob {
    const int32_t *partial;  // [rows][m]
    int32_t rows;
    int32_t m;
    int64_t *vcec;           // [m] scratch
    int64_t *chi;            // [m] output
    uint32_t *status;        // device status word of the image (cleared here)
    uint32_t *status_out;    // optional copy for the caller
};
// Batched merge of the table's images: column sums into each image's vcec,
// then each image's scan into its curve (fixed grids, loops over the work).
int launch_batch_merge(const void *table_dev, int colsum_grid, int scan_grid, hipStream_t stream);

// Order-preserving 32-bit key of a float's bits: -0 is folded into +0; sign
// bit set: all bits flipped, else the sign bit set.
__device__ __forceinline__ uint32_t f32_key(uint32_t u) {
    u = __float_as_uint(__uint_as_float(u) + 0.0f);  // -0 + 0 = +0; other values stay (denormals too)
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// The inclusive prefix sum over a wave by lane shifts: within rows of 16, then
// the rows' last sums into the rows behind.  (__shfl_up goes through LDS: the
// batched scan, 16 sums per thread, takes 11 us for the 96 images of the mixed
// batch, 16 with it.)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t shifted(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t shifted(int64_t x) {
    return (int64_t)((uint64_t)shifted<CTRL, ROWS>((uint32_t)((uint64_t)x >> 32)) << 32 | shifted<CTRL, ROWS>((uint32_t)x));
}
template <typename T>
__device__ __forceinline__ T wave_prefix(T x) {
    x += shifted<0x111, 0xF>(x);  // row_shr by 1, 2, 4, 8
    x += shifted<0x112, 0xF>(x);
    x += shifted<0x114, 0xF>(x);
    x += shifted<0x118, 0xF>(x);
    x += shifted<0x142, 0xA>(x);  // the last lane of rows 0 and 2 to rows 1 and 3
    x += shifted<0x143, 0xC>(x);  // lane 31 to rows 2 and 3
    return x;
}

// Change kernel (ecc_change.hip): planes [e0, e1) of axis 0 of an image with
// one to three in-plane axes.
struct ChangeJob {
    PlaneSrc src;
    int nl;               // in-plane axes besides the last: 0, 1 (y) or 2 (y and z)
    int32_t nx, ny, nz;   // in-plane extents (1 where the axis is absent), the last axis nx
    int32_t e0, e1;       // planes to emit, buffer coordinates
    int32_t lo_inf, hi_inf;  // planes e0-1 and e1 lie outside the image
    int dtype;            // ECC_F32 or, with nl = 2, an integer type
    int invert;           // u8, u14: values read as m-1-v
};
// The float image's records (key << 32 | change as uint32, for the voxels
// whose change is not zero): region i holds its cnt[i] records from
// rec[i * region_slots] on.
int change_regions(const ChangeJob &job, int64_t *regions, int64_t *region_slots);
int launch_change_records(const ChangeJob &job, uint64_t *rec, uint32_t *cnt, hipStream_t stream);
// Integer images with four axes longer than 1: change_count_rows count rows of
// m int32 each, merged as the integer kernel's.  A value >= m sets kStatusRange.
int change_count_rows(const ChangeJob &job, int *rows);
int launch_change_counts(const ChangeJob &job, int32_t *partial, uint32_t *status, hipStream_t stream);

// Float path (ecc_float.hip, ecc_sort.hip).
// The change kernel's job for a float image.
int float_job(const float *img_dev, const ecc_dims *dims, ChangeJob *job);
// nz_off (regions + 1 entries): the regions' offsets, an exclusive scan of
// nz_cnt (sums: radix_scan_tiles(regions + 1)), and the record count into
// *total_host (host-mapped).
int launch_nz_total(const uint32_t *nz_cnt, uint32_t *nz_off, int64_t regions, uint32_t *sums, int64_t *total_host,
                    hipStream_t stream);
// The regions' records, densely.
int launch_nz_compact(const uint64_t *nz, const uint32_t *nz_cnt, const uint32_t *nz_off, int64_t regions,
                      int64_t region_slots, uint64_t *rec, hipStream_t stream);
// Tiles of the radix sort for n words of elem (4 or 8) bytes.
int64_t radix_tiles(int64_t n, int elem);
int64_t radix_scan_tiles(int64_t entries);
// Digit-table entries of a sort of n words of elem bytes (digits of up to
// 9 bits for keys, 8 for records); sums: radix_scan_tiles of that.
int64_t radix_count_entries(int64_t n, int elem);
// The keys (f32_key) of the n floats of img in tiles of kSplitTile, each in
// order of its keys' lowest 9 bits; starts: the first slot of each of the
// kSplitBuckets values of these bits, per tile; head: the mask of the top
// bytes that occur (8 words), the buckets' totals, then scratch.  The mask is also,
// complete at the event `noted`, at mask_host_dev (the device's view of 8
// words of host memory).  A NaN sets kStatusNaN.
constexpr int64_t kSplitTile = 16384;
constexpr int kSplitBuckets = 512;
size_t split_head_bytes(int64_t n);
// Sorts key[0] in place (four passes): the keys and starts of launch_split.
int radix_sort_keys(uint32_t *key[2], int64_t n, const uint16_t *starts, uint32_t *counts, uint32_t *sums,
                    hipStream_t stream);
int launch_split(const float *img, int64_t n, uint32_t *keys, uint16_t *starts, uint32_t *head, uint32_t *mask_host_dev,
                 uint32_t *status, hipEvent_t noted, hipStream_t stream);
// The distinct values and the curve at them (ecc_distinct.hip), for images
// whose keys hold at most kMaxDistinctBytes top bytes; keys, starts and head
// from launch_split, scratch: distinct_scratch_bytes.  Their number goes to
// *count (device memory) and, with the status word, to host-mapped memory.
constexpr int kMaxDistinctBytes = 32;
size_t distinct_scratch_bytes(int present, int64_t n);
int launch_distinct_curve(int64_t n, int present, const uint32_t *keys, const uint16_t *starts, const uint32_t *head,
                          void *scratch, const uint64_t *nz, const uint32_t *nz_cnt, int64_t regions,
                          int64_t region_slots, float *out_keys, int64_t *out_chi, int64_t *count, int64_t *count_host,
                          const uint32_t *status, uint32_t *status_host, hipStream_t stream);
// Sorts rec[0] in place (an even number of passes).
int radix_sort_records(uint64_t *rec[2], int64_t n, uint32_t *counts, uint32_t *sums, hipStream_t stream);
int64_t float_tiles(int64_t n);
// From the sorted keys and the sorted records: the K distinct keys as
// float32 (out_keys) and the curve (out_chi), K written to *kcount.
// tile_cnt: float_tiles(n) uint32; sums: radix_scan_tiles(float_tiles(n));
// tile_sum: float_tiles(n) int64; bound: float_tiles(n) + 1 int64; prefix:
// nnz int64.
int launch_float_curve(const uint32_t *key, int64_t n, const uint64_t *rec, int64_t nnz, int64_t *prefix,
                       uint32_t *tile_cnt, uint32_t *sums, int64_t *tile_sum, int64_t *bound, int64_t *kcount,
                       float *out_keys, int64_t *out_chi, hipStream_t stream);
// Exclusive scan of n uint32 in place; sums: radix_scan_tiles(n) entries.
int exclusive_scan_u32(uint32_t *a, int64_t n, uint32_t *sums, hipStream_t stream);
// Keys where chi changes, compacted (count written on the device).
int launch_change_points(const float *keys, const int64_t *chi, int64_t K, uint32_t *pos, uint32_t *sums,
                         float *out_keys, int64_t *out_chi, int64_t *count, hipStream_t stream);
// Float image to integer bins (elem = 1 or 2 bytes), NaN -> kStatusNaN.
int launch_quantize(const float *img, int64_t n, float lo, float scale, int m, int elem, void *out,
                    uint32_t *status, hipStream_t stream);

// Streaming internals for the serving loop (ecc_stream.cpp).
int stream_finish_async(ecc_stream *st, int64_t *chi_dev, uint32_t *status_dev);
int64_t stream_plane_bytes(const ecc_stream *st);

// Optional event timing of the per-voxel kernels (ecc_profile.cpp).
int profile_begin(hipStream_t s, void **token);
int profile_end(hipStream_t s, void *token);

}  // namespace ecc
