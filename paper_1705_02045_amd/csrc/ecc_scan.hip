// Merging the per-workgroup change vectors and the prefix sum (Sec. 3,
// "Post-Processing": the VCECs of all workers are summed and the curve is
// their running sum).
#include "ecc_internal.h"

namespace ecc {

__global__ void zero_kernel(uint32_t *p, size_t words) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

int launch_zero(void *p, size_t bytes, hipStream_t stream) {
    if (bytes % 4) {
        set_error("launch_zero: size %zu not a multiple of 4", bytes);
        return ECC_E_ARG;
    }
    const size_t words = bytes / 4;
    const int threads = 256;
    int blocks = (int)((words + threads - 1) / threads);
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(threads), 0, stream, (uint32_t *)p, words);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// Merge of the per-workgroup rows [rows][m] (int32) into the int64 change
// vector and its prefix sum, in kernels that follow each other on the stream
// (the kernel boundary orders their memory):
//  1. colsum_kernel: a workgroup sums all rows of 64 columns (64 rows at a
//     time, 16 threads of 4 columns each: 256-byte runs; 16 rows at a time
//     where there are at most 64, with a quarter of the threads to start) into
//     vcec and, for a scan, their total into totals; before a scan it also
//     hands the status word over (status[1]) and clears it;
//  2. scan_kernel: a workgroup scans 1024 columns, from the sum of the totals
//     before them.
// Two launches where the sums of some rows at a time, their fold with the
// scan of 1024 columns and the offsets of those took three of 4 to 5 us each
// at least (117 rows of 16384 columns: 10.8 -> 8.5 us, a 97 x 130 x 75 call
// 39.7 -> 38.3 us; 1024 rows: 12.8 + 6.2 + 5.6 -> 13.9 + 5.3 us).
// With `reverse`, column c of the rows lands at m-1-c (the largest-value
// convention: the kernel counted at m-1-value); with `negate` the sums change
// sign.  vcec is overwritten, or added to with `accumulate`.
// clear (may be null): m further entries to set to zero, with their totals.
constexpr int kColBlock = 64;
template <int RG>
__global__ void __launch_bounds__(16 * RG) colsum_kernel(const int32_t *__restrict__ partial, int rows, int m,
                                                         int64_t *__restrict__ vcec, int accumulate, int reverse, int negate,
                                                         int64_t *__restrict__ totals, int64_t *__restrict__ clear,
                                                         int hand, uint32_t *status) {
    constexpr int kWaves = RG / 4;
    __shared__ int64_t part[kWaves][kColBlock];  // per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (hand && blockIdx.x == 0 && tid == 0) {
        status[1] = status[0];
        status[0] = 0u;
    }
    const int c4 = tid & 15;
    const size_t stride4 = (size_t)m / 4;
    const int4 *p = reinterpret_cast<const int4 *>(partial) + (size_t)blockIdx.x * (kColBlock / 4) + c4;
    int64_t v[4] = {0, 0, 0, 0};
    int r = tid >> 4;
    for (; r + 3 * RG < rows; r += 4 * RG) {
        int4 a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = p[(size_t)(r + u * RG) * stride4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[0] += a[u].x;
            v[1] += a[u].y;
            v[2] += a[u].z;
            v[3] += a[u].w;
        }
    }
    for (; r < rows; r += RG) {
        const int4 a = p[(size_t)r * stride4];
        v[0] += a.x;
        v[1] += a.y;
        v[2] += a.z;
        v[3] += a.w;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] += __shfl_xor(v[j], 16, 64);
        v[j] += __shfl_xor(v[j], 32, 64);
        if (lane < 16) part[wave][c4 * 4 + j] = v[j];
    }
    __syncthreads();
    if (tid >= kColBlock) return;
    int64_t s = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += part[w][tid];
    const int c = blockIdx.x * kColBlock + tid;
    const int at = reverse ? m - 1 - c : c;
    if (negate) s = -s;
    if (accumulate) s += vcec[at];
    vcec[at] = s;
    if (clear != nullptr) {
        clear[c] = 0;
        if (tid == 0) totals[gridDim.x + blockIdx.x] = 0;
    }
    if (totals == nullptr) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (tid == 0) totals[reverse ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x] = s;
}

// Sum over the workgroup's 1024 threads, in every thread.
__device__ __forceinline__ int64_t block_sum_1024(int64_t v, int64_t *sh) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += sh[w];
    __syncthreads();
    return t;
}

// Columns [1024 b, 1024 b + 1024) of the curve.  With totals (at most 1024 of
// them) the columns before come from those, without from vcec itself.  The
// status comes from status[1] where the column sums have handed it over, else
// from the status word, which the last workgroup to have read it clears
// (status[4] counts them).  The curve is written only with a clear status.
__global__ void __launch_bounds__(1024) scan_kernel(const int64_t *__restrict__ vcec, int m,
                                                    const int64_t *__restrict__ totals, int handed,
                                                    int64_t *__restrict__ chi, uint32_t *status, uint32_t *status_out) {
    __shared__ int64_t sh[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = blockIdx.x * 1024;
    const int64_t v = c0 + tid < m ? vcec[c0 + tid] : 0;
    const uint32_t stv = handed ? status[1] : *(volatile uint32_t *)status;
    int64_t before = 0;
    if (totals != nullptr) {
        if (tid < c0 / kColBlock) before = totals[tid];
    } else {
        int c = tid;
        for (; c + 3 * 1024 < c0; c += 4 * 1024) {
            int64_t a[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = vcec[c + u * 1024];
            before += a[0] + a[1] + a[2] + a[3];
        }
        for (; c < c0; c += 1024) before += vcec[c];
    }
    before = block_sum_1024(before, sh);
    int64_t x = v;
    x = wave_prefix(x);
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before += sh[w];
    if (stv == 0 && c0 + tid < m) chi[c0 + tid] = before + x;
    if (blockIdx.x == 0 && tid == 0 && status_out) *status_out = stv;
    if (!handed && tid == 0) {
        // (every thread of this workgroup has read the status word: the
        // barriers above follow the reads)
        if (atomicAdd(&status[4], 1u) == gridDim.x - 1) {
            status[4] = 0u;
            status[0] = 0u;
        }
    }
}

// ----------------------------------------------------------------------------
// Batched merge over the images of a batch table (fixed grids: the graph of
// a batched run does not change with its contents).
// batch_colsum_kernel: item i = (image j, 1024-column group g), j found in
// the table's item prefix: sums image j's rows over those columns into its
// vcec.  batch_scan_kernel: image j (blocks loop over images) writes its
// curve if its status word is clear, copies the status out and clears it.

__device__ __forceinline__ int find_prefix(const int32_t *begin, int n, int v) {
    int lo = 0, hi = n - 1;  // last j with begin[j] <= v
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (begin[mid] <= v) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256) batch_colsum_kernel(const uint8_t *__restrict__ table) {
    const BatchHeader *H = (const BatchHeader *)table;
    const MergeJob *jobs = (const MergeJob *)(table + H->off_merge);
    const int32_t *item_begin = (const int32_t *)(table + H->off_item_begin);
    for (int i = blockIdx.x; i < H->nitems; i += gridDim.x) {
        const int j = __builtin_amdgcn_readfirstlane(find_prefix(item_begin, H->njobs, i));
        const MergeJob J = jobs[j];
        const int c0 = (i - item_begin[j]) * 1024 + threadIdx.x * 4;
        if (c0 >= J.m) continue;
        const int4 *p = reinterpret_cast<const int4 *>(J.partial);
        const size_t stride4 = (size_t)J.m / 4;
        int64_t s0 = 0, s1 = 0, s2 = 0, s3 = 0;
        int r = 0;
        for (; r + 8 <= J.rows; r += 8) {  // eight rows of loads in flight
            int4 a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = p[(size_t)(r + u) * stride4 + c0 / 4];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                s0 += a[u].x;
                s1 += a[u].y;
                s2 += a[u].z;
                s3 += a[u].w;
            }
        }
        for (; r < J.rows; ++r) {
            const int4 a = p[(size_t)r * stride4 + c0 / 4];
            s0 += a.x;
            s1 += a.y;
            s2 += a.z;
            s3 += a.w;
        }
        J.vcec[c0] = s0;
        J.vcec[c0 + 1] = s1;
        J.vcec[c0 + 2] = s2;
        J.vcec[c0 + 3] = s3;
    }
}

// One image per workgroup of 1024 threads, chunks of 16384 entries: thread t
// holds entries c0 + k * 1024 + t (k < 16: sixteen rows, every load and
// store coalesced).  Each row is scanned across the wave with shuffles; the
// wave totals per row go to LDS, where 16 threads turn them into per-wave
// prefixes and row totals; every thread then adds the rows before its row and
// the waves before its wave.  The running carry is the same in all threads.
__global__ void __launch_bounds__(1024) batch_scan_kernel(const uint8_t *__restrict__ table) {
    __shared__ int64_t ws[16][17];   // [row][wave]: wave totals, then exclusive prefixes over the waves
    __shared__ int64_t rowtot[16];
    const BatchHeader *H = (const BatchHeader *)table;
    const MergeJob *jobs = (const MergeJob *)(table + H->off_merge);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int jb = blockIdx.x; jb < H->njobs; jb += gridDim.x) {
        const MergeJob J = jobs[jb];
        const uint32_t stv = *J.status;
        __syncthreads();  // every wave holds the status before thread 0 clears it below
        if (stv == 0) {
            int64_t carry = 0;
            for (int c0 = 0; c0 < J.m; c0 += 1024 * 16) {
                int64_t v[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int i = c0 + k * 1024 + tid;
                    v[k] = i < J.m ? J.vcec[i] : 0;
                }
#pragma unroll
                for (int k = 0; k < 16; ++k) v[k] = wave_prefix(v[k]);
                if (lane == 63) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) ws[k][wave] = v[k];
                }
                __syncthreads();
                if (tid < 16) {  // row tid: exclusive prefix over the waves, and the row total
                    int64_t run = 0;
                    for (int w = 0; w < 16; ++w) {
                        const int64_t x = ws[tid][w];
                        ws[tid][w] = run;
                        run += x;
                    }
                    rowtot[tid] = run;
                }
                __syncthreads();
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int i = c0 + k * 1024 + tid;
                    if (i < J.m) J.chi[i] = carry + ws[k][wave] + v[k];
                    carry += rowtot[k];
                }
                __syncthreads();  // ws and rowtot are rewritten by the next chunk
            }
        }
        if (tid == 0) {
            if (J.status_out) *J.status_out = stv;
            *J.status = 0u;
        }
        __syncthreads();  // the status of the next image of this workgroup
    }
}

int launch_batch_merge(const void *table_dev, int colsum_grid, int scan_grid, hipStream_t stream) {
    hipLaunchKernelGGL(batch_colsum_kernel, dim3(colsum_grid), dim3(256), 0, stream, (const uint8_t *)table_dev);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(batch_scan_kernel, dim3(scan_grid), dim3(1024), 0, stream, (const uint8_t *)table_dev);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// ----------------------------------------------------------------------------
// Dual complex helpers: strided gather of a face of the box, signed sum of
// the faces' curves.

template <typename T>
__global__ void __launch_bounds__(256) gather_kernel(const T *__restrict__ src, int64_t base, int64_t s0, int64_t s1,
                                                     int64_t s2, int64_t n1, int64_t n2, int64_t total,
                                                     T *__restrict__ dst) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const int64_t i2 = i % n2, r = i / n2;
        const int64_t i1 = r % n1, i0 = r / n1;
        dst[i] = src[base + i0 * s0 + i1 * s1 + i2 * s2];
    }
}

int launch_gather(const void *src, int elem, int64_t base, int64_t s0, int64_t s1, int64_t s2, int64_t n0,
                  int64_t n1, int64_t n2, void *dst, hipStream_t stream) {
    const int64_t total = n0 * n1 * n2;
    if (total <= 0) return ECC_OK;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (elem == 1)
        hipLaunchKernelGGL(gather_kernel<uint8_t>, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint8_t *)src,
                           base, s0, s1, s2, n1, n2, total, (uint8_t *)dst);
    else
        hipLaunchKernelGGL(gather_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, stream,
                           (const uint16_t *)src, base, s0, s1, s2, n1, n2, total, (uint16_t *)dst);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

__global__ void __launch_bounds__(256) signed_sum_kernel(const int64_t *__restrict__ curves, int nf, uint64_t neg0,
                                                         uint64_t neg1, uint64_t skip0, uint64_t skip1, int sign,
                                                         int m, int64_t *__restrict__ out) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m) return;
    int64_t acc = 0;
    for (int f = 0; f < nf; ++f) {
        const uint64_t skip = f < 64 ? skip0 >> f : skip1 >> (f - 64);
        const uint64_t neg = f < 64 ? neg0 >> f : neg1 >> (f - 64);
        if (skip & 1) continue;
        const int64_t v = curves[(size_t)f * m + t];
        acc += (neg & 1) ? -v : v;
    }
    out[t] = sign < 0 ? -acc : acc;
}

int launch_signed_sum(const int64_t *curves, int nf, const uint64_t neg_mask[2], const uint64_t skip_mask[2],
                      int sign, int m, int64_t *out, hipStream_t stream) {
    if (nf > 128) {
        set_error("internal error: %d faces", nf);
        return ECC_E_ARG;
    }
    hipLaunchKernelGGL(signed_sum_kernel, dim3((m + 255) / 256), dim3(256), 0, stream, curves, nf, neg_mask[0],
                       neg_mask[1], skip_mask[0], skip_mask[1], sign, m, out);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// Faces of the box of at most two dimensions, largest-value convention, with
// their signs: all of them in one launch, into count rows that are merged with
// the volume's (each face had a gather, a kernel and two merge launches of its
// own before: 400 x 413 x 390 takes 115 us per dual curve, from
// 187; a 2000 x 3000 image 46, from 91).
// A face of na x nb voxels has the cells (interval or vertex) x (interval or
// vertex); position (i, j), 0 <= i <= na and 0 <= j <= nb, stands for vertex i
// by vertex j, and for interval i by vertex j where i < na, and so on; a
// cell's value is the largest of the voxels around it.  An axis that the face
// does not have (n = 0) has one vertex with one voxel.  Values >= m are
// skipped (the volume's own launch reports them as range errors).
// A wave's unit is 64 columns of up to kFaceRows consecutive rows of one face:
// it walks them four rows of loads at a time, the row before and the columns
// to the left already in its registers.  The loads' latency bounds it, so the
// units are short and spread over up to one workgroup per CU; a workgroup's
// waves count in one LDS histogram and write it out as a row, at m-1-v as the
// volume's kernel does (most bins are touched, so adding them to one vector by
// global atomics costs more than the rows).  The six 2-D faces of 400 x 413 x
// 390: 16 us with 8 rows a unit and 128 workgroups that write rows; 51 us with
// 32 rows, 35 workgroups and atomics, beside the volume.
constexpr int kFaceRows = 8;
struct FaceTable {
    BoxFace f[kFacesPerLaunch];
    int32_t first[kFacesPerLaunch + 1];  // units before face k
    int32_t strips[kFacesPerLaunch];     // 64-column strips of face k
    int32_t n;
};

template <typename T, int M>
__global__ void __launch_bounds__(1024) box_faces_kernel(const T *__restrict__ img, FaceTable t,
                                                         int32_t *__restrict__ out) {
    __shared__ __align__(16) int32_t hist[M];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < M; i += 1024) hist[i] = 0;
    __syncthreads();
    auto add = [&](bool ok, uint32_t v, int s) {
        if (ok && v < (uint32_t)M) atomicAdd(&hist[M - 1 - v], s);
    };
    int k = 0;
    for (int unit = (int)blockIdx.x * 16 + __builtin_amdgcn_readfirstlane(wave); unit < t.first[t.n];
         unit += (int)gridDim.x * 16) {
        while (k + 1 < t.n && t.first[k + 1] <= unit) ++k;
        const BoxFace F = t.f[k];
        const int u = unit - t.first[k];
        const int64_t r0 = (int64_t)(u / t.strips[k]) * kFaceRows;
        const int64_t r1 = r0 + kFaceRows < F.na + 1 ? r0 + kFaceRows : F.na + 1;
        const int64_t j = (int64_t)(u % t.strips[k]) * 64 + lane;
        const bool pos = j <= F.nb, mid = j < F.nb || F.nb == 0, edge = lane == 0 && j > 0;
        const int s = F.sign;
        // the value at (i, j), and at (i, j - 1); 0 where there is none
        auto load = [&](int64_t i, uint32_t &v, uint32_t &left) {
            const bool here = i >= 0 && (i < F.na || (F.na == 0 && i == 0));
            const T *p = img + F.base + i * F.sa + j * F.sb;
            v = here && mid ? p[0] : 0u;
            left = here && edge ? p[-F.sb] : 0u;
        };
        auto with_left = [&](uint32_t v, uint32_t left) {  // lane 0 keeps its own load
            return (uint32_t)__builtin_amdgcn_update_dpp((int)left, (int)v, 0x138, 0xF, 0xF, false);
        };
        uint32_t v01, v00;
        load(r0 - 1, v01, v00);
        v00 = with_left(v01, v00);
        for (int64_t i = r0; i < r1; i += 4) {
            uint32_t v[4], left[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) load(i + q < r1 ? i + q : -1, v[q], left[q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t v11 = v[q], v10 = with_left(v11, left[q]);
                const uint32_t a = max(v10, v11), b = max(v01, v11);
                const bool row = pos && i + q < r1, ia = row && i + q < F.na, ib = row && j < F.nb;
                add(row, max(max(a, b), v00), s);
                add(ia, a, -s);
                add(ib, b, -s);
                add(ia && ib, v11, s);
                v01 = v11;
                v00 = v10;
            }
        }
    }
    __syncthreads();
    int32_t *row = out + (size_t)blockIdx.x * M;
    for (int i = tid * 4; i < M; i += 4096) *(int4 *)&row[i] = *(const int4 *)&hist[i];
}

static int64_t face_units(const BoxFace &F) { return (F.nb / 64 + 1) * (F.na / kFaceRows + 1); }

// The faces of the launch that starts with face f0: as many as its table holds,
// with up to 2^30 units in all, so that a thread's next unit stays below 2^31
// (2^31 - 5 x 2 x 2 voxels take two launches), and up to 2^37 positions, so that
// a workgroup's int32 bins hold its share (a position changes a bin by at most
// 2).  One face alone is within both: one that is not is a face of a volume
// beyond the card's memory.
static int faces_of_launch(const BoxFace *faces, int nfaces, int f0, int64_t *units) {
    int n = 0;
    int64_t positions = 0;
    *units = 0;
    while (n < kFacesPerLaunch && f0 + n < nfaces) {
        const BoxFace &F = faces[f0 + n];
        const int64_t u = face_units(F), p = (F.na + 1) * (F.nb + 1);
        if (n > 0 && (*units + u > INT32_MAX / 2 || positions + p > (int64_t)1 << 37)) break;
        *units += u;
        positions += p;
        ++n;
    }
    return n;
}

int box_face_rows(const BoxFace *faces, int nfaces, int max_rows) {
    int rows = 0;
    for (int f0 = 0; f0 < nfaces;) {
        int64_t units = 0;
        f0 += faces_of_launch(faces, nfaces, f0, &units);
        const int64_t wgs = (units + 15) / 16;
        rows += (int)(wgs < max_rows ? wgs : max_rows);
    }
    return rows;
}

int launch_box_faces(const void *img, int elem, const BoxFace *faces, int nfaces, int max_rows, int32_t *rows,
                     hipStream_t stream) {
    for (int f0 = 0; f0 < nfaces;) {
        int64_t units = 0;
        FaceTable t{};
        t.n = faces_of_launch(faces, nfaces, f0, &units);
        if (units > INT32_MAX / 2) {
            set_error("ecc_compute_dual: face too large");
            return ECC_E_UNSUPPORTED;
        }
        for (int k = 0; k < t.n; ++k) {
            t.f[k] = faces[f0 + k];
            t.strips[k] = (int32_t)(t.f[k].nb / 64 + 1);
            t.first[k + 1] = t.first[k] + (int32_t)face_units(t.f[k]);
        }
        const int grid = box_face_rows(faces + f0, t.n, max_rows);
        if (elem == 1)
            hipLaunchKernelGGL((box_faces_kernel<uint8_t, 256>), dim3(grid), dim3(1024), 0, stream, (const uint8_t *)img, t,
                               rows);
        else
            hipLaunchKernelGGL((box_faces_kernel<uint16_t, 16384>), dim3(grid), dim3(1024), 0, stream,
                               (const uint16_t *)img, t, rows);
        ECC_HIP(hipGetLastError());
        rows += (size_t)grid * (elem == 1 ? 256 : 16384);
        f0 += t.n;
    }
    return ECC_OK;
}

__global__ void minmax_init_kernel(uint32_t *out) {
    out[0] = 0xFFFFFFFFu;
    out[1] = 0u;
}

__global__ void __launch_bounds__(256) minmax_u16_kernel(const uint16_t *__restrict__ img, int64_t n, int vec,
                                                         uint32_t *out) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t n8 = vec ? n / 8 : 0;  // 16-byte groups when the image is 16-byte aligned
    const uint4 *v8 = reinterpret_cast<const uint4 *>(img);
    auto fold = [&](const uint4 q) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t a = w[j] & 0xFFFFu, b = w[j] >> 16;
            lo = min(lo, min(a, b));
            hi = max(hi, max(a, b));
        }
    };
    // each workgroup streams one contiguous chunk, four independent 16-byte
    // loads in flight per thread
    const int64_t chunk = (n8 + gridDim.x - 1) / gridDim.x;
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = beg + chunk < n8 ? beg + chunk : n8;
    const int64_t bd = blockDim.x;
    int64_t i = beg + threadIdx.x;
    for (; i + 3 * bd < end; i += 4 * bd) {
        uint4 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = v8[i + u * bd];
#pragma unroll
        for (int u = 0; u < 4; ++u) fold(q[u]);
    }
    for (; i < end; i += bd) fold(v8[i]);
    for (int64_t i = n8 * 8 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        lo = min(lo, (uint32_t)img[i]);
        hi = max(hi, (uint32_t)img[i]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMin(&out[0], lo);
        atomicMax(&out[1], hi);
    }
}

int launch_minmax_u16(const uint16_t *img, int64_t n, uint32_t *out, hipStream_t stream) {
    hipLaunchKernelGGL(minmax_init_kernel, dim3(1), dim3(1), 0, stream, out);
    ECC_HIP(hipGetLastError());
    int64_t blocks = (n / 8 + 255) / 256;
    const int64_t cap = 8 * (int64_t)device_cu_count();  // eight workgroups of 4 waves per CU
    if (blocks < 1) blocks = 1;
    if (blocks > cap) blocks = cap;
    const int vec = ((uintptr_t)img % 16) == 0;
    hipLaunchKernelGGL(minmax_u16_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, img, n, vec, out);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

// Curves of at most 1024 thresholds from at most kSmallMergeRows rows: both
// steps in one workgroup, for the latency of small images (m / 4 threads per
// row, 4096 / m rows at a time).  The column sums are placed through LDS (with
// `reverse`, column c lands at m-1-c); then vcec, the scan into chi (only
// with a clear status word), and the status copy and clear.  One workgroup
// reads few bytes per second: 5.6 us for 256 rows of 256 columns, 12.4 us for
// 1024, where the two launches take 8.5 us and the wait between them.
constexpr int kSmallMergeRows = 256;
__global__ void __launch_bounds__(1024) merge_scan_small_kernel(const int32_t *__restrict__ partial, int rows, int m,
                                                                int64_t *__restrict__ vcec, int accumulate, int reverse,
                                                                int negate, int64_t *__restrict__ chi, uint32_t *status,
                                                                uint32_t *status_out) {
    __shared__ unsigned long long col[1024];
    __shared__ int64_t sh[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t stv = *(volatile uint32_t *)status;  // cleared below, after a barrier
    col[tid] = 0;
    __syncthreads();
    if (rows > 0) {
        const int per = m / 4, step = 1024 / per;
        const int c0 = (tid % per) * 4;
        int r = tid / per;
        if (r < step) {
            int64_t v[4] = {0, 0, 0, 0};
            const int4 *p = reinterpret_cast<const int4 *>(partial) + c0 / 4;
            const size_t stride4 = (size_t)per;
            for (; r + 7 * step < rows; r += 8 * step) {
                int4 a[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) a[u] = p[(size_t)(r + u * step) * stride4];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    v[0] += a[u].x;
                    v[1] += a[u].y;
                    v[2] += a[u].z;
                    v[3] += a[u].w;
                }
            }
            for (; r < rows; r += step) {
                const int4 a = p[(size_t)r * stride4];
                v[0] += a.x;
                v[1] += a.y;
                v[2] += a.z;
                v[3] += a.w;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) atomicAdd(&col[reverse ? m - 1 - (c0 + j) : c0 + j], (unsigned long long)v[j]);
        }
        __syncthreads();
    }
    const bool own = tid < m;
    int64_t v = 0;
    if (own) {
        if (rows == 0 || accumulate) v = vcec[tid];
        v += negate ? -(int64_t)col[tid] : (int64_t)col[tid];
        if (rows > 0) vcec[tid] = v;
    }
    int64_t x = v;
    x = wave_prefix(x);
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    for (int w = 0; w < wave; ++w) x += sh[w];
    if (own && stv == 0) chi[tid] = x;
    if (tid == 0) {
        status[1] = stv;
        if (status_out) *status_out = stv;
        status[0] = 0u;
    }
}

static int64_t *merge_totals(uint32_t *status) { return reinterpret_cast<int64_t *>(status) + kStatusTotalsOffset / 8; }

static int launch_colsum(const int32_t *partial, int rows, int m, int64_t *vcec, bool accumulate, int64_t *totals,
                         int64_t *clear, bool hand, uint32_t *status, hipStream_t stream, bool reverse, bool negate) {
    if (rows <= 64)
        hipLaunchKernelGGL(colsum_kernel<16>, dim3(m / kColBlock), dim3(256), 0, stream, partial, rows, m, vcec,
                           accumulate ? 1 : 0, reverse ? 1 : 0, negate ? 1 : 0, totals, clear, hand ? 1 : 0, status);
    else
        hipLaunchKernelGGL(colsum_kernel<64>, dim3(m / kColBlock), dim3(1024), 0, stream, partial, rows, m, vcec,
                           accumulate ? 1 : 0, reverse ? 1 : 0, negate ? 1 : 0, totals, clear, hand ? 1 : 0, status);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

int launch_merge(const int32_t *partial, int rows, int m, int64_t *vcec, bool accumulate, bool do_scan, int64_t *chi,
                 uint32_t *status, uint32_t *status_out, hipStream_t stream, bool reverse, bool negate) {
    if (m % 256 != 0 || m > 65536 || (m < 1024 && 1024 % m != 0)) {
        set_error("launch_merge: m = %d not supported", m);
        return ECC_E_ARG;
    }
    if (do_scan && m <= 1024 && rows <= kSmallMergeRows) {
        hipLaunchKernelGGL(merge_scan_small_kernel, dim3(1), dim3(1024), 0, stream, partial, rows, m, vcec,
                           accumulate ? 1 : 0, reverse ? 1 : 0, negate ? 1 : 0, chi, status, status_out);
        ECC_HIP(hipGetLastError());
        return ECC_OK;
    }
    int64_t *totals = merge_totals(status);
    if (rows > 0) {
        int rc = launch_colsum(partial, rows, m, vcec, accumulate, do_scan ? totals : nullptr, nullptr, do_scan, status,
                               stream, reverse, negate);
        if (rc) return rc;
    }
    if (do_scan) {
        hipLaunchKernelGGL(scan_kernel, dim3((m + 1023) / 1024), dim3(1024), 0, stream, (const int64_t *)vcec, m,
                           rows > 0 ? (const int64_t *)totals : (const int64_t *)nullptr, rows > 0 ? 1 : 0, chi, status,
                           status_out);
        ECC_HIP(hipGetLastError());
    }
    return ECC_OK;
}

// A 16-bit image's pass over one half of 0..65535: its column sums and totals
// into that half; clear: the other half (the upper) is set to zero.
int launch_merge_half(const int32_t *partial, int rows, int64_t *vcec16, int half, bool clear, uint32_t *status,
                      hipStream_t stream) {
    constexpr int m = 32768;
    return launch_colsum(partial, rows, m, vcec16 + half * m, false, merge_totals(status) + half * (m / kColBlock),
                         clear ? vcec16 + m : nullptr, false, status, stream, false, false);
}

int launch_scan_halves(const int64_t *vcec16, int64_t *chi, uint32_t *status, uint32_t *status_out, hipStream_t stream) {
    hipLaunchKernelGGL(scan_kernel, dim3(64), dim3(1024), 0, stream, vcec16, 65536,
                       (const int64_t *)merge_totals(status), 0, chi, status, status_out);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

}  // namespace ecc
