// The distinct values of a float image and the curve at them (Sec. 3, "Other
// Ranges of Gray Values"), without sorting the keys: the keys (f32_key) that
// can occur are few enough for one bit each.  An image whose keys hold P
// different top bytes (sign and high exponent bits; at most 32) has its keys
// among P * 2^24 values: the byte's rank among those present and the low 24
// bits, in the keys' own order, give a key's position p.
//
// A bit per position in memory, set by every voxel, would be bound by atomics
// (27 G/s at random places on MI355X: 10 ms for 2^28 voxels).  So the keys
// are first put in order of their lowest 9 bits, which are spread evenly in
// any image of many values, within tiles of 16384; the keys of one of the 512
// buckets are then a run in each tile, and a bucket's bits, one per remaining
// value (P * 2^15), are set in LDS:
//  1. split_kernel: the tiles' keys by bucket, the buckets' first slots in
//     each tile and their totals; also which top bytes occur;
//  2. bucket_bits_kernel: a workgroup per bucket (large ones are shared) sets
//     the bits of its runs in LDS, P * 4 KiB, and adds them to
//     bits[bucket][p >> 9];
//  3. order_bits_kernel: bits[bucket][idx] to the order of p (idx first, then
//     the bucket), with the count of set bits before each block of 256;
//  4. expand_kernel: the k-th set bit is the k-th distinct value; its chi is
//     cleared;
//  5. add_records_kernel: each record's change is added to chi at its key's
//     rank (the set bits before it);
//  6. chi_sums_kernel, chi_scan_kernel, chi_prefix_kernel: the running sum.
#include <algorithm>

#include "ecc_internal.h"

namespace ecc {

namespace {

constexpr int kBucketBits = 9;
constexpr int kBuckets = 1 << kBucketBits;
constexpr int kIdxPerByte = 1 << (24 - kBucketBits);  // idx values per top byte
constexpr int kWordsPerByte = kIdxPerByte / 32;       // words of a bucket's bits per top byte

// rank[t]: present top bytes below t; called by every thread of a workgroup
// of at least 256, ends with a barrier
__device__ __forceinline__ void rank_table(const uint32_t *__restrict__ mask, uint8_t *rank) {
    const int t = threadIdx.x;
    if (t < 256) {
        uint32_t c = 0;
        for (int w = 0; w < (t >> 5); ++w) c += (uint32_t)__builtin_popcount(mask[w]);
        c += (uint32_t)__builtin_popcount(mask[t >> 5] & ((1u << (t & 31)) - 1u));
        rank[t] = (uint8_t)c;
    }
    __syncthreads();
}

// ---- 1. Bound by memory (a read and a write of every key, both in whole
// lines): 2^28 keys take 440 us.  (Scattering the keys to the buckets instead
// took 530 us, and counting them per tile and digit before it 320.)  The next
// tile is not loaded ahead: two workgroups per CU overlap.
constexpr int kThreads = 1024;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;
static_assert(kTile == kSplitTile && kBuckets == kSplitBuckets, "the tiles that the caller makes room for");

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8)))
split_kernel(const float *__restrict__ img, int64_t n, int64_t tiles, uint32_t *__restrict__ out,
             uint16_t *__restrict__ starts, uint32_t *__restrict__ rows, uint32_t *__restrict__ mask,
             uint32_t *status) {
    __shared__ __align__(16) uint32_t buf[kTile];  // the tile's keys by bucket
    __shared__ uint32_t cnt[kBuckets];             // keys per bucket, then the bucket's first slot
    __shared__ uint32_t ws[kBuckets / 64];
    __shared__ uint8_t present[256];  // top bytes seen
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < kBuckets) cnt[tid] = 0;
    if (tid < 256) present[tid] = 0;
    __syncthreads();
    uint32_t mine = 0;     // this thread's bucket's keys
    uint32_t last = 256u;  // the top byte this thread noted last (neighbouring voxels share theirs)
    bool nan = false;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t t0 = tile * kTile;
        const int valid = (int)std::min<int64_t>(kTile, n - t0);
        uint32_t key[kItems], at[kItems / 2];  // at: places in the buckets, two per word
        const uint32_t *src = reinterpret_cast<const uint32_t *>(img) + t0;
        const bool vec = valid == kTile && (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
        if (vec) {
#pragma unroll
            for (int q = 0; q < kItems / 4; ++q) {
                const uint4 w = reinterpret_cast<const uint4 *>(src)[q * kThreads + tid];
                key[4 * q] = w.x;
                key[4 * q + 1] = w.y;
                key[4 * q + 2] = w.z;
                key[4 * q + 3] = w.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < kItems; ++j) key[j] = j * kThreads + tid < valid ? src[j * kThreads + tid] : 0u;
        }
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            nan |= (key[j] & 0x7FFFFFFFu) > 0x7F800000u;
            key[j] = f32_key(key[j]);
            uint32_t a = 0;
            if (vec || j * kThreads + tid < valid) {
                const uint32_t top = key[j] >> 24;
                if (top != last) {
                    present[top] = 1;
                    last = top;
                }
                a = atomicAdd(&cnt[key[j] & (kBuckets - 1)], 1u);
            }
            if (j & 1) at[j / 2] |= a << 16;
            else at[j / 2] = a;
        }
        __syncthreads();
        // first slot of each bucket
        uint32_t c = 0, x = 0;
        if (tid < kBuckets) {
            c = x = cnt[tid];
            x = wave_prefix(x);
            if (lane == 63) ws[tid >> 6] = x;
        }
        __syncthreads();
        if (tid < kBuckets) {
            uint32_t s = x - c;
            for (int w = 0; w < (tid >> 6); ++w) s += ws[w];
            cnt[tid] = s;
            starts[tile * kBuckets + tid] = (uint16_t)s;
            mine += c;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kItems; ++j)
            if (vec || j * kThreads + tid < valid) buf[cnt[key[j] & (kBuckets - 1)] + (j & 1 ? at[j / 2] >> 16 : at[j / 2] & 0xFFFFu)] = key[j];
        __syncthreads();
        if (tid < kBuckets) cnt[tid] = 0;
        if (valid == kTile) {
#pragma unroll
            for (int q = 0; q < kItems / 4; ++q) {
                const int i = q * kThreads + tid;
                reinterpret_cast<uint4 *>(out + t0)[i] = reinterpret_cast<const uint4 *>(buf)[i];
            }
        } else {
            for (int i = tid; i < valid; i += kThreads) out[t0 + i] = buf[i];
        }
        __syncthreads();  // cnt is zero, buf is read
    }
    // (a row per workgroup: added to one by atomics, all on 512 words, they
    // made the launch 5 us longer)
    if (tid < kBuckets) rows[(size_t)blockIdx.x * kBuckets + tid] = mine;
    if (__builtin_amdgcn_ballot_w64(nan) != 0 && lane == 0) atomicOr(status, kStatusNaN);
    if (tid < 256) {  // wave w: bytes 64 w .. 64 w + 63, mask words 2 w and 2 w + 1
        const uint64_t b = __builtin_amdgcn_ballot_w64(present[tid] != 0);
        if (lane == 0 && (uint32_t)b != 0u) atomicOr(&mask[2 * (tid >> 6)], (uint32_t)b);
        if (lane == 0 && (uint32_t)(b >> 32) != 0u) atomicOr(&mask[2 * (tid >> 6) + 1], (uint32_t)(b >> 32));
    }
}

// The buckets' totals, 64 per workgroup; the first also copies the presence
// mask to host-mapped memory (read by the host after an event, to choose
// between the bits of the values and the sort).
__global__ void __launch_bounds__(1024) bucket_totals_kernel(const uint32_t *__restrict__ rows, int nrows,
                                                             uint32_t *__restrict__ totals,
                                                             const uint32_t *__restrict__ mask, uint32_t *host) {
    __shared__ uint32_t part[16][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x == 0 && tid < 8) host[tid] = mask[tid];
    const int c = blockIdx.x * 64 + lane;
    uint32_t s = 0;
#pragma unroll 8
    for (int r = wave; r < nrows; r += 16) s += rows[(size_t)r * kBuckets + c];
    part[wave][lane] = s;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < 16; ++w) s += part[w][lane];
    totals[c] = s;
}

// ---- 2. A bucket of more than `share` keys is cut into shares of at most
// that many on average, each taking every ns-th tile; a workgroup takes one
// share (at most kBuckets + n / share of them).  A bucket of one share is
// stored, the others are OR-ed (bits is zero before the launch).
// A wave takes the runs of up to 46 tiles as one sequence of keys, 64 per load
// and 12 loads in flight (a run is 32 keys on average): which run a lane's key
// is in is the count of run ends before it.  Neighbouring buckets run on one XCD at the same pace, so the
// lines that hold the ends of their runs and their first slots are fetched
// once.  2^28 keys take 371 us (430 with a half-wave per run, whose lanes
// past the run idle).
__global__ void __launch_bounds__(kThreads) bucket_bits_kernel(const uint32_t *__restrict__ keys, int64_t n, int tiles,
                                                               const uint16_t *__restrict__ starts,
                                                               const uint32_t *__restrict__ totals,
                                                               const uint32_t *__restrict__ mask, uint32_t share,
                                                               int words, uint32_t *__restrict__ bits) {
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t ws[kBuckets / 64];
    __shared__ uint32_t my[3];  // bucket, share, shares of the bucket
    constexpr int kWaves = kThreads / 64;
    constexpr uint32_t kMaxKeys = 2304;  // of a group: three rounds of loads, 1.56 the mean
    __shared__ uint32_t marks[kWaves][kMaxKeys / 32];
    __shared__ uint8_t rank[256];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (of evenly filled buckets the first kBuckets workgroups have work)
    const uint32_t block = blockIdx.x < kBuckets ? xcd_block(blockIdx.x, kBuckets) : blockIdx.x;
    if (tid == 0) my[2] = 0;
    uint32_t ns = 0, x = 0;
    if (tid < kBuckets) {
        ns = x = (totals[tid] + share - 1) / share;
        x = wave_prefix(x);
        if (lane == 63) ws[tid >> 6] = x;
    }
    rank_table(mask, rank);
    if (tid < kBuckets) {
        uint32_t s = x - ns;  // this bucket's first workgroup
        for (int w = 0; w < (tid >> 6); ++w) s += ws[w];
        if (block >= s && block < s + ns) {
            my[0] = (uint32_t)tid;
            my[1] = block - s;
            my[2] = ns;
        }
    }
    __syncthreads();
    const int b = __builtin_amdgcn_readfirstlane((int)my[0]), first = __builtin_amdgcn_readfirstlane((int)my[1]);
    const int step = __builtin_amdgcn_readfirstlane((int)my[2]);
    if (step == 0) return;  // (uniform) past the last share
    for (int i = tid; i < words; i += kThreads) lds[i] = 0;
    __syncthreads();
    auto set = [&](uint32_t k) {
        atomicOr(&lds[((uint32_t)rank[k >> 24] << 10) | ((k >> 14) & 0x3FFu)], 1u << ((k >> 9) & 31u));
    };
    // this share's tiles: first + step * i, i < count
    const int count = first < tiles ? (tiles - first + step - 1) / step : 0;
    constexpr int kGroup = 46, kSteps = 12;
    const int group = std::min(kGroup, (count + kWaves - 1) / kWaves);
    // lane: the run of tile i0 + lane (loaded a group ahead)
    auto fetch = [&](int i0, uint32_t &beg, uint32_t &end) {
        beg = end = 0;
        if (lane < group && i0 + lane < count) {
            const int64_t t = first + (int64_t)step * (i0 + lane);
            const uint16_t *s = starts + t * kBuckets + b;
            beg = s[0];
            end = b + 1 < kBuckets ? (uint32_t)s[1] : (uint32_t)std::min<int64_t>(kTile, n - t * kTile);
        }
    };
    uint32_t beg1, end1;
    fetch(wave * group, beg1, end1);
    for (int i0 = wave * group; i0 < count; i0 += kWaves * group) {
        const uint32_t pos = ((uint32_t)first + (uint32_t)step * (uint32_t)(i0 + lane)) * kTile + beg1, len = end1 - beg1;
        fetch(i0 + kWaves * group, beg1, end1);
        uint32_t x = len;
        x = wave_prefix(x);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)x, 63), before = x - len;
        if (total > kMaxKeys) {  // (uniform) a crowded bucket: long runs
            for (int r = 0; r < group; ++r) {
                const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)pos, r);
                const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)len, r);
                uint32_t j = lane;
                for (; j + 192u < l; j += 256u) {
                    uint32_t k[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) k[q] = keys[p + j + 64u * (uint32_t)q];
#pragma unroll
                    for (int q = 0; q < 4; ++q) set(k[q]);
                }
                for (; j < l; j += 64u) set(keys[p + j]);
            }
            continue;
        }
        // the runs that are not empty to the first lanes: where key g of the
        // group lies, less g
        const uint64_t some = __builtin_amdgcn_ballot_w64(len != 0);
        const uint32_t slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
        const uint32_t dst = len != 0 ? slot : (uint32_t)__builtin_popcountll(some) + (uint32_t)lane - slot;
        const uint32_t base = (uint32_t)__builtin_amdgcn_ds_permute((int)(dst * 4u), (int)(pos - before));
        // a bit per key: the last key of a run with another behind it
        marks[wave][lane] = 0;
        if (lane < (int)kMaxKeys / 32 - 64) marks[wave][64 + lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (len != 0 && before != 0) atomicOr(&marks[wave][(before - 1) >> 5], 1u << ((before - 1) & 31u));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        uint32_t ended = 0;  // runs that end before the step
        for (uint32_t g0 = 0; g0 < total; g0 += 64u * kSteps) {
            uint32_t k[kSteps];
#pragma unroll
            for (uint32_t q = 0; q < kSteps; ++q) {
                const uint32_t lo = marks[wave][(g0 >> 5) + 2 * q], hi = marks[wave][(g0 >> 5) + 2 * q + 1];
                const uint32_t r = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, ended));
                ended += (uint32_t)__builtin_popcount(lo) + (uint32_t)__builtin_popcount(hi);
                const uint32_t at = (uint32_t)__shfl((int)base, (int)r, 64) + g0 + 64u * q + (uint32_t)lane;
                // (a lane past the last key reads a word in range, unused)
                k[q] = *(const uint32_t *)((const char *)keys + std::min(at, (uint32_t)n - 1u) * 4u);
            }
            if (g0 + 64u * kSteps <= total) {
#pragma unroll
                for (uint32_t q = 0; q < kSteps; ++q) set(k[q]);
            } else {
#pragma unroll
                for (uint32_t q = 0; q < kSteps; ++q)
                    if (g0 + 64u * q + (uint32_t)lane < total) set(k[q]);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    uint32_t *dst = bits + (size_t)b * words;
    const bool whole = step == 1;
    for (int w = tid; w < words; w += kThreads) {
        const uint32_t v = lds[w];
        if (v == 0) continue;
        if (whole) dst[w] = v;
        else atomicOr(&dst[w], v);
    }
}

// ---- 3. A tile: 16 words of every bucket, i.e. 512 idx by 512 buckets, 2^18
// positions.  A thread transposes 32 x 32 bits in registers: the words w of
// the buckets 32 g .. 32 g + 31 become, for the 32 idx of word w, word g of
// the idx's row of 16.
constexpr int kTileWords = 16;
constexpr int kOrdWords = kTileWords * kBuckets;  // 8192 words in p order
constexpr int kBlockWords = 8;                    // words per counted block
constexpr int kTileBlocks = kOrdWords / kBlockWords;

template <int S, uint32_t LOW>
__device__ __forceinline__ void transpose_step(uint32_t (&a)[32]) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        if (i & S) continue;
        const uint32_t t = ((a[i] >> S) ^ a[i + S]) & LOW;
        a[i] ^= t << S;
        a[i + S] ^= t;
    }
}
// afterwards bit i of a[j] is the former bit j of a[i]
__device__ __forceinline__ void transpose32(uint32_t (&a)[32]) {
    transpose_step<16, 0x0000FFFFu>(a);
    transpose_step<8, 0x00FF00FFu>(a);
    transpose_step<4, 0x0F0F0F0Fu>(a);
    transpose_step<2, 0x33333333u>(a);
    transpose_step<1, 0x55555555u>(a);
}

__global__ void __launch_bounds__(256) order_bits_kernel(const uint32_t *__restrict__ bits, int words,
                                                         uint32_t *__restrict__ ord, uint32_t *__restrict__ blk,
                                                         uint32_t *__restrict__ total) {
    __shared__ __attribute__((aligned(16))) uint32_t t[kOrdWords + kOrdWords / 8];
    __shared__ uint32_t ws[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w0 = blockIdx.x * kTileWords;
    uint32_t any = 0;
    // 4 threads load a bucket's 16 words; word w of bucket d is kept at
    // d * 16 + (w + d / 32) % 16 (the threads of one w and 16 g then read
    // 16 banks)
    for (int i = tid; i < kBuckets * 4; i += 256) {
        const int d = i >> 2, q = i & 3;
        const uint4 v = *reinterpret_cast<const uint4 *>(bits + (size_t)d * words + w0 + 4 * q);
        const int r = d >> 5;
        t[d * 16 + ((4 * q + 0 + r) & 15)] = v.x;
        t[d * 16 + ((4 * q + 1 + r) & 15)] = v.y;
        t[d * 16 + ((4 * q + 2 + r) & 15)] = v.z;
        t[d * 16 + ((4 * q + 3 + r) & 15)] = v.w;
        any |= v.x | v.y | v.z | v.w;
    }
    const bool empty = __syncthreads_or((int)(any != 0)) == 0;
    uint32_t *dst = ord + (size_t)blockIdx.x * kOrdWords;
    uint32_t *db = blk + (size_t)blockIdx.x * kTileBlocks;
    if (empty) {  // (uniform) nothing reads the words or the blocks of an empty tile
        if (tid == 0) total[blockIdx.x] = 0;
        return;
    }
    const int g = tid & 15, w = tid >> 4;
    uint32_t a[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) a[i] = t[(32 * g + i) * 16 + ((w + g) & 15)];
    transpose32(a);
    __syncthreads();
    // in p order, with 4 words of padding per 32: idx w * 32 + j, word g
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const int o = (w * 32 + j) * 16 + g;
        t[o + (o >> 5) * 4] = a[j];
    }
    __syncthreads();
    // a thread counts 32 consecutive words: four blocks
    uint32_t c[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        c[b] = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint4 v = *reinterpret_cast<const uint4 *>(&t[tid * 36 + b * 8 + q * 4]);
            c[b] += __builtin_popcount(v.x) + __builtin_popcount(v.y) + __builtin_popcount(v.z) + __builtin_popcount(v.w);
        }
    }
    const uint32_t s = c[0] + c[1] + c[2] + c[3];
    uint32_t x = s;
    x = wave_prefix(x);
    if (lane == 63) ws[wave] = x;
    __syncthreads();
    uint32_t p = x - s;
    for (int v = 0; v < wave; ++v) p += ws[v];
    *reinterpret_cast<uint4 *>(db + tid * 4) = make_uint4(p, p + c[0], p + c[0] + c[1], p + c[0] + c[1] + c[2]);
    if (tid == 255) total[blockIdx.x] = p + s;
    for (int i = tid; i < kOrdWords / 4; i += 256) {
        const int o = 4 * i;
        *reinterpret_cast<uint4 *>(dst + o) = *reinterpret_cast<const uint4 *>(&t[o + (o >> 5) * 4]);
    }
}

// The exclusive scan of the tiles' totals (base[tiles] = their sum, also to
// *count; base[tiles + 1]: whether a bucket has `crowded` keys or more) and the
// list of the tiles that are not empty (list[0]: how many): one workgroup.  The count and the status word also go to host-mapped memory,
// where the host finds them after its wait for the curve.
__global__ void __launch_bounds__(1024) tile_base_kernel(const uint32_t *__restrict__ total, int tiles,
                                                         const uint32_t *__restrict__ buckets, uint32_t crowded,
                                                         uint32_t *__restrict__ base, uint32_t *__restrict__ list,
                                                         int64_t *count, int64_t *count_host, const uint32_t *status,
                                                         uint32_t *status_host) {
    __shared__ uint32_t ws[16], wf[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int crowd = __syncthreads_or((int)(tid < kBuckets && buckets[tid] >= crowded));
    uint32_t carry = 0, full = 0;
    for (int c0 = 0; c0 < tiles; c0 += 1024) {
        const int i = c0 + tid;
        const uint32_t v = i < tiles ? total[i] : 0u;
        uint32_t x = v;
        x = wave_prefix(x);
        if (lane == 63) ws[wave] = x;
        const uint64_t some = __builtin_amdgcn_ballot_w64(v != 0);
        if (lane == 0) wf[wave] = (uint32_t)__builtin_popcountll(some);
        __syncthreads();
        uint32_t p = carry, f = full;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) p += ws[w], f += wf[w];
            carry += ws[w];
            full += wf[w];
        }
        if (i < tiles) base[i] = p + x - v;
        if (v != 0)
            list[1 + f + __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u))] = (uint32_t)i;
        __syncthreads();
    }
    if (tid == 0) {
        base[tiles] = carry;
        base[tiles + 1] = crowd != 0;
        list[0] = full;
        *count = (int64_t)carry;
        *count_host = (int64_t)carry;
        *status_host = *status;
    }
}

// ---- 4. A wave takes 64 words (eight blocks) at a time: each lane's set
// bits are put, in order, into LDS, and leave as one run.  The workgroups
// share the parts of the tiles that are not empty (a workgroup per part of
// every tile: 27 us for 190 x 211 x 170 noise, much of it the launch of
// workgroups without work; now 21).
constexpr int kExpandWaves = 4;
constexpr int kExpandParts = 32;  // of a tile: a chunk per wave
constexpr int kExpandWords = 64;

__global__ void __launch_bounds__(64 * kExpandWaves) expand_kernel(const uint32_t *__restrict__ ord,
                                                                   const uint32_t *__restrict__ blk,
                                                                   const uint32_t *__restrict__ base,
                                                                   const uint32_t *__restrict__ list,
                                                                   const uint32_t *__restrict__ mask,
                                                                   float *__restrict__ out_keys,
                                                                   int64_t *__restrict__ out_chi) {
    __shared__ uint32_t st[kExpandWaves][kExpandWords * 33];
    __shared__ uint8_t byte_of[256];  // top byte of a rank
    static_assert(kOrdWords == kExpandWords * kExpandWaves * kExpandParts, "a chunk per wave and part");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    {
        uint32_t c = 0;
        for (int w = 0; w < (tid >> 5); ++w) c += (uint32_t)__builtin_popcount(mask[w]);
        const uint32_t m = mask[tid >> 5];
        c += (uint32_t)__builtin_popcount(m & ((1u << (tid & 31)) - 1u));
        if ((m >> (tid & 31)) & 1u) byte_of[c] = (uint8_t)tid;
    }
    __syncthreads();
    const uint32_t items = list[0] * kExpandParts;
    for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
        const uint32_t tile = list[1 + item / kExpandParts], part = item % kExpandParts;
        const uint32_t w0 = tile * kOrdWords + (part * kExpandWaves + (uint32_t)wave) * kExpandWords;
        uint32_t v = ord[w0 + lane];
        const uint32_t first = base[tile] + blk[w0 / kBlockWords];
        const uint32_t c = (uint32_t)__builtin_popcount(v);
        uint32_t x = c;
        x = wave_prefix(x);
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        if (cnt == 0) continue;
        const uint32_t p0 = (w0 + lane) * 32u;
        const uint32_t top = (uint32_t)byte_of[p0 >> 24] << 24;
        uint32_t q = x - c;
        while (v != 0) {
            const uint32_t bit = (uint32_t)__builtin_ctz(v);
            v &= v - 1;
            st[wave][q + (q >> 5)] = top | ((p0 + bit) & 0xFFFFFFu);
            ++q;
        }
        // (one wave's own LDS operations take effect in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t i = lane; i < cnt; i += 64) {
            const uint32_t k = st[wave][i + (i >> 5)];
            out_keys[first + i] = __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
            out_chi[first + i] = 0;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// ---- 5. A wave per region of records.  Up to kFewValues values (images of
// whole numbers, say) are added in LDS first: a workgroup's int32 sums (at
// most 2^26: a record's change is at most 16), then one global add per value
// and workgroup.  (All of a card's adds on 4096 values, without LDS: 2.5 ms
// for 2^26 voxels, 0.47 with it.)  More values take a global add per record, and
// the adds, which all go to memory, bound it: 7.3 million of 2^28 voxels of smooth
// noise take 0.37 ms (20 G/s; the gathers before them and the records move 0.11
// GB), those of 2^26 of white noise 2.2 ms (27 G/s).  Adds to one value wait
// for each other (0.2 G/s), and images that are clipped, or mostly zero, have
// most of their records at one or two values.  Such a value shows in its bucket's
// total: where one is an eighth above the mean, the first values that a workgroup
// meets are summed in LDS, in kHot slots found by a hash of the rank, two tries;
// a value that occurs often is among them before they are full.  (2^24 voxels of noise clipped at
// both ends: 43 ms without, 0.62 with them; where no bucket stands out the slots
// would make 6.8 million voxels of smooth noise 3 % slower.)
constexpr int kFewValues = 16384;
constexpr uint32_t kFewGroups = 512;
constexpr uint32_t kHotBits = 11, kHot = 1u << kHotBits;

__global__ void __launch_bounds__(1024) add_records_kernel(const uint64_t *__restrict__ nz,
                                                           const uint32_t *__restrict__ nz_cnt, int64_t regions,
                                                           int64_t region_slots, const uint32_t *__restrict__ ord,
                                                           const uint32_t *__restrict__ blk,
                                                           const uint32_t *__restrict__ base, int tiles,
                                                           const uint32_t *__restrict__ mask,
                                                           int64_t *__restrict__ chi) {
    __shared__ int32_t acc[kFewValues];
    __shared__ uint8_t rank[256];
    const uint32_t K = base[tiles];
    const bool few = K <= (uint32_t)kFewValues;
    const uint32_t groups = few ? std::min(gridDim.x, kFewGroups) : gridDim.x;
    if (blockIdx.x >= groups) return;
    uint32_t *hot = reinterpret_cast<uint32_t *>(acc);  // many values: the slots' ranks, then their sums
    int32_t *hot_sum = acc + kHot;
    const bool slots = !few && base[tiles + 1] != 0;
    for (uint32_t i = threadIdx.x; i < (few ? K : slots ? 2 * kHot : 0u); i += 1024) acc[i] = few || i >= kHot ? 0 : -1;
    rank_table(mask, rank);
    const int lane = threadIdx.x & 63;
    for (int64_t reg = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 6); reg < regions; reg += (int64_t)groups * 16) {
        const uint32_t c = nz_cnt[reg];
        const uint64_t *src = nz + reg * region_slots;
        auto add = [&](uint64_t r) {
            const uint32_t k = (uint32_t)(r >> 32);
            const uint32_t p = ((uint32_t)rank[k >> 24] << 24) | (k & 0xFFFFFFu);
            const uint32_t b = p >> 8;
            uint32_t at = base[p >> 18] + blk[b];
            const uint4 *w4 = reinterpret_cast<const uint4 *>(ord + (size_t)b * kBlockWords);
            const uint4 a0 = w4[0], a1 = w4[1];
            const uint32_t w[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const uint32_t wi = (p >> 5) & 7u, below = (1u << (p & 31u)) - 1u;
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j)
                at += (uint32_t)__builtin_popcount(w[j] & (j < wi ? 0xFFFFFFFFu : j == wi ? below : 0u));
            const int32_t chg = (int32_t)(uint32_t)r;
            if (few) {
                atomicAdd(&acc[at], chg);
                return;
            }
            const uint32_t h = (at * 0x9E3779B1u) >> (32 - kHotBits);
#pragma unroll
            for (uint32_t q = 0; slots && q < 2; ++q) {
                uint32_t *slot = &hot[h ^ q];
                uint32_t owner = *(volatile uint32_t *)slot;
                if (owner == ~0u) {
                    owner = atomicCAS(slot, ~0u, at);
                    if (owner == ~0u) owner = at;
                }
                if (owner == at) {
                    atomicAdd(&hot_sum[h ^ q], chg);
                    return;
                }
            }
            atomicAdd((unsigned long long *)&chi[at], (unsigned long long)(int64_t)chg);
        };
        uint32_t i = lane;
        for (; i + 192 < c; i += 256) {  // four records of loads in flight
            uint64_t r[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = src[i + 64 * q];
#pragma unroll
            for (int q = 0; q < 4; ++q) add(r[q]);
        }
        for (; i < c; i += 64) add(src[i]);
    }
    if (!few && !slots) return;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < (few ? K : kHot); i += 1024) {
        const int32_t v = few ? acc[i] : hot_sum[i];
        if (v != 0) atomicAdd((unsigned long long *)&chi[few ? i : hot[i]], (unsigned long long)(int64_t)v);
    }
}

// ---- 6. Tiles of kChiTile entries, K of them known on the device only.
constexpr int kChiThreads = 256;
constexpr int kChiItems = 16;
constexpr int kChiTile = kChiThreads * kChiItems;

__global__ void __launch_bounds__(kChiThreads) chi_sums_kernel(const int64_t *__restrict__ chi,
                                                               const int64_t *__restrict__ count,
                                                               int64_t *__restrict__ sums) {
    __shared__ int64_t sh[kChiThreads / 64];
    const int64_t K = *count, nt = (K + kChiTile - 1) / kChiTile;
    const int tid = threadIdx.x;
    for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        int64_t s = 0;
#pragma unroll
        for (int j = 0; j < kChiItems; ++j) {
            const int64_t i = t * kChiTile + (int64_t)j * kChiThreads + tid;
            if (i < K) s += chi[i];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if ((tid & 63) == 0) sh[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) sums[t] = sh[0] + sh[1] + sh[2] + sh[3];
        __syncthreads();
    }
}

__global__ void __launch_bounds__(1024) chi_scan_kernel(const int64_t *__restrict__ count, int64_t *__restrict__ sums) {
    __shared__ int64_t ws[16];
    const int64_t nt = (*count + kChiTile - 1) / kChiTile;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t carry = 0;
    // four entries per thread and round
    for (int64_t c0 = 0; c0 < nt; c0 += 4096) {
        const int64_t i0 = c0 + 4 * (int64_t)tid;
        int64_t v[4], s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = i0 + j < nt ? sums[i0 + j] : 0;
            s += v[j];
        }
        int64_t x = s;
        x = wave_prefix(x);
        if (lane == 63) ws[wave] = x;
        __syncthreads();
        int64_t p = carry + x - s;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) p += ws[w];
            carry += ws[w];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (i0 + j < nt) sums[i0 + j] = p;
            p += v[j];
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kChiThreads) chi_prefix_kernel(int64_t *__restrict__ chi,
                                                                 const int64_t *__restrict__ count,
                                                                 const int64_t *__restrict__ sums) {
    // LDS slot of entry i: one pad word per 16, so that a thread's run of 16
    // spreads over the banks
    __shared__ int64_t st[kChiTile + kChiTile / 16];
    __shared__ int64_t ws[kChiThreads / 64];
    const int64_t K = *count, nt = (K + kChiTile - 1) / kChiTile;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
        const int64_t t0 = t * kChiTile;
#pragma unroll
        for (int j = 0; j < kChiItems; ++j) {
            const int i = j * kChiThreads + tid;
            st[i + (i >> 4)] = t0 + i < K ? chi[t0 + i] : 0;
        }
        __syncthreads();
        int64_t v[kChiItems], s = 0;
#pragma unroll
        for (int j = 0; j < kChiItems; ++j) {
            v[j] = st[tid * 17 + j];
            s += v[j];
        }
        int64_t x = s;
        x = wave_prefix(x);
        if (lane == 63) ws[wave] = x;
        __syncthreads();
        int64_t p = sums[t] + x - s;
        for (int w = 0; w < wave; ++w) p += ws[w];
#pragma unroll
        for (int j = 0; j < kChiItems; ++j) {
            p += v[j];
            st[tid * 17 + j] = p;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kChiItems; ++j) {
            const int i = j * kChiThreads + tid;
            if (t0 + i < K) chi[t0 + i] = st[i + (i >> 4)];
        }
        __syncthreads();
    }
}

size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }

// scratch of P top bytes and up to n values
struct Layout {
    size_t bits, ord, blk, total, base, list, sums, bytes;
    int words, tiles;
};
Layout layout(int present, int64_t n) {
    Layout L{};
    L.words = present * kWordsPerByte;
    L.tiles = L.words / kTileWords;
    const size_t all = up256((size_t)L.words * kBuckets * 4);
    L.bits = 0;
    L.ord = all;
    L.blk = 2 * all;
    L.total = L.blk + up256((size_t)L.tiles * kTileBlocks * 4);
    L.base = L.total + up256((size_t)L.tiles * 4);
    L.list = L.base + up256((size_t)(L.tiles + 2) * 4);
    L.sums = L.list + up256((size_t)(L.tiles + 1) * 4);
    L.bytes = L.sums + up256((size_t)((n + kChiTile - 1) / kChiTile) * 8);
    return L;
}

}  // namespace

size_t distinct_scratch_bytes(int present, int64_t n) { return layout(present, n).bytes; }

static int split_grid(int64_t n) {
    return (int)std::min<int64_t>((n + kTile - 1) / kTile, 2 * device_cu_count());
}
size_t split_head_bytes(int64_t n) { return (8 + (size_t)(1 + split_grid(n)) * kBuckets) * 4; }

int launch_split(const float *img, int64_t n, uint32_t *keys, uint16_t *starts, uint32_t *head, uint32_t *mask_host_dev,
                 uint32_t *status, hipEvent_t noted, hipStream_t stream) {
    if (n < 1 || n >= ((int64_t)1 << 30)) {
        set_error("internal error: split of %lld values", (long long)n);
        return ECC_E_ARG;
    }
    int rc = launch_zero(head, 8 * 4, stream);
    if (rc) return rc;
    const int64_t tiles = (n + kTile - 1) / kTile;
    const int grid = split_grid(n);
    uint32_t *totals = head + 8, *rows = totals + kBuckets;
    hipLaunchKernelGGL(split_kernel, dim3((unsigned)grid), dim3(kThreads), 0, stream, img, n, tiles, keys, starts, rows,
                       head, status);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(bucket_totals_kernel, dim3(kBuckets / 64), dim3(1024), 0, stream, (const uint32_t *)rows, grid,
                       totals, (const uint32_t *)head, mask_host_dev);
    ECC_HIP(hipGetLastError());
    ECC_HIP(hipEventRecord(noted, stream));
    return ECC_OK;
}

int launch_distinct_curve(int64_t n, int present, const uint32_t *keys, const uint16_t *starts, const uint32_t *head,
                          void *scratch, const uint64_t *nz, const uint32_t *nz_cnt, int64_t regions,
                          int64_t region_slots, float *out_keys, int64_t *out_chi, int64_t *count, int64_t *count_host,
                          const uint32_t *status, uint32_t *status_host, hipStream_t stream) {
    if (present < 1 || present > kMaxDistinctBytes || n < 1 || n >= ((int64_t)1 << 30)) {
        set_error("internal error: %d top bytes, %lld values", present, (long long)n);
        return ECC_E_ARG;
    }
    const uint32_t *mask = head, *totals = head + 8;
    const Layout L = layout(present, n);
    uint8_t *b = (uint8_t *)scratch;
    uint32_t *bits = (uint32_t *)(b + L.bits), *ord = (uint32_t *)(b + L.ord), *blk = (uint32_t *)(b + L.blk);
    uint32_t *total = (uint32_t *)(b + L.total), *base = (uint32_t *)(b + L.base), *list = (uint32_t *)(b + L.list);
    int64_t *sums = (int64_t *)(b + L.sums);
    const int64_t tiles = (n + kTile - 1) / kTile;
    int rc = launch_zero(bits, (size_t)L.words * kBuckets * 4, stream);
    if (rc) return rc;
    // evenly filled buckets are one share each (a fifth above the mean)
    const int64_t share = std::max<int64_t>(4096, n / kBuckets + n / kBuckets / 5);
    const int64_t grid = kBuckets + n / share;
    hipLaunchKernelGGL(bucket_bits_kernel, dim3((unsigned)grid), dim3(kThreads), (size_t)L.words * 4, stream, keys, n,
                       (int)tiles, starts, totals, mask, (uint32_t)share, L.words, bits);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(order_bits_kernel, dim3((unsigned)L.tiles), dim3(256), 0, stream, (const uint32_t *)bits, L.words,
                       ord, blk, total);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(tile_base_kernel, dim3(1), dim3(1024), 0, stream, (const uint32_t *)total, L.tiles, totals,
                       (uint32_t)(n / kBuckets + n / kBuckets / 8 + 64), base, list, count, count_host, status, status_host);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(expand_kernel, dim3((unsigned)std::min(L.tiles * kExpandParts, 16 * device_cu_count())),
                       dim3(64 * kExpandWaves), 0, stream, (const uint32_t *)ord, (const uint32_t *)blk,
                       (const uint32_t *)base, (const uint32_t *)list, mask, out_keys, out_chi);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(add_records_kernel, dim3((unsigned)std::min<int64_t>((regions + 15) / 16, 2048)),
                       dim3(1024), 0, stream, nz, nz_cnt, regions, region_slots, (const uint32_t *)ord,
                       (const uint32_t *)blk, (const uint32_t *)base, L.tiles, mask, out_chi);
    ECC_HIP(hipGetLastError());
    // (K is at most n)
    const unsigned cg = (unsigned)std::min<int64_t>((n + kChiTile - 1) / kChiTile, 4096);
    hipLaunchKernelGGL(chi_sums_kernel, dim3(cg), dim3(kChiThreads), 0, stream, (const int64_t *)out_chi,
                       (const int64_t *)count, sums);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(chi_scan_kernel, dim3(1), dim3(1024), 0, stream, (const int64_t *)count, sums);
    ECC_HIP(hipGetLastError());
    hipLaunchKernelGGL(chi_prefix_kernel, dim3(cg), dim3(kChiThreads), 0, stream, out_chi, (const int64_t *)count,
                       (const int64_t *)sums);
    ECC_HIP(hipGetLastError());
    return ECC_OK;
}

}  // namespace ecc
