// Per-voxel changes of images that are not counted value by value in the
// integer kernel's histograms: float images (every voxel whose change is not
// zero leaves a record) and integer images with four axes longer than 1.
//
// The change of the curve at a voxel's value is the signed count of the cells
// whose value the voxel gives (Sec. 3, Algorithm 1; Sec. 2, "Sublevel Set
// Filtration": a cell's value is the minimum over the voxels that contain
// it).  Any choice among equal minima gives the same curve, since the cell's
// value is what is counted.
//
// Algorithm 1 inspects the 3^d - 1 neighbours of a voxel.  Here each cell is
// looked at once instead: of the 2^d cell types per voxel (an axis of a cell
// is an interval, the voxel's own, or a vertex between two voxels), the
// minimum of a type with one more vertex axis is the smaller of two minima
// of the type without it, so one comparison per cell tells which of the two
// gave it (2^d - 1 comparisons and minima per voxel: 15 in place of 80 for
// d = 4), and the cell's sign is passed along these comparisons, axis by
// axis, to the voxel that gave the minimum:
//  1. axis 0 (walked): for every set S of the other axes, the field F_S is
//     the 2-window minimum of the image along the axes of S.  Edge i of a
//     line of F_S along axis 0 keeps r_S = c_{i-1} - c_i, c_i = [F_S at i+1 <
//     F_S at i] (a vertex goes to the smaller of its two edges and cancels
//     it); c = 1 before the first and 0 after the last plane;
//  2. the last axis x: r_{S+x} goes to the position x-1 if F_{S+x} < F_S
//     there (the left value is strictly smaller), else to x, and is
//     subtracted from r_S;
//  3. the other in-plane axes y, then z, in the same way.
// What is left at a voxel, times (-1)^(in-plane axes), is its change.  On the
// far edge of an in-plane axis, the field with and the field without it have
// equal lines and cancel, so the field without it is skipped there and the
// field with it never reaches past the edge (as in the integer kernel).
//
// Layout.  A lane holds A x B voxels: rows y0 .. y0+A-1 of the planes z0 ..
// z0+B-1, at one x, and walks axis 0.  It loads those rows and one row on
// either side per axis ((A+2)(B+2) values per plane, clamped into the image:
// equal values never pass anything outwards).  The lanes of a wave are 64
// consecutive positions of the flattened (row group, x) index, so that lines
// of any length fill the waves; the first and the last lane serve their
// neighbours only (62 of 64 emit, all of them at the ends of the index).  A
// value at x-1 comes from the lane before (wave shift), and what goes to x-1
// goes to the lane before.
// The r of up to four types (without and with y, z) of one position are the
// bytes of one word: the comparison masks are pushed into the low bits
// of a word, spread to bytes by one 24-bit product, and steps 1 and 2 work
// on whole words.
// Bound by vector instructions: a 128^4 float image takes 0.99 ms, of which
// 132 instructions per voxel take 0.90 ms to issue (1.06 ms with the planes
// after the last one made by moves and stores under branches).
#include <algorithm>

#include "ecc_internal.h"

namespace ecc {

namespace {

constexpr uint32_t kBufWord3 = 0x00020000;
constexpr int kShr1 = 0x138;  // lane i reads lane i-1
constexpr int kShl1 = 0x130;  // lane i reads lane i+1

struct ChangeParams {
    PlaneSrc src;
    int32_t nx, ny, nz;      // in-plane extents (1 where the axis is absent)
    int32_t lanes;           // flattened length: row groups * nx
    int32_t wu;              // waves over it
    int32_t nzt;             // groups of B planes along z
    int32_t e0, e1;          // emitted planes of axis 0, buffer coordinates
    int32_t lo_inf, hi_inf;  // planes e0-1 and e1 lie outside the image
    int32_t zc;              // planes of axis 0 per walk
    int64_t items;           // waves of work
    uint32_t invert;         // integers: values read as v ^ invert
    // records (float): item i's region is rec[i * region ..], its count cnt[i]
    uint64_t *rec;
    uint32_t *cnt;
    uint32_t region;
    // integers: count rows, one per workgroup or (kAtomic) `rows` shared ones
    int32_t *partial;
    uint32_t rows;
    uint32_t *status;
    uint32_t limit;  // integers: values >= limit are an error
};

template <typename T>
struct Val {
    using type = uint32_t;
};
template <>
struct Val<float> {
    using type = float;
};

__device__ __forceinline__ uint32_t vmin(uint32_t a, uint32_t b) { return a < b ? a : b; }
// (as written, without the quieting of its inputs that fminf adds: a NaN
// input only occurs in an image that is rejected, or as the absent left
// value below, where the other input is returned)
__device__ __forceinline__ float vmin(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ uint32_t bits_of(uint32_t v) { return v; }
__device__ __forceinline__ uint32_t bits_of(float v) { return __float_as_uint(v); }
__device__ __forceinline__ void from_bits(uint32_t b, uint32_t &v) { v = b; }
__device__ __forceinline__ void from_bits(uint32_t b, float &v) { v = __uint_as_float(b); }

// The comparisons x < y of two or four pairs as the low bits of a word, the
// first pair's highest.  A vector instruction may read a mask only two wait
// states after the comparison that wrote it, and the compiler does not add
// them around inline assembly: each block holds its comparisons and what reads
// their masks, the ones of the other pairs in between.
#define ECC_CMP(type, mask, x, y) "v_cmp_lt_" type "_e64 " mask ", " x ", " y "\n\t"
#define ECC_PUSH(mask) "v_addc_co_u32_e64 %0, %1, %0, %0, " mask "\n\t"  // m = 2 m + (lane bit)
#define ECC_LT2(type)                                                                                       \
    uint32_t m;                                                                                             \
    uint64_t k1, k0;                                                                                        \
    asm(ECC_CMP(type, "%1", "%3", "%4") ECC_CMP(type, "%2", "%5", "%6") "s_nop 0\n\t"                       \
        "v_cndmask_b32_e64 %0, 0, 1, %1\n\t" ECC_PUSH("%2")                                                 \
        : "=&v"(m), "=&s"(k1), "=&s"(k0)                                                                    \
        : "v"(x1), "v"(y1), "v"(x0), "v"(y0));                                                              \
    return m;
#define ECC_LT4(type)                                                                                       \
    uint32_t m;                                                                                             \
    uint64_t k3, k2, k1, k0;                                                                                \
    asm(ECC_CMP(type, "%1", "%5", "%6") ECC_CMP(type, "%2", "%7", "%8") ECC_CMP(type, "%3", "%9", "%10")      \
        ECC_CMP(type, "%4", "%11", "%12") "v_cndmask_b32_e64 %0, 0, 1, %1\n\t" ECC_PUSH("%2") ECC_PUSH("%3") \
        ECC_PUSH("%4")                                                                                      \
        : "=&v"(m), "=&s"(k3), "=&s"(k2), "=&s"(k1), "=&s"(k0)                                              \
        : "v"(x3), "v"(y3), "v"(x2), "v"(y2), "v"(x1), "v"(y1), "v"(x0), "v"(y0));                          \
    return m;
__device__ __forceinline__ uint32_t lt2(float x1, float y1, float x0, float y0) { ECC_LT2("f32") }
__device__ __forceinline__ uint32_t lt2(uint32_t x1, uint32_t y1, uint32_t x0, uint32_t y0) { ECC_LT2("u32") }
__device__ __forceinline__ uint32_t lt4(float x3, float y3, float x2, float y2, float x1, float y1, float x0, float y0) {
    ECC_LT4("f32")
}
__device__ __forceinline__ uint32_t lt4(uint32_t x3, uint32_t y3, uint32_t x2, uint32_t y2, uint32_t x1, uint32_t y1,
                                        uint32_t x0, uint32_t y0) {
    ECC_LT4("u32")
}
#undef ECC_LT4
#undef ECC_LT2
#undef ECC_PUSH
#undef ECC_CMP

// Cell types of a position: bit 0: y is a vertex axis, bit 1: z is one; type
// t's byte of a word is byte t.  At row position a == A (the row past the
// lane's own) only the types with y are needed, at b == B only those with z.
template <int NL, int A, int B>
struct Types {
    static constexpr bool has(int a, int b, int t) {
        if ((t & 1) && NL < 1) return false;
        if ((t & 2) && NL < 2) return false;
        if (a == A && !(t & 1)) return false;
        if (b == B && !(t & 2)) return false;
        return true;
    }
    // The packed bits (present types, ascending from bit 0) to the low bits of
    // their bytes: one product, whose terms do not meet (other bits of the
    // bytes may be set); a single type's bit is shifted, since a factor of
    // 2^24 is beyond the 24-bit product.
    static __device__ __forceinline__ uint32_t spread(uint32_t m, int a, int b) {
        uint32_t f = 0;
        int j = 0, last = 0;
        for (int t = 0; t < 4; ++t)
            if (has(a, b, t)) f += 1u << (8 * t - j), ++j, last = t;
        return j == 1 ? m << (8 * last) : __umul24(m, f);
    }
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
enum { kRecords = 0, kHistogram = 1, kAtomic = 2 };

// EMIT: kRecords (float), kHistogram (integers, m = M bins in LDS, one count
// row per workgroup), kAtomic (integers, adds to the rows in memory, workgroup b
// to row b modulo their number).
template <typename T, int NL, int EMIT, int M, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) change_kernel(ChangeParams P) {
    using V = typename Val<T>::type;
    constexpr int A = NL == 0 ? 1 : NL == 1 ? 4 : 2;
    constexpr int B = NL == 2 ? 2 : 1;
    constexpr int HY = NL >= 1, HZ = NL == 2;
    constexpr int RA = A + 2 * HY, RB = B + 2 * HZ;  // loaded rows
    constexpr int PA = A + HY, PB = B + HZ;          // positions
    using Ty = Types<NL, A, B>;
    constexpr uint32_t kBias = 0x08080808u;
    __shared__ int32_t hist[EMIT == kHistogram ? M : 1];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if constexpr (EMIT == kHistogram) {
        for (int i = threadIdx.x; i < M; i += 64 * WAVES) hist[i] = 0;
        __syncthreads();
    }
    uint32_t orv = 0;
    int32_t *shared_row = nullptr;
    if constexpr (EMIT == kAtomic) shared_row = P.partial + (size_t)(blockIdx.x % P.rows) * 65536u;
    const uint32_t blk = xcd_block(blockIdx.x, gridDim.x);
    for (int64_t item = (int64_t)blk * WAVES + wave; item < P.items; item += (int64_t)gridDim.x * WAVES) {
        const int32_t k = (int32_t)(item % P.wu);
        const int32_t rest = (int32_t)(item / P.wu);
        const int32_t zt = rest % P.nzt;
        const int32_t zs = P.e0 + (rest / P.nzt) * P.zc;
        const int32_t ze = min(zs + P.zc, P.e1);
        const int32_t z0 = zt * B;

        const int32_t u = 62 * k + lane;
        const bool in = u < P.lanes;
        const int32_t uc = min(u, P.lanes - 1);
        const int32_t yt = uc / P.nx, x = uc - yt * P.nx;
        const int32_t y0 = yt * A;
        // lanes that emit: all but the first (unless it starts the index)
        // and the last (unless it ends it)
        const uint64_t emit = __builtin_amdgcn_ballot_w64(in && (lane > 0 || k == 0) && (lane < 63 || u == P.lanes - 1));

        // loaded rows: per lane the row's byte offset with x, per wave the
        // plane's offset along z
        uint32_t vo[RA], zo[RB];
#pragma unroll
        for (int a = 0; a < RA; ++a)
            vo[a] = ((uint32_t)min(max(y0 + a - HY, 0), P.ny - 1) * (uint32_t)P.nx + (uint32_t)x) * (uint32_t)sizeof(T);
#pragma unroll
        for (int b = 0; b < RB; ++b)
            zo[b] = (uint32_t)min(max(z0 + b - HZ, 0), P.nz - 1) * (uint32_t)P.ny * (uint32_t)P.nx * (uint32_t)sizeof(T);
        const uint32_t x0m = x == 0 ? 0xFFFFFFFFu : 0u;  // no left value
        // validity of the types per row and plane position (low bits of the
        // bytes): a type without an axis stops before its last index
        uint32_t my[PA], myx[PA], mz[PB];
#pragma unroll
        for (int a = 0; a < PA; ++a) {
            const int32_t y = y0 + a;
            my[a] = 0;
            if (in) my[a] = (HY == 0 || y <= P.ny - 2 ? 0x00010001u : 0u) | (HY && y <= P.ny - 1 ? 0x01000100u : 0u);
            myx[a] = x <= P.nx - 2 ? my[a] : 0u;
        }
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            const int32_t z = z0 + b;
            mz[b] = (HZ == 0 || z <= P.nz - 2 ? 0x00000101u : 0u) | (HZ && z <= P.nz - 1 ? 0x01010000u : 0u);
        }

        auto plane_ptr = [&](int32_t p) { return (p < 0 ? P.src.lo_base : P.src.base) + (int64_t)p * P.src.plane_bytes; };
        auto load = [&](int32_t p, V (&f)[RA][RB]) {
            __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)plane_ptr(p), (short)0,
                                                                          (int)(uint32_t)P.src.plane_bytes, kBufWord3);
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    if constexpr (sizeof(T) == 4) from_bits(__builtin_amdgcn_raw_buffer_load_b32(rs, vo[a], zo[b], 0), f[a][b]);
                    else if constexpr (sizeof(T) == 2) from_bits(__builtin_amdgcn_raw_buffer_load_b16(rs, vo[a], zo[b], 0), f[a][b]);
                    else from_bits(__builtin_amdgcn_raw_buffer_load_b8(rs, vo[a], zo[b], 0), f[a][b]);
                }
        };
        // fields of a plane: g[a][b][t][0] without x, [1] with x
        auto fields = [&](const V (&f0)[RA][RB], V (&g)[PA][PB][4][2]) {
            V f[RA][RB][2];
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int b = 0; b < RB; ++b) {
                    V v = f0[a][b];
                    if constexpr (sizeof(T) < 4) v ^= P.invert;
                    f[a][b][0] = v;
                    // the left value: all ones at x = 0 (a NaN, or the
                    // largest integer), which the minimum passes over
                    const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)bits_of(v), kShr1, 0xF, 0xF, true) | x0m;
                    V left;
                    from_bits(l, left);
                    f[a][b][1] = vmin(v, left);
                }
#pragma unroll
            for (int xi = 0; xi < 2; ++xi) {
                V fy[PA][RB];
                if constexpr (HY) {
#pragma unroll
                    for (int a = 0; a < PA; ++a)
#pragma unroll
                        for (int b = 0; b < RB; ++b) fy[a][b] = vmin(f[a][b][xi], f[a + 1][b][xi]);
                }
#pragma unroll
                for (int a = 0; a < PA; ++a)
#pragma unroll
                    for (int b = 0; b < PB; ++b) {
                        g[a][b][0][xi] = f[a + HY][b + HZ][xi];
                        if constexpr (HY) g[a][b][1][xi] = fy[a][b + HZ];
                        if constexpr (HZ) {
                            g[a][b][2][xi] = vmin(f[a + HY][b][xi], f[a + HY][b + 1][xi]);
                            g[a][b][3][xi] = vmin(fy[a][b], fy[a][b + 1]);
                        }
                    }
            }
        };
        // x(t) < y(t) for the types t at a position, spread to their bytes
        auto gather = [&](int a, int b, auto &&x, auto &&y) -> uint32_t {
            int ty[4], n = 0;
#pragma unroll
            for (int t = 3; t >= 0; --t)
                if (Ty::has(a, b, t)) ty[n++] = t;
            uint32_t m;
            if (n == 4) m = lt4(x(ty[0]), y(ty[0]), x(ty[1]), y(ty[1]), x(ty[2]), y(ty[2]), x(ty[3]), y(ty[3]));
            else if (n == 2) m = lt2(x(ty[0]), y(ty[0]), x(ty[1]), y(ty[1]));
            else m = x(ty[0]) < y(ty[0]) ? 1u : 0u;  // (no position has three types)
            return Ty::spread(m, a, b);
        };
        // c of plane i from the fields of planes i and i+1: words without x
        // and with x
        auto compare = [&](const V (&gn)[PA][PB][4][2], const V (&gc)[PA][PB][4][2], int a, int b, uint32_t valid,
                           uint32_t &ca, uint32_t &cb) {
            ca = gather(a, b, [&](int t) { return gn[a][b][t][0]; }, [&](int t) { return gc[a][b][t][0]; }) & myx[a] & valid;
            cb = gather(a, b, [&](int t) { return gn[a][b][t][1]; }, [&](int t) { return gc[a][b][t][1]; }) & my[a] & valid;
        };
        const bool lo_real = !(zs == P.e0 && P.lo_inf);
        const bool hi_real = !(ze == P.e1 && P.hi_inf);

        V gc[PA][PB][4][2];
        uint32_t xw[PA][PB], cw[PA][PB];  // c(without x) - c(with x); c(with x), of the plane before
        V nx[RA][RB];
        load(zs, nx);
        fields(nx, gc);
        if (lo_real) {
            V gl[PA][PB][4][2];
            load(zs - 1, nx);
            fields(nx, gl);
#pragma unroll
            for (int a = 0; a < PA; ++a)
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    uint32_t ca, cb;
                    compare(gc, gl, a, b, mz[b], ca, cb);
                    xw[a][b] = ca - cb;
                    cw[a][b] = cb;
                }
        } else {  // (c = 1 before the first plane)
#pragma unroll
            for (int a = 0; a < PA; ++a)
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    uint32_t tm = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (Ty::has(a, b, t)) tm |= 1u << (8 * t);
                    cw[a][b] = my[a] & mz[b] & tm;
                    xw[a][b] = (myx[a] & mz[b] & tm) - cw[a][b];
                }
        }
        uint32_t count = 0;  // records of this item
        __amdgpu_buffer_rsrc_t records = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(P.rec + (EMIT == kRecords ? item * P.region : 0)), (short)0, (int)(P.region * 8u), kBufWord3);
        // the planes after the last one that is read repeat it
        const int32_t plast = hi_real ? ze : ze - 1;
        auto load_next = [&](int32_t p) { load(min(p, plast), nx); };
        load_next(zs + 1);
        // one plane: fields gc; those of the next plane are left in gn
        auto step = [&](const V (&gc)[PA][PB][4][2], V (&gn)[PA][PB][4][2], int32_t z) {
            uint32_t on[PB];  // c = 0 after the last plane
#pragma unroll
            for (int b = 0; b < PB; ++b) on[b] = z + 1 > plast ? 0u : mz[b];
            fields(nx, gn);
            // (moved up, the loads would need registers of their own and 32
            // copies per plane)
            __builtin_amdgcn_sched_barrier(0);
            load_next(z + 2);
            // steps 1 and 2 at every position: the r of its types, biased by
            // 8 per byte
            uint32_t r[PA][PB];
#pragma unroll
            for (int a = 0; a < PA; ++a)
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    uint32_t ca, cb;
                    compare(gn, gc, a, b, on[b], ca, cb);
                    // types whose left value is strictly smaller
                    const uint32_t m =
                        gather(a, b, [&](int t) { return gc[a][b][t][1]; }, [&](int t) { return gc[a][b][t][0]; });
                    const uint32_t xn = ca - cb;
                    // (what goes to the left, negated, and the rest kept
                    // opaque: the shifted value is then only ever added.  A
                    // subtraction with a shifted operand may be compiled to
                    // v_subrev_u32 with the shift on its first source, and
                    // that form shifted the second source on the card.)
                    const uint32_t left = (cb & m) - (cw[a][b] & m);
                    uint32_t rest = (xw[a][b] + kBias) - xn - left;
                    asm("" : "+v"(rest));
                    r[a][b] = rest + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)left, kShl1, 0xF, 0xF, true);
                    xw[a][b] = xn;
                    cw[a][b] = cb;
                }
            auto byte = [&](uint32_t w, int t) -> int32_t { return (int32_t)((w >> (8 * t)) & 0xFFu); };
            // steps y and z.  u: per position b, what is left at row a of the
            // types without y; biases cancel where y exists (8 - 8), else 8
            constexpr int kOff = NL == 0 ? 8 : 0;
            int32_t fin[A][B];
            V val[A][B];
#pragma unroll
            for (int a = 0; a < A; ++a) {
                int32_t uz[PB];  // the type z at this row
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    auto pass_y = [&](int t0, int t1) -> int32_t {  // type t0 less what comes back of type t1 = t0 + y
                        int32_t s = byte(r[a][b], t0);
                        if constexpr (HY) {
                            const int32_t own = byte(r[a][b], t1);
                            s -= own - (gc[a][b][t1][0] < gc[a][b][t0][0] ? own : 8);
                            s -= gc[a + 1][b][t1][0] < gc[a + 1][b][t0][0] ? byte(r[a + 1][b], t1) : 8;
                        }
                        return s;
                    };
                    if (b < B) {
                        fin[a][b] = pass_y(0, 1);
                        val[a][b] = gc[a][b][0][0];
                    }
                    if constexpr (HZ) uz[b] = pass_y(2, 3);
                }
                if constexpr (HZ) {
#pragma unroll
                    for (int b = 0; b < B; ++b) {
                        const int32_t lz = gc[a][b][2][0] < gc[a][b][0][0] ? uz[b] : 0;
                        const int32_t lz1 = gc[a][b + 1][2][0] < gc[a][b + 1][0][0] ? uz[b + 1] : 0;
                        fin[a][b] -= uz[b] - lz + lz1;
                    }
                }
            }
#pragma unroll
            for (int a = 0; a < A; ++a)
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const uint64_t nz = __builtin_amdgcn_ballot_w64(fin[a][b] != kOff) & emit;
                    const int32_t chg = NL == 1 ? fin[a][b] - kOff : kOff - fin[a][b];
                    if constexpr (EMIT == kRecords) {
                        // (a lane without a record stores past the region's
                        // end, where a buffer store is dropped: with no branch
                        // around the stores their number is known, and the
                        // wait for the next plane's loads, which are older,
                        // need not wait for them)
                        const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(nz >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)nz, 0u));
                        const uint32_t to = __builtin_amdgcn_inverse_ballot_w64(nz) ? at * 8u : 0x80000000u;
                        const u32x2 record = {(uint32_t)chg, f32_key(bits_of(val[a][b]))};
                        __builtin_amdgcn_raw_buffer_store_b64(record, records, to, count * 8u, 0);
                        count += (uint32_t)__builtin_popcountll(nz);
                    } else {
                        if (__builtin_amdgcn_inverse_ballot_w64(emit) && y0 + a < P.ny && z0 + b < P.nz) orv |= bits_of(val[a][b]);
                        if (__builtin_amdgcn_inverse_ballot_w64(nz)) {
                            const uint32_t v = bits_of(val[a][b]);
                            if constexpr (EMIT == kHistogram) {
                                if (v < (uint32_t)M) atomicAdd(&hist[v], chg);
                            } else {
                                if (v < P.limit) atomicAdd(&shared_row[v], chg);
                            }
                        }
                    }
                }
        };
        if constexpr (EMIT == kRecords) {
            // (dropped; as many stores behind the loads as after a step, so
            // that the wait at the loop's head is the same on both ways in)
#pragma unroll
            for (int k = 0; k < A * B; ++k)
                __builtin_amdgcn_raw_buffer_store_b64((u32x2){0u, 0u}, records, 0x80000000u, 0, 0);
        }
        V gd[PA][PB][4][2];
        for (int32_t z = zs;; z += 2) {
            step(gc, gd, z);
            if (z + 1 >= ze) break;
            step(gd, gc, z + 1);
            if (z + 2 >= ze) break;
        }
        if constexpr (EMIT == kRecords) {
            if (lane == 0) P.cnt[item] = count;
        }
    }
    if constexpr (EMIT != kRecords) {
        if (__builtin_amdgcn_ballot_w64(orv >= P.limit) != 0 && lane == 0) atomicOr(P.status, kStatusRange);
    }
    if constexpr (EMIT == kHistogram) {
        __syncthreads();
        int32_t *dst = P.partial + (size_t)blockIdx.x * M;
        for (int i = threadIdx.x; i < M; i += 64 * WAVES) dst[i] = hist[i];
    }
}

}  // namespace

// Geometry of a launch.
static int change_params(const ChangeJob &job, int per_lane_a, int per_lane_b, ChangeParams *p) {
    p->src = job.src;
    p->nx = job.nx;
    p->ny = job.ny;
    p->nz = job.nz;
    const int64_t lanes = (int64_t)((job.ny + per_lane_a - 1) / per_lane_a) * job.nx;
    if (lanes > INT32_MAX || job.src.plane_bytes > (int64_t)UINT32_MAX) {
        set_error("change kernel: plane too large");
        return ECC_E_UNSUPPORTED;
    }
    p->lanes = (int32_t)lanes;
    p->wu = lanes <= 64 ? 1 : (int32_t)((lanes - 2 + 61) / 62);
    p->nzt = (job.nz + per_lane_b - 1) / per_lane_b;
    p->e0 = job.e0;
    p->e1 = job.e1;
    p->lo_inf = job.lo_inf;
    p->hi_inf = job.hi_inf;
    const int64_t planes = job.e1 - job.e0, per_plane = (int64_t)p->wu * p->nzt;
    const int64_t target = (int64_t)device_cu_count() * 48;
    int64_t chunks = (target + per_plane - 1) / per_plane;
    int64_t zc = chunks >= planes ? 1 : (planes + chunks - 1) / chunks;
    if (zc < 8) zc = 8;
    if (zc > planes) zc = planes;
    p->zc = (int32_t)zc;
    p->items = per_plane * ((planes + zc - 1) / zc);
    if (p->items / p->wu > INT32_MAX) {
        set_error("change kernel: too many lines");
        return ECC_E_UNSUPPORTED;
    }
    p->invert = 0;
    return ECC_OK;
}

static int lane_rows(int nl) { return nl == 0 ? 1 : nl == 1 ? 4 : 2; }
static int lane_planes(int nl) { return nl == 2 ? 2 : 1; }

// Records of one walk at most: a voxel of each of the wave's lanes (planes of
// fewer than 64 positions have fewer lanes that emit) per plane.
static int64_t walk_records(const ChangeParams &p, int a, int b) {
    return (int64_t)std::min(64, p.lanes) * a * b * p.zc;
}

int change_regions(const ChangeJob &job, int64_t *regions, int64_t *region_slots) {
    ChangeParams p{};
    const int a = lane_rows(job.nl), b = lane_planes(job.nl);
    int rc = change_params(job, a, b, &p);
    if (rc) return rc;
    *regions = p.items;
    *region_slots = walk_records(p, a, b);
    return ECC_OK;
}

int launch_change_records(const ChangeJob &job, uint64_t *rec, uint32_t *cnt, hipStream_t stream) {
    ChangeParams p{};
    const int a = lane_rows(job.nl), b = lane_planes(job.nl);
    int rc = change_params(job, a, b, &p);
    if (rc) return rc;
    p.rec = rec;
    p.cnt = cnt;
    p.region = (uint32_t)walk_records(p, a, b);
    void *tok = nullptr;
    rc = profile_begin(stream, &tok);
    if (rc) return rc;
    const dim3 grid((unsigned)((p.items + 3) / 4)), block(256);
    switch (job.nl) {
    case 0: hipLaunchKernelGGL((change_kernel<float, 0, kRecords, 1, 4>), grid, block, 0, stream, p); break;
    case 1: hipLaunchKernelGGL((change_kernel<float, 1, kRecords, 1, 4>), grid, block, 0, stream, p); break;
    default: hipLaunchKernelGGL((change_kernel<float, 2, kRecords, 1, 4>), grid, block, 0, stream, p); break;
    }
    ECC_HIP(hipGetLastError());
    return profile_end(stream, tok);
}

// Integer images: 4-D only (nl = 2).  Eight waves per workgroup share a
// 16384-bin histogram (64 KiB of LDS), one workgroup per CU (two waves per
// SIMD at the kernel's registers); the 256-bin form has four per workgroup.
// The workgroups take items in turn, so there is one count row per workgroup
// of a grid of at most one (16384 bins) or four (256 bins) per CU.  Bins and
// rows are int32: a launch has less than 2^30 values (of a resident image, and
// of a stream's launches), its items go round all workgroups of a full grid, so
// that one counts at most some 2^23 voxels, and a voxel's change is at most 16.
static int int_geometry(const ChangeJob &job, ChangeParams *p, int *waves, int64_t *grid) {
    if (job.nl != 2) {
        set_error("internal error: integer change kernel on %d line axes", job.nl);
        return ECC_E_ARG;
    }
    int rc = change_params(job, lane_rows(2), lane_planes(2), p);
    if (rc) return rc;
    const bool wide = job.dtype == ECC_U14;
    *waves = wide ? 8 : 4;
    *grid = std::min<int64_t>((p->items + *waves - 1) / *waves, (int64_t)device_cu_count() * (wide ? 1 : 4));
    p->invert = job.invert ? (uint32_t)threshold_count(job.dtype) - 1u : 0u;
    p->limit = (uint32_t)threshold_count(job.dtype);
    return ECC_OK;
}

// 16-bit images (more bins than a workgroup's LDS holds) add to rows in memory.
// Adds to one line wait for each other (0.2 G/s, 27 G/s on many lines), and an
// image of few values makes all its adds on few lines: with one row, 60^4 voxels
// of two values took 30 ms.  A row per 8192 voxels, up to 64, keeps that to the
// rate of the adds; the rows' clearing and merging then take about as long as
// the launch of a small image.
int change_count_rows(const ChangeJob &job, int *rows) {
    ChangeParams p{};
    int waves = 0;
    int64_t grid = 0;
    int rc = int_geometry(job, &p, &waves, &grid);
    if (rc) return rc;
    const int64_t voxels = (int64_t)(job.e1 - job.e0) * job.nx * job.ny * job.nz;
    // (a multiple of 8: the workgroups of a row are then on one XCD)
    *rows = job.dtype == ECC_U16 ? (int)std::min<int64_t>(64, (voxels / 8192 + 8) / 8 * 8) : (int)grid;
    return ECC_OK;
}

int launch_change_counts(const ChangeJob &job, int32_t *partial, uint32_t *status, hipStream_t stream) {
    ChangeParams p{};
    int waves = 0, rows = 0;
    int64_t grid = 0;
    int rc = int_geometry(job, &p, &waves, &grid);
    if (!rc) rc = change_count_rows(job, &rows);
    if (!rc && job.dtype == ECC_U16) rc = launch_zero(partial, (size_t)rows * 65536 * sizeof(int32_t), stream);
    if (rc) return rc;
    p.partial = partial;
    p.rows = (uint32_t)rows;
    p.status = status;
    void *tok = nullptr;
    rc = profile_begin(stream, &tok);
    if (rc) return rc;
    const dim3 g((unsigned)grid);
    switch (job.dtype) {
    case ECC_U8: hipLaunchKernelGGL((change_kernel<uint8_t, 2, kHistogram, 256, 4>), g, dim3(256), 0, stream, p); break;
    case ECC_U14: hipLaunchKernelGGL((change_kernel<uint16_t, 2, kHistogram, 16384, 8>), g, dim3(512), 0, stream, p); break;
    default: hipLaunchKernelGGL((change_kernel<uint16_t, 2, kAtomic, 1, 4>), g, dim3(256), 0, stream, p); break;
    }
    ECC_HIP(hipGetLastError());
    return profile_end(stream, tok);
}

}  // namespace ecc
