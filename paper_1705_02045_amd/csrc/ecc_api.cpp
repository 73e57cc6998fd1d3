// C ABI of libecc: argument checks, views, workspaces and the resident path.
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <tuple>
#include <mutex>
#include <utility>
#include <vector>

#include "ecc_internal.h"

#include <algorithm>
#include <atomic>

namespace ecc {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}

void g_err_clear() { g_err[0] = 0; }

int hip_fail(hipError_t e, const char *what) {
    set_error("%s failed: %s", what, hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? ECC_E_NOMEM : ECC_E_HIP;
}

int64_t threshold_count(int dtype) {
    switch (dtype) {
    case ECC_U8: return 256;
    case ECC_U14: return 16384;
    case ECC_U16: return 65536;
    default: return -1;
    }
}

size_t elem_bytes(int dtype) {
    switch (dtype) {
    case ECC_U8: return 1;
    case ECC_U14:
    case ECC_U16: return 2;
    case ECC_F32: return 4;
    default: return 0;
    }
}

int device_cu_count() {
    static std::atomic<int> known[16] = {};  // per device, 0: not asked yet
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (dev >= 0 && dev < 16 && (cus = known[dev].load(std::memory_order_relaxed)) > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 256;
    if (dev >= 0 && dev < 16) known[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// Allocation-failure injection (testing the error paths): with
// ECC_FAIL_ALLOC=k set, the k-th and every later device or pinned-host
// allocation the library attempts fails as out of memory; the count restarts
// whenever the variable's value changes.
static std::mutex g_fail_mu;
static std::string g_fail_val;
static int64_t g_fail_count = 0;

static bool injected_failure() {
    const char *v = getenv("ECC_FAIL_ALLOC");
    std::lock_guard<std::mutex> lk(g_fail_mu);
    const std::string cur = v ? v : "";
    if (cur != g_fail_val) {
        g_fail_val = cur;
        g_fail_count = 0;
    }
    if (cur.empty()) return false;
    const int64_t k = atoll(cur.c_str());
    return k > 0 && ++g_fail_count >= k;
}

// Device blocks of finished ecc_stream objects, kept for the next ones (a
// block is given to one object at a time, and comes back when the work that
// used it is done).  At most kCacheBlocks blocks and kCacheBytes are kept, the
// oldest making room, none above kCacheBlock; ecc_release_workspaces frees them,
// and so does any allocation that finds no memory.
constexpr size_t kCacheBytes = (size_t)256 << 20, kCacheBlock = (size_t)64 << 20;
constexpr int kCacheBlocks = 64;
struct CachedBlock {
    int dev;
    void *p;
    size_t bytes;
};
static std::mutex g_cache_mu;
static CachedBlock g_cache[kCacheBlocks];  // oldest first
static int g_cache_n = 0;
static size_t g_cache_held = 0;

// Takes block i out (g_cache_mu held).
static CachedBlock cache_take(int i) {
    const CachedBlock c = g_cache[i];
    g_cache_held -= c.bytes;
    for (--g_cache_n; i < g_cache_n; ++i) g_cache[i] = g_cache[i + 1];
    return c;
}

hipError_t cache_release(int dev) {
    CachedBlock mine[kCacheBlocks];
    int n = 0;
    {
        std::lock_guard<std::mutex> lk(g_cache_mu);
        for (int i = 0; i < g_cache_n;) {
            if (g_cache[i].dev == dev) mine[n++] = cache_take(i);
            else ++i;
        }
    }
    hipError_t first = hipSuccess;
    for (int i = 0; i < n; ++i) {
        const hipError_t e = hipFree(mine[i].p);
        if (e != hipSuccess && first == hipSuccess) first = e;
    }
    return first;
}

// hipMalloc on dev, the current device; where there is no memory, again
// without the kept blocks.  (The runtime's own record of the failure is
// cleared: the caller reports it, and no later launch does.)
static hipError_t malloc_without_cache(int dev, void **p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    (void)cache_release(dev);
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

hipError_t dev_malloc(void **p, size_t bytes) {
    if (injected_failure()) return hipErrorOutOfMemory;
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    return e == hipSuccess ? malloc_without_cache(dev, p, bytes) : e;
}

hipError_t cache_malloc(int dev, void **p, size_t bytes, size_t *got) {
    if (injected_failure()) return hipErrorOutOfMemory;
    bytes = (bytes + 4095) & ~(size_t)4095;
    {
        std::lock_guard<std::mutex> lk(g_cache_mu);
        int best = -1;  // the smallest that fits and is at most a quarter larger
        for (int i = 0; i < g_cache_n; ++i)
            if (g_cache[i].dev == dev && g_cache[i].bytes >= bytes && g_cache[i].bytes <= bytes + bytes / 4 &&
                (best < 0 || g_cache[i].bytes < g_cache[best].bytes))
                best = i;
        if (best >= 0) {
            const CachedBlock c = cache_take(best);
            *p = c.p;
            *got = c.bytes;
            return hipSuccess;
        }
    }
    *got = bytes;
    return malloc_without_cache(dev, p, bytes);
}

void cache_free(int dev, void *p, size_t bytes) {
    if (!p) return;
    if (bytes > kCacheBlock) {
        (void)hipFree(p);
        return;
    }
    CachedBlock out[kCacheBlocks];
    int n = 0;
    {
        std::lock_guard<std::mutex> lk(g_cache_mu);
        while (g_cache_n == kCacheBlocks || g_cache_held + bytes > kCacheBytes) out[n++] = cache_take(0);
        g_cache[g_cache_n++] = {dev, p, bytes};
        g_cache_held += bytes;
    }
    for (int i = 0; i < n; ++i) (void)hipFree(out[i].p);
}

hipError_t host_malloc(void **p, size_t bytes, unsigned flags) {
    if (injected_failure()) return hipErrorOutOfMemory;
    return hipHostMalloc(p, bytes, flags);
}

int ensure_bytes(void **ptr, size_t *cap, size_t need) {
    if (*cap >= need && *ptr) return ECC_OK;
    if (*ptr) {
        ECC_HIP(hipFree(*ptr));
        *ptr = nullptr;
        *cap = 0;
    }
    size_t sz = need < 256 ? 256 : need;
    ECC_HIP(dev_malloc((void **)ptr, sz));
    *cap = sz;
    return ECC_OK;
}

int ws_ensure(Workspace *ws, void **ptr, size_t *cap, size_t need) {
    if (!ws->fixed) return ensure_bytes(ptr, cap, need);
    if (*ptr && *cap >= need) return ECC_OK;
    set_error("fixed scratch too small: %zu bytes needed, %zu held", need, *cap);
    return ECC_E_NOMEM;
}

static std::mutex g_ws_mu;
static std::map<std::pair<int, void *>, Workspace *> g_ws;

int get_workspace(void *stream, Workspace **out) {
    int dev = 0;
    ECC_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_ws_mu);
    auto key = std::make_pair(dev, stream);
    auto it = g_ws.find(key);
    if (it == g_ws.end()) {
        Workspace *w = new Workspace();
        w->device = dev;
        w->stream = stream;
        void *p = nullptr;
        hipError_t e = dev_malloc((void **)&p, kStatusBytes);
        if (e != hipSuccess) {
            delete w;
            return hip_fail(e, "hipMalloc(status)");
        }
        w->status = (uint32_t *)p;
        void *hp = nullptr, *hd = nullptr;
        e = host_malloc((void **)&hp, 64, hipHostMallocMapped | hipHostMallocCoherent);
        if (e == hipSuccess) e = hipHostGetDevicePointer(&hd, hp, 0);
        if (e != hipSuccess) {
            if (hp) (void)hipHostFree(hp);
            (void)hipFree(p);
            delete w;
            return hip_fail(e, "hipHostMalloc(status word)");
        }
        w->host_status = (volatile uint32_t *)hp;
        w->host_status_dev = (uint32_t *)hd;
        int rc = launch_zero(p, kStatusBytes, (hipStream_t)stream);
        if (rc) {
            (void)hipHostFree(hp);
            (void)hipFree(p);
            delete w;
            return rc;
        }
        it = g_ws.emplace(key, w).first;
    }
    *out = it->second;
    return ECC_OK;
}

// Side streams of a caller's stream: the faces of a 4-D image's dual complex
// run on them, concurrently with the full box on the caller's stream (a fork
// at the call's start, a join before the faces' changes are summed).  Created
// on first use per (device, caller's stream) with the default priority,
// non-blocking, and kept for the process; each has its own workspace.
struct SideStreams {
    static constexpr int kCount = 4;
    hipStream_t s[kCount] = {};
    hipEvent_t fork = nullptr;
    hipEvent_t join[kCount] = {};
};
static std::mutex g_side_mu;
static std::map<std::pair<int, void *>, SideStreams *> g_side;

static int get_side_streams(void *stream, SideStreams **out) {
    int dev = 0;
    ECC_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_side_mu);
    auto key = std::make_pair(dev, stream);
    auto it = g_side.find(key);
    if (it == g_side.end()) {
        SideStreams *p = new SideStreams();
        hipError_t e = hipEventCreateWithFlags(&p->fork, hipEventDisableTiming);
        for (int k = 0; e == hipSuccess && k < SideStreams::kCount; ++k) {
            e = hipStreamCreateWithFlags(&p->s[k], hipStreamNonBlocking);
            if (e == hipSuccess) e = hipEventCreateWithFlags(&p->join[k], hipEventDisableTiming);
        }
        if (e != hipSuccess) {
            for (int k = 0; k < SideStreams::kCount; ++k) {
                if (p->join[k]) (void)hipEventDestroy(p->join[k]);
                if (p->s[k]) (void)hipStreamDestroy(p->s[k]);
            }
            if (p->fork) (void)hipEventDestroy(p->fork);
            delete p;
            return hip_fail(e, "side streams");
        }
        it = g_side.emplace(key, p).first;
    }
    *out = it->second;
    return ECC_OK;
}

int check_dims(const ecc_dims *dims, int64_t *total) {
    if (!dims) {
        set_error("dims is NULL");
        return ECC_E_ARG;
    }
    if (dims->ndim < 1 || dims->ndim > 4) {
        set_error("ndim %d outside 1..4", (int)dims->ndim);
        return ECC_E_ARG;
    }
    int64_t t = 1;
    for (int k = 0; k < dims->ndim; ++k) {
        if (dims->n[k] < 1) {
            set_error("n[%d] = %lld < 1", k, (long long)dims->n[k]);
            return ECC_E_ARG;
        }
        if (t > ((int64_t)1 << 62) / dims->n[k]) {
            set_error("image size overflows");
            return ECC_E_ARG;
        }
        t *= dims->n[k];
    }
    *total = t;
    return ECC_OK;
}

// Axes of length 1 are dropped: the complex of such an image is the product of
// the complex of the remaining axes with a closed unit interval, and taking
// that product changes no Euler characteristic of any threshold.
bool normalize_int_view(const ecc_dims *dims, IntView *v, int *unsupported) {
    int64_t ns[4];
    int k = 0;
    for (int i = 0; i < dims->ndim; ++i)
        if (dims->n[i] > 1) ns[k++] = dims->n[i];
    *unsupported = 0;
    if (k == 0) ns[k++] = 1;
    if (k == 1) {
        v->nin = 1; v->n0 = 1; v->n1 = 1;
        if (ns[0] > INT32_MAX) { *unsupported = 1; return false; }
        v->n2 = (int32_t)ns[0];
    } else if (k == 2) {
        v->nin = 1; v->n0 = ns[0]; v->n1 = 1;
        if (ns[1] > INT32_MAX) { *unsupported = 1; return false; }
        v->n2 = (int32_t)ns[1];
    } else if (k == 3) {
        v->nin = 2; v->n0 = ns[0];
        if (ns[1] > INT32_MAX || ns[2] > INT32_MAX || ns[1] * ns[2] > INT32_MAX) { *unsupported = 1; return false; }
        v->n1 = (int32_t)ns[1]; v->n2 = (int32_t)ns[2];
    } else {
        *unsupported = 1;
        return false;
    }
    if (v->n0 > INT32_MAX - 4) { *unsupported = 1; return false; }
    return true;
}

static int env_int(const char *name, int dflt) {
    const char *s = getenv(name);
    return (s && *s) ? atoi(s) : dflt;
}

// Tuning overrides (measurement only): ECC_INT_ROWS, ECC_INT_MODE, ECC_INT_PD, ECC_INT_WX, ECC_U16_TILES_PER_CU,
// ECC_U16_WINDOWS (1: 16-bit images in the window form),
// ECC_INT_WAVES, ECC_INT_TILES_PER_CU, ECC_INT_TILE_STRIDE, ECC_INT_PAIR (0: no row pairs),
// ECC_INT_PLAN (0: exactly the tiles per CU asked for).
// Waves along x of a plane of xs 64-column segments and ys rows of waves, at
// most cap: the fewest idle waves (whole tiles cover the plane) and wave slots
// of 16 (whole rows of waves fill a workgroup), from 4 on (narrower tiles touch
// more pages per byte); the widest of equals up to 8.  Wider than 8 where that
// leaves a seventh fewer idle.  Planes of few rows leave rows of waves idle:
// 10000 planes of 5 x 2048, three rows of waves, take 100 us at 8 bits and 118
// at 14 in workgroups of 4 x 3 waves, 125 and 168 in 8 x 2; of 9 x 2048, five
// rows of waves, 152 at 14 bits in 16 x 1, 158 in 8 x 2.
static int choose_wx(int64_t xs, int64_t ys, int cap, int max_waves) {
    const auto use = [&](int w) {
        const int64_t wy = std::min<int64_t>(ys, max_waves / w);
        const int64_t tx = (xs + w - 1) / w, ty = (ys + wy - 1) / wy;
        return (double)(xs * ys) / (double)(tx * w * ty * wy) * (double)(max_waves / w * w) / max_waves;
    };
    const int narrowest = (int)std::min<int64_t>(xs, 4);
    int best = (int)std::min<int64_t>(xs, std::min(xs <= 16 ? 16 : 8, cap));
    for (int w = best - 1; w >= narrowest; --w)
        if (use(w) > use(best) + 1e-9) best = w;
    for (int w = (int)std::min<int64_t>(xs, cap); w > 8 && xs > 16; --w)
        if (use(w) > use(best) * 1.15) best = w;
    return best;
}

// The tiling for given parameters: R rows per wave, up to wx_cap waves
// along x (16-wave workgroups), about tiles_per_cu workgroups per CU.
// planned: at most that many.  The number of workgroups is then the one with
// the least estimated time, over 1 .. tiles_per_cu per CU: the planes that the
// fullest CU walks, each walk 4 planes longer than its tile (its prologue); a
// sixth more for a workgroup that has its CU to itself; and the count rows,
// each worth row_cost planes of one workgroup (its 64 KiB are cleared, written
// and read again).  The 4 and row_cost are fitted to 248 launches of 0.5 to
// 600 million voxels (9 % off on average).  512^3 at 14 bits in 512 workgroups,
// two per CU, takes 104 us where 1024 took 149; 400 x 413 x 390 82 us where
// 1040 workgroups, most CUs idle in their last round, took 91.
IntTiling make_int_tiling(const IntView &v, int64_t planes, int rows, int tiles_per_cu, int wx_cap,
                          int max_grid = 0, bool planned = false, double row_cost = 0, bool small_bins = false) {
    IntTiling t{};
    t.rows = rows;
    t.mode = env_int("ECC_INT_MODE", 0);
    const int cus = device_cu_count();
    const int max_waves = env_int("ECC_INT_WAVES", 16);
    int64_t tiles_xy;
    if (v.nin == 1) {
        const int64_t segs = (v.n2 + (int64_t)kWave * t.rows - 1) / ((int64_t)kWave * t.rows);
        t.wx = (int)(segs < max_waves ? segs : max_waves);
        t.wy = 1;
        tiles_xy = (segs + t.wx - 1) / t.wx;
    } else {
        const int64_t xs = (v.n2 + kWave - 1) / kWave, ys = (v.n1 + t.rows - 1) / t.rows;
        auto shape = [&](int wx) {
            const int64_t wy = max_waves / wx;
            t.wx = wx;
            t.wy = (int)(ys < wy ? ys : wy);
            return ((xs + t.wx - 1) / t.wx) * ((ys + t.wy - 1) / t.wy);
        };
        tiles_xy = shape((int)(xs < wx_cap ? xs : wx_cap));
        // (fewer tiles than CUs are not made fewer still: 19 x 10 x 598 at 8
        // bits 17 us in 15 workgroups of ten waves, 20 in 12 of fifteen)
        if (planned && tiles_xy * ((planes + 7) / 8) >= cus)
            tiles_xy = shape(choose_wx(xs, ys, wx_cap, max_waves));
    }
    // The plan counts a workgroup as its CU's work.  8-bit workgroups of up to
    // four waves (planes of a few hundred voxels) run many to a CU, their 1 KiB
    // histograms beside each other, each bound by its walk's latency, so they
    // are split as finely as the rule says (300000 x 64: 50 us, planned 74;
    // 100000 x 4 x 4: 38 and 56; from seven waves on the plan is as fast), unless
    // that leaves walks of fewer than 16 planes (8000 x 64: 13.5 us, planned
    // 13.0).  At 14 bits the 64 KiB histograms admit two to a CU however small.
    if (small_bins && t.wx * t.wy <= 4 && planes * tiles_xy >= (int64_t)16 * cus * tiles_per_cu) planned = false;
    // split axis 0 until there are about tiles_per_cu tiles per CU; planes
    // with more tiles than that get several tiles per workgroup, so the
    // per-workgroup rows stay about tiles_per_cu per CU
    auto walk_for = [&](int64_t tz) {
        if (tz < 1) tz = 1;
        if (tz > planes) tz = planes;
        int64_t zc = (planes + tz - 1) / tz;
        if (zc < 8 && planes >= 8) zc = 8;
        return zc;
    };
    int64_t zc = 0, per = 0;
    auto fit = [&](int64_t target, int64_t tz) {
        const int64_t z = walk_for(tz);
        const int64_t tiles = tiles_xy * ((planes + z - 1) / z);
        int64_t p = tiles > target ? (tiles + target - 1) / target : 1;
        // a cap on the workgroups (fixed scratch): more tiles per workgroup
        if (max_grid > 0 && (tiles + p - 1) / p > max_grid) p = (tiles + max_grid - 1) / max_grid;
        const int64_t grid = (tiles + p - 1) / p;
        zc = z;
        per = p;
        t.grid = (int)grid;
        const int64_t rounds = (grid + cus - 1) / cus;
        return ((double)rounds + (rounds % 2 ? 1.0 / 6 : 0.0)) * (double)(p * (z + 4)) + row_cost * (double)grid;
    };
    if (planned) {
        double best = 0;
        int64_t best_target = 0, best_tz = 0;
        auto consider = [&](int64_t target, int64_t tz, double margin) {
            const double c = fit(target, tz);
            if (best_target == 0 || c * margin < best) {
                best = c;
                best_target = target;
                best_tz = tz;
            }
        };
        for (int k = 1; k <= tiles_per_cu; ++k) {
            const int64_t target = (int64_t)cus * k;
            for (int64_t tz = target / tiles_xy; tz <= target / tiles_xy + 1; ++tz) consider(target, tz, 1.0);
        }
        // Several shorter tiles per workgroup, where the splits above leave many
        // CUs idle: 264 tiles of a plane at one workgroup per CU make 132 of two
        // (16-bit passes over 2000 x 700 x 700: 1685 us per call, 1431 with four
        // workgroups per CU, 1003 in 235 of nine).
        if (tiles_xy * 4 > cus)
            for (int k = 1; k <= tiles_per_cu; ++k)
                for (int64_t tz = 2; tz <= 32; tz *= 2) consider((int64_t)cus * k, tz, 1.1);
        (void)fit(best_target, best_tz);
    } else {
        const int64_t target = (int64_t)cus * tiles_per_cu;
        (void)fit(target, (target + tiles_xy - 1) / tiles_xy);
    }
    t.zc = (int)zc;
    // planes of loads in flight: two on walks of 128 planes and more (1024^3:
    // 2 % faster, 512 x 4096^2: 7 %), one on shorter walks, where the longer
    // prologue costs more than it hides (14 x 8192^2: 20 % slower with two);
    // two with four rows per wave, whose register budget (one workgroup per
    // CU) holds them without spills (64-plane slabs of 14450^2: 2 % faster)
    // with one in-plane axis one (16384^2 at 14 bits: 148 us against 160)
    t.pd = env_int("ECC_INT_PD", ((zc >= 128 && v.nin == 2) || rows >= 4) ? 2 : 1);
    t.per_wg = (int)per;
    t.tile_stride = env_int("ECC_INT_TILE_STRIDE", 0);
    t.pair = env_int("ECC_INT_PAIR", 1);
    return t;
}

// Tilings chosen by ecc_autotune, per (dtype, rank, n1, n2, planes).
struct TuneKey {
    int dtype, nin;
    int32_t n1, n2;
    int64_t planes;
    bool operator<(const TuneKey &o) const {
        return std::tie(dtype, nin, n1, n2, planes) < std::tie(o.dtype, o.nin, o.n1, o.n2, o.planes);
    }
};
static std::mutex g_tune_mu;
static std::map<TuneKey, ecc_tiling> g_tuned;

static bool tuned_tiling(const IntView &v, int dtype, int64_t planes, ecc_tiling *out) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tuned.find(TuneKey{dtype, v.nin, v.n1, v.n2, planes});
    if (it == g_tuned.end()) return false;
    *out = it->second;
    return true;
}

// Launch-size rule (measured on MI355X): below 256 MiB four tiles per CU are
// fastest, above it eight.  From 4 GiB on (e.g. 62 planes of 8192^2 or of
// 14450^2) four rows per wave run at about 2.8 TB/s where two rows reach
// 2.0-2.4; below 2 GiB two rows are faster.  Likely cause: four rows keep
// half as many workgroups in flight, so fewer distinct 2 MiB pages per plane
// step need translating once a plane spans many pages.
// Between 256 MiB and 4 GiB, four tiles per CU when that gives walks of 256
// planes or more (1024^3: 512-plane walks, the same kernel time as eight
// tiles per CU and half the count rows to merge: 0.770 vs 0.781 ms per
// curve), else eight (62 x 4096^2: 0.735 vs 0.831 ms).
static ecc_tiling rule_tiling(const IntView &v, int dtype, int64_t planes) {
    const int64_t launch_bytes = planes * (int64_t)v.n1 * v.n2 * (dtype == ECC_U8 ? 1 : 2);
    ecc_tiling c{};
    c.rows = launch_bytes >= ((int64_t)4 << 30) ? 4 : 2;
    // four rows: workgroups two waves tall (64-plane slabs of 14450^2: 2 %
    // faster than one row of 16 waves)
    c.waves_x = c.rows == 4 ? 8 : 16;
    if (launch_bytes < ((int64_t)256 << 20)) c.tiles_per_cu = 4;
    else if (c.rows == 4) c.tiles_per_cu = 16;
    else c.tiles_per_cu = make_int_tiling(v, planes, c.rows, 4, c.waves_x).zc >= 256 ? 4 : 8;
    return c;
}

// Parameters: ECC_INT_* environment overrides (measurement), else a tiling
// ecc_autotune stored for this shape, else the launch-size rule.
static ecc_tiling tiling_params(const IntView &v, int dtype, int64_t planes) {
    ecc_tiling c{};
    if (!tuned_tiling(v, dtype, planes, &c)) c = rule_tiling(v, dtype, planes);
    c.rows = env_int("ECC_INT_ROWS", c.rows);
    c.tiles_per_cu = env_int("ECC_INT_TILES_PER_CU", c.tiles_per_cu);
    c.waves_x = env_int("ECC_INT_WX", c.waves_x);
    return c;
}

// Whether a launch's workgroups are planned (make_int_tiling): by the rule's
// parameters, 14-bit launches below 2^30 voxels, 8-bit ones below 2^27.  Above
// that, finer splits than the plan's were as fast or faster (1024^3 at 14 bits:
// 649 us in 1024 workgroups, 658 in 512; 128 x 1024^2 at 8 bits: 102 us against
// 104).  Other parameters (a tuned or loaded tiling, ECC_INT_*) are taken as
// they are: they were timed so.
static bool planned_tiling(const IntView &v, int dtype, int64_t planes, const ecc_tiling &c) {
    if (planes * (int64_t)v.n1 * v.n2 >= (int64_t)1 << (dtype == ECC_U8 ? 27 : 30) || env_int("ECC_INT_PLAN", 1) == 0)
        return false;
    const ecc_tiling r = rule_tiling(v, dtype, planes);
    return c.rows == r.rows && c.tiles_per_cu == r.tiles_per_cu && c.waves_x == r.waves_x;
}
static IntTiling tiling_from(const IntView &v, int dtype, int64_t planes, const ecc_tiling &c, int max_grid) {
    const bool planned = planned_tiling(v, dtype, planes, c);
    return make_int_tiling(v, planes, c.rows, c.tiles_per_cu, c.waves_x, max_grid, planned,
                           dtype == ECC_U8 ? 0.0075 : 0.045, dtype == ECC_U8);
}

IntTiling choose_int_tiling(const IntView &v, int dtype, int64_t planes, int max_grid) {
    return tiling_from(v, dtype, planes, tiling_params(v, dtype, planes), max_grid);
}

// Enqueue the whole integer computation for a device-resident image.
static int enqueue_int(const void *image_dev, const IntView &v, int dtype, int64_t *chi_dev,
                       uint32_t *status_out, hipStream_t stream, Workspace *ws, bool max_entry = false) {
    const int m = (int)threshold_count(dtype);
    const size_t eb = elem_bytes(dtype);
    IntTiling tl = choose_int_tiling(v, dtype, v.n0, ws->max_grid);
    int rc = ws_ensure(ws, (void **)&ws->partial, &ws->partial_bytes, (size_t)tl.grid * m * sizeof(int32_t));
    if (rc) return rc;
    rc = ws_ensure(ws, (void **)&ws->vcec, &ws->vcec_bytes, (size_t)m * sizeof(int64_t));
    if (rc) return rc;
    IntJob job{};
    job.src.base = (const uint8_t *)image_dev;
    job.src.lo_base = job.src.base;
    job.src.plane_bytes = (int64_t)v.n1 * v.n2 * (int64_t)eb;
    job.view = v;
    job.e0 = 0;
    job.e1 = (int32_t)v.n0;
    job.lo_inf = 1;
    job.hi_inf = 1;
    job.dtype = dtype;
    job.invert = max_entry ? 1 : 0;
    rc = launch_int_partial(job, tl, ws->partial, ws->status, nullptr, stream);
    if (rc) return rc;
    return launch_merge(ws->partial, tl.grid, m, ws->vcec, false, true, chi_dev, ws->status, status_out,
                        stream, max_entry);
}

// 16-bit images (m = 65536): the workgroup histograms hold 16384 bins, so
// one launch counts one window of values.  The kernel reads
// bin = clamp(v - shift, 0, 16383); bins [klo, khi] are values
// [shift + klo, shift + khi].  A window needs a guard bin only on a side
// where the image has values outside it: bin 0 when values below exist
// (klo = 1), bin 16383 when values above exist (khi = 16382).  The guard
// bins are dropped; the monotone clamp keeps every comparison that decides a
// kept bin (each involves the counted value itself).  Each pass's column
// sums go to their place in the 65536-bin changes vector, scanned once.
int plan_u16_windows(uint32_t vmin, uint32_t vmax, U16Window *w) {
    int n = 0;
    int64_t v = vmin;
    while (v <= (int64_t)vmax) {
        U16Window x;
        x.klo = v > (int64_t)vmin ? 1 : 0;
        x.shift = (int32_t)(v - x.klo);
        x.khi = (int64_t)x.shift + 16383 >= (int64_t)vmax ? (int)((int64_t)vmax - x.shift) : 16382;
        w[n++] = x;
        v = (int64_t)x.shift + x.khi + 1;
    }
    return n;
}

// Tiling of a 32768-bin pass: two rows per wave, two planes of look-ahead,
// one workgroup per CU (the 128 KiB histogram admits one at a time, and each
// further one writes another row of 128 KiB to be summed: 463 x 512^2, two
// passes: 278 us in all, 305 with two per CU, 357 with four).
IntTiling range_pass_tiling(const IntView &v, int64_t planes) {
    IntTiling tl = make_int_tiling(v, planes, 2, env_int("ECC_U16_TILES_PER_CU", 1), 16, 0, true);
    tl.pd = 2;
    tl.mode = 0;
    return tl;
}

// 16-bit images in 32768-bin passes (a 128 KiB workgroup histogram, one
// workgroup per CU): the fields and comparisons take the raw values and each
// pass adds the changes at values [lo, lo + 32768) exactly, with no guard
// bins: [0, 32768), then [32768, 65536), each skipping the adds of values
// outside its half.  Each pass's column sums go to their half of the
// 65536-bin changes vector, scanned once.
// The synchronous call (adaptive) lets the first pass note whether any value
// lies above its half (a word of host memory, read after the pass), and runs
// the second only then.  No separate read for the image's range: images
// below 32768 take one pass (1024^3 14-bit and 15-bit data: 0.92 ms, against
// 1.15 and 2.54 ms for the range read and one or two windows), full ranges
// two (1.80 ms, against 3.94 ms in five windows); an image whose values all
// lie above 32768 reads it once in vain.  The other calls run both.
static int enqueue_u16_passes(const void *image_dev, const IntView &v, int64_t *chi_dev, uint32_t *status_out,
                              hipStream_t stream, Workspace *ws, bool adaptive) {
    constexpr int mpass = 32768, mtot = 65536;
    const IntTiling tl = range_pass_tiling(v, v.n0);
    int rc = ensure_bytes((void **)&ws->partial, &ws->partial_bytes, (size_t)tl.grid * mpass * sizeof(int32_t));
    if (rc) return rc;
    rc = ensure_bytes((void **)&ws->vcec16, &ws->vcec16_bytes, (size_t)mtot * sizeof(int64_t));
    if (rc) return rc;
    volatile uint32_t *high = ws->host_status + 1;
    if (adaptive) *high = 0u;
    IntJob job{};
    job.src.base = (const uint8_t *)image_dev;
    job.src.lo_base = job.src.base;
    job.src.plane_bytes = (int64_t)v.n1 * v.n2 * 2;
    job.view = v;
    job.e0 = 0;
    job.e1 = (int32_t)v.n0;
    job.lo_inf = 1;
    job.hi_inf = 1;
    job.dtype = ECC_U16;
    job.range_pass = 2;
    for (int i = 0; i < 2; ++i) {
        job.win_shift = i * mpass;
        job.high_flag = adaptive && i == 0 ? ws->host_status_dev + 1 : nullptr;
        rc = launch_int_partial(job, tl, ws->partial, ws->status, nullptr, stream);
        if (rc) return rc;
        rc = launch_merge_half(ws->partial, tl.grid, ws->vcec16, i, adaptive && i == 0, ws->status, stream);
        if (rc) return rc;
        if (adaptive && i == 0) {
            ECC_HIP(hipStreamSynchronize(stream));
            if (*high == 0u) break;
        }
    }
    return launch_scan_halves(ws->vcec16, chi_dev, ws->status, status_out, stream);
}

// Planned from a known range (the entry point that allocates nothing, whose
// fixed scratch holds count rows of 16384 bins, and the asynchronous calls,
// which plan for 0..65535): values that fit one window take the window form
// (16384-bin passes, eight waves per SIMD; 1024^3: 1.15 ms against 1.25 ms in
// a 32768-bin pass), wider ranges the 32768-bin passes (full range: 2.2 ms
// against 4.0 ms in five windows).
static int enqueue_u16(const void *image_dev, const IntView &v, int64_t *chi_dev, uint32_t *status_out,
                       hipStream_t stream, Workspace *ws, uint32_t vmin, uint32_t vmax) {
    constexpr int mloc = 16384, mtot = 65536;
    U16Window win[kU16MaxWindows + 1];
    const int nwin = plan_u16_windows(vmin, vmax, win);
    if (nwin > 1 && !ws->fixed && env_int("ECC_U16_WINDOWS", 0) == 0)
        return enqueue_u16_passes(image_dev, v, chi_dev, status_out, stream, ws, false);
    IntTiling tl = choose_int_tiling(v, ECC_U16, v.n0, ws->max_grid);
    int rc = ws_ensure(ws, (void **)&ws->partial, &ws->partial_bytes, (size_t)tl.grid * mloc * sizeof(int32_t));
    if (rc) return rc;
    rc = ws_ensure(ws, (void **)&ws->vcec, &ws->vcec_bytes, (size_t)mloc * sizeof(int64_t));
    if (rc) return rc;
    rc = ws_ensure(ws, (void **)&ws->vcec16, &ws->vcec16_bytes, (size_t)mtot * sizeof(int64_t));
    if (rc) return rc;
    rc = launch_zero(ws->vcec16, (size_t)mtot * sizeof(int64_t), stream);
    if (rc) return rc;
    IntJob job{};
    job.src.base = (const uint8_t *)image_dev;
    job.src.lo_base = job.src.base;
    job.src.plane_bytes = (int64_t)v.n1 * v.n2 * 2;
    job.view = v;
    job.e0 = 0;
    job.e1 = (int32_t)v.n0;
    job.lo_inf = 1;
    job.hi_inf = 1;
    job.dtype = ECC_U16;
    for (int i = 0; i < nwin; ++i) {
        job.win_shift = win[i].shift;
        rc = launch_int_partial(job, tl, ws->partial, ws->status, nullptr, stream);
        if (rc) return rc;
        rc = launch_merge(ws->partial, tl.grid, mloc, ws->vcec, false, false, nullptr, ws->status,
                          nullptr, stream);
        if (rc) return rc;
        ECC_HIP(hipMemcpyAsync(ws->vcec16 + win[i].shift + win[i].klo, ws->vcec + win[i].klo,
                               (size_t)(win[i].khi - win[i].klo + 1) * sizeof(int64_t), hipMemcpyDeviceToDevice,
                               stream));
    }
    return launch_merge(nullptr, 0, mtot, ws->vcec16, true, true, chi_dev, ws->status, status_out, stream);
}

int u16_curve_async(const void *image_dev, const IntView &v, int64_t *chi_dev, uint32_t *status_out,
                    hipStream_t stream) {
    Workspace *ws = nullptr;
    int rc = get_workspace(stream, &ws);
    if (rc) return rc;
    return enqueue_u16(image_dev, v, chi_dev, status_out, stream, ws, 0, 65535);
}

// Count rows only (no merge) of a device image in the largest-value convention
// (entries at m-1-v) into ws->partial, with room for extra_rows more behind
// the *rows written; a range error stays set in ws->status for a later scan to
// report.
static int enqueue_max_entry_rows(const void *image_dev, const IntView &v, int dtype, int extra_rows, int *rows,
                                  hipStream_t stream, Workspace *ws) {
    const int m = (int)threshold_count(dtype);
    IntTiling tl = choose_int_tiling(v, dtype, v.n0);
    int rc = ensure_bytes((void **)&ws->partial, &ws->partial_bytes,
                          (size_t)(tl.grid + extra_rows) * m * sizeof(int32_t));
    if (rc) return rc;
    *rows = tl.grid;
    IntJob job{};
    job.src.base = (const uint8_t *)image_dev;
    job.src.lo_base = job.src.base;
    job.src.plane_bytes = (int64_t)v.n1 * v.n2 * (int64_t)elem_bytes(dtype);
    job.view = v;
    job.e0 = 0;
    job.e1 = (int32_t)v.n0;
    job.lo_inf = 1;
    job.hi_inf = 1;
    job.dtype = dtype;
    job.invert = 1;
    return launch_int_partial(job, tl, ws->partial, ws->status, nullptr, stream);
}

static bool is_device_ptr(const void *p) {
    hipPointerAttribute_t attr;
    memset(&attr, 0, sizeof attr);
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return attr.type == hipMemoryTypeDevice || attr.type == hipMemoryTypeManaged;
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Integer images with four axes longer than 1 (the integer kernel takes at
// most two in-plane axes): every voxel's change from the change kernel
// (ecc_change.hip).  The image's planes along its first longer axis.
static int four_d_job(const void *img_dev, const ecc_dims *dims, int64_t total, int dtype, bool max_entry,
                      ChangeJob *job) {
    if (total * 4 > (int64_t)UINT32_MAX) {
        set_error("integer images with four axes longer than 1 are limited to 2^30 elements");
        return ECC_E_UNSUPPORTED;
    }
    int64_t n[4];
    int d = 0;
    for (int i = 0; i < dims->ndim; ++i)
        if (dims->n[i] > 1) n[d++] = dims->n[i];
    if (d != 4) {
        set_error("integer path: shape not supported (an extent beyond 2^31)");
        return ECC_E_UNSUPPORTED;
    }
    *job = ChangeJob{};
    job->dtype = dtype;
    job->nl = 2;
    job->nx = (int32_t)n[3];
    job->ny = (int32_t)n[2];
    job->nz = (int32_t)n[1];
    job->src.base = job->src.lo_base = (const uint8_t *)img_dev;
    job->src.plane_bytes = n[1] * n[2] * n[3] * (int64_t)elem_bytes(dtype);
    job->e1 = (int32_t)n[0];
    job->lo_inf = job->hi_inf = 1;
    job->invert = max_entry ? 1 : 0;
    return ECC_OK;
}

// The curve of such an image into chi_dev, or, with changes_out, only its
// changes vector there (a range error then stays set in ws->status for a
// later scan to report).  max_entry: counted at m-1-v and merged reversed, as
// in three dimensions.
static int enqueue_four_d(const ChangeJob &job, bool max_entry, int64_t *chi_dev, int64_t *changes_out,
                          uint32_t *status_out, hipStream_t s, Workspace *ws) {
    const int m = (int)threshold_count(job.dtype);
    int rows = 0;
    int rc = change_count_rows(job, &rows);
    if (rc) return rc;
    rc = ensure_bytes((void **)&ws->partial, &ws->partial_bytes, (size_t)rows * m * sizeof(int32_t));
    if (rc) return rc;
    rc = ensure_bytes((void **)&ws->vcec, &ws->vcec_bytes, (size_t)m * sizeof(int64_t));
    if (rc) return rc;
    rc = launch_change_counts(job, ws->partial, ws->status, s);
    if (rc) return rc;
    if (changes_out)
        return launch_merge(ws->partial, rows, m, changes_out, false, false, nullptr, ws->status, nullptr, s,
                            max_entry);
    return launch_merge(ws->partial, rows, m, ws->vcec, false, true, chi_dev, ws->status, status_out, s,
                        max_entry);
}

// Synchronous integer curve: host or device image and curve.  max_entry:
// each cell's value is the maximum over its voxels (the kernel reads M-1-v
// and the merge writes the rows reversed).
// With `bins`, image is a float image, quantised into the workspace first: a
// NaN sets its bit in the status word, the scan then writes nothing and
// reports it (no wait between the two: 1537 x 2048 to 8 bits takes 34 us per
// curve, 60 with the flag of its own that the host read first).
struct Quantizer {
    float lo, scale;
};
static int compute_int(const void *image, const ecc_dims *dims, int64_t total, ecc_dtype dtype, ecc_curve *curve,
                       hipStream_t s, bool max_entry, const Quantizer *bins = nullptr) {
    if (dtype == ECC_U16 && max_entry) {
        set_error("the largest-value convention is available for u8 and u14");
        return ECC_E_UNSUPPORTED;
    }
    const int64_t m = threshold_count(dtype);
    if (m < 0) {
        set_error("unknown dtype %d", (int)dtype);
        return ECC_E_ARG;
    }
    if (curve->capacity < m) {
        curve->count = m;
        set_error("curve capacity %lld < %lld", (long long)curve->capacity, (long long)m);
        return ECC_E_BUFFER_TOO_SMALL;
    }
    IntView v{};
    ChangeJob four{};
    int unsup = 0;
    const bool four_d = !normalize_int_view(dims, &v, &unsup);
    if (four_d) {
        int rc = four_d_job(nullptr, dims, total, dtype, max_entry, &four);
        if (rc) return rc;
    }
    Workspace *ws = nullptr;
    int rc = get_workspace(s, &ws);
    if (rc) return rc;
    const void *img_dev = image;
    const size_t up_bytes = is_device_ptr(image) ? 0 : (size_t)total * (bins ? 4 : elem_bytes(dtype));
    const size_t qoff = align256(up_bytes);  // the image's copy, then its bins
    if (up_bytes || bins) {
        rc = ensure_bytes(&ws->img_tmp, &ws->img_tmp_bytes, bins ? qoff + (size_t)total * elem_bytes(dtype) : up_bytes);
        if (rc) return rc;
    }
    if (up_bytes) {
        ECC_HIP(hipMemcpyAsync(ws->img_tmp, image, up_bytes, hipMemcpyHostToDevice, s));
        img_dev = ws->img_tmp;
    }
    const bool chi_dev = is_device_ptr(curve->chi);
    int64_t *chi_target = curve->chi;
    if (!chi_dev) {
        rc = ensure_bytes((void **)&ws->chi_tmp, &ws->chi_tmp_bytes, (size_t)m * sizeof(int64_t));
        if (rc) return rc;
        chi_target = ws->chi_tmp;
    }
    if (bins) {
        void *q = (uint8_t *)ws->img_tmp + qoff;
        rc = launch_quantize((const float *)img_dev, total, bins->lo, bins->scale, (int)m, (int)elem_bytes(dtype), q,
                             ws->status, s);
        if (rc) return rc;
        img_dev = q;
    }
    if (four_d) {
        four.src.base = four.src.lo_base = (const uint8_t *)img_dev;
        *ws->host_status = 0xFFFFFFFFu;  // overwritten by the scan
        rc = enqueue_four_d(four, max_entry, chi_target, nullptr, ws->host_status_dev, s, ws);
    } else if (dtype == ECC_U16 && !ws->fixed && env_int("ECC_U16_WINDOWS", 0) == 0) {
        *ws->host_status = 0xFFFFFFFFu;  // overwritten by the scan
        rc = enqueue_u16_passes(img_dev, v, chi_target, ws->host_status_dev, s, ws, true);
    } else if (dtype == ECC_U16) {  // only the windows between the image's minimum and maximum
        uint32_t *mm = ws->status + kStatusMinMaxOffset / 4;
        rc = launch_minmax_u16((const uint16_t *)img_dev, total, mm, s);
        if (rc) return rc;
        uint32_t range[2] = {0, 0};
        ECC_HIP(hipMemcpyAsync(range, mm, sizeof range, hipMemcpyDeviceToHost, s));
        ECC_HIP(hipStreamSynchronize(s));
        *ws->host_status = 0xFFFFFFFFu;  // overwritten by the scan
        rc = enqueue_u16(img_dev, v, chi_target, ws->host_status_dev, s, ws, range[0], range[1]);
    } else {
        *ws->host_status = 0xFFFFFFFFu;
        rc = enqueue_int(img_dev, v, dtype, chi_target, ws->host_status_dev, s, ws, max_entry);
    }
    if (rc) {
        if (bins) (void)launch_zero(ws->status, 4, s);  // (no scan may follow that clears the NaN bit)
        (void)hipStreamSynchronize(s);                  // the scan may still write the host word
        return rc;
    }
    ECC_HIP(hipStreamSynchronize(s));
    const uint32_t st = *ws->host_status;
    if (st == 0xFFFFFFFFu) {
        set_error("internal error: the scan did not report a status");
        return ECC_E_HIP;
    }
    if (bins && (st & kStatusNaN)) {
        set_error("a float image holds a NaN");
        return ECC_E_NAN;
    }
    if (st & kStatusRange) {
        set_error("a 14-bit image holds a value >= 16384");
        return ECC_E_RANGE;
    }
    if (st != 0) {
        set_error("internal error: device status 0x%08x", st);
        return ECC_E_HIP;
    }
    if (!chi_dev) {
        ECC_HIP(hipMemcpyAsync(curve->chi, ws->chi_tmp, (size_t)m * sizeof(int64_t), hipMemcpyDeviceToHost, s));
        ECC_HIP(hipStreamSynchronize(s));
    }
    curve->count = m;
    return ECC_OK;
}

// A call that gives up after its kernels were launched: the status word that
// they may have set (a NaN) is cleared, so that the next call on the stream does
// not report it, and they are waited for, since the caller may free the image.
struct StatusCleanup {
    Workspace *ws;
    hipStream_t s;
    bool armed = false;
    ~StatusCleanup() {
        if (!armed) return;
        (void)launch_zero(ws->status, 4, s);
        (void)hipStreamSynchronize(s);
    }
};

// steps_only: the output keeps the keys where chi changes (chi = 0 before
// the first key), compacted after the full curve is built.
static int compute_float(const void *image, const ecc_dims *dims, int64_t n, ecc_curve *curve, hipStream_t s,
                         bool steps_only) {
    if (!curve->keys) {
        set_error("ECC_F32 needs curve->keys");
        return ECC_E_ARG;
    }
    Workspace *ws = nullptr;
    int rc = get_workspace(s, &ws);
    if (rc) return rc;
    const float *img_dev = (const float *)image;
    if (!is_device_ptr(image)) {
        const size_t bytes = (size_t)n * 4;
        rc = ensure_bytes(&ws->img_tmp, &ws->img_tmp_bytes, bytes);
        if (rc) return rc;
        ECC_HIP(hipMemcpyAsync(ws->img_tmp, image, bytes, hipMemcpyHostToDevice, s));
        img_dev = (const float *)ws->img_tmp;
    }
    // carve the float scratch: two key buffers (sort), the record regions
    // (after the records are compacted, the change-point output's chi), the
    // region counts and offsets, the split's first slots and head, the digit
    // table and its scan sums, the curve's tile sums, the counts
    ChangeJob job{};
    rc = float_job(img_dev, dims, &job);
    if (rc) return rc;
    int64_t regions = 0, region_slots = 0;
    rc = change_regions(job, &regions, &region_slots);
    if (rc) return rc;
    // (the change points' chi goes to the regions once the records are compacted)
    const int64_t slots = std::max(regions * region_slots, steps_only ? n : 0);
    const int64_t digit_entries = std::max(radix_count_entries(n, 4), radix_count_entries(n, 8));
    const int64_t ft = float_tiles(n);
    enum { kKey0, kKey1, kNz, kNzCnt, kNzOff, kStarts, kHead, kCounts, kSums, kTileA, kTileB, kBound, kCnt, kSteps, kNbuf };
    size_t off[kNbuf], total = 0;
    const int64_t scan_entries = std::max(std::max(digit_entries, regions + 1), steps_only ? n : 0);
    const size_t sz[kNbuf] = {(size_t)n * 4, (size_t)n * 4, (size_t)slots * 8, (size_t)regions * 4,
                              (size_t)(regions + 1) * 4,
                              (size_t)((n + kSplitTile - 1) / kSplitTile * kSplitBuckets) * 2, split_head_bytes(n),
                              (size_t)digit_entries * 4,
                              (size_t)radix_scan_tiles(scan_entries) * 4, (size_t)ft * 8, (size_t)ft * 8,
                              (size_t)(ft + 1) * 8, 64,
                              steps_only ? (size_t)n * 4 : 0};
    for (int i = 0; i < kNbuf; ++i) {
        off[i] = total;
        total += align256(sz[i]);
    }
    // curve staging unless the caller's buffers are device memory that holds
    // any possible count (n entries)
    const bool direct = !steps_only && curve->capacity >= n && is_device_ptr(curve->chi) &&
                        is_device_ptr(curve->keys);
    const size_t out_k = total, out_c = out_k + align256((size_t)n * 4);
    if (!direct) total = out_c + align256((size_t)n * 8);
    rc = ensure_bytes(&ws->fbuf, &ws->fbuf_bytes, total);
    if (rc) return rc;
    uint8_t *b = (uint8_t *)ws->fbuf;
    uint32_t *key[2] = {(uint32_t *)(b + off[kKey0]), (uint32_t *)(b + off[kKey1])};
    uint64_t *nz = (uint64_t *)(b + off[kNz]);
    uint32_t *nz_cnt = (uint32_t *)(b + off[kNzCnt]);
    uint32_t *nz_off = (uint32_t *)(b + off[kNzOff]);
    uint32_t *counts = (uint32_t *)(b + off[kCounts]);
    uint32_t *sums = (uint32_t *)(b + off[kSums]);
    int64_t *tile_a = (int64_t *)(b + off[kTileA]);
    int64_t *tile_b = (int64_t *)(b + off[kTileB]);
    int64_t *bound = (int64_t *)(b + off[kBound]);
    int64_t *count_dev = (int64_t *)(b + off[kCnt] + 8);
    int64_t *count2_dev = (int64_t *)(b + off[kCnt] + 16);
    uint16_t *starts = (uint16_t *)(b + off[kStarts]);
    uint32_t *head = (uint32_t *)(b + off[kHead]);
    float *out_keys = direct ? curve->keys : (float *)(b + out_k);
    int64_t *out_chi = direct ? curve->chi : (int64_t *)(b + out_c);
    // the host reads which top bytes occur while the change kernel runs
    hipEvent_t ev = nullptr;
    ECC_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    StatusCleanup cleanup{ws, s, true};
    rc = launch_split(img_dev, n, key[0], starts, head, ws->host_status_dev + 4, ws->status, ev, s);
    if (!rc) rc = launch_change_records(job, nz, nz_cnt, s);
    hipError_t e = hipEventSynchronize(ev);
    int present = 0;
    for (int w = 0; w < 8; ++w) present += __builtin_popcount((ws->host_status + 4)[w]);
    bool by_bits = !rc && e == hipSuccess && present <= kMaxDistinctBytes;
    if (by_bits) {
        rc = ensure_bytes(&ws->fbits, &ws->fbits_bytes, distinct_scratch_bytes(present, n));
        if (rc == ECC_E_NOMEM) {  // the sort's buffers are there, and its records' are as small as the image
            g_err_clear();
            rc = ECC_OK;
            by_bits = false;
        } else if (rc) {
            (void)hipEventDestroy(ev);
            return rc;
        }
    }
    if (by_bits) {
        (void)hipEventDestroy(ev);
        rc = launch_distinct_curve(n, present, key[0], starts, head, ws->fbits, nz, nz_cnt, regions, region_slots,
                                   out_keys, out_chi, count_dev, (int64_t *)(ws->host_status_dev + 12), ws->status,
                                   ws->host_status_dev + 14, s);
        if (rc) return rc;
    } else {
        // the record count, read on the host while the keys are sorted: a
        // word of the host-mapped status block
        volatile int64_t *nnz_host = (volatile int64_t *)(ws->host_status + 2);
        *nnz_host = -1;
        if (!rc && e == hipSuccess) {
            rc = launch_nz_total(nz_cnt, nz_off, regions, sums, (int64_t *)(ws->host_status_dev + 2), s);
            if (!rc) e = hipEventRecord(ev, s);
            if (!rc && e == hipSuccess) {
                rc = radix_sort_keys(key, n, starts, counts, sums, s);
                e = hipEventSynchronize(ev);
            }
        }
        (void)hipEventDestroy(ev);
        ECC_HIP(e);
        if (rc) return rc;
        const int64_t nnz = *nnz_host;
        if (nnz < 0 || nnz > n) {
            set_error("internal error: %lld change records for %lld voxels", (long long)nnz, (long long)n);
            return ECC_E_HIP;
        }
        // the dense records (two sort buffers) and their prefix
        const size_t rb = align256((size_t)nnz * 8);
        rc = ensure_bytes(&ws->frec, &ws->frec_bytes, 3 * rb + 256);
        if (rc) return rc;
        uint64_t *rec[2] = {(uint64_t *)ws->frec, (uint64_t *)((uint8_t *)ws->frec + rb)};
        int64_t *prefix = (int64_t *)((uint8_t *)ws->frec + 2 * rb);
        if (nnz > 0) {
            rc = launch_nz_compact(nz, nz_cnt, nz_off, regions, region_slots, rec[0], s);
            if (rc) return rc;
            rc = radix_sort_records(rec, nnz, counts, sums, s);
            if (rc) return rc;
        }
        rc = launch_float_curve(key[0], n, rec[0], nnz, prefix, (uint32_t *)tile_b, sums, tile_a, bound, count_dev,
                                out_keys, out_chi, s);
        if (rc) return rc;
    }
    uint32_t st = 0;
    int64_t kcount = 0;
    if (by_bits) {
        ECC_HIP(hipStreamSynchronize(s));
        st = ws->host_status[14];
        kcount = *(volatile int64_t *)(ws->host_status + 12);
    } else {
        ECC_HIP(hipMemcpyAsync(&st, ws->status, 4, hipMemcpyDeviceToHost, s));
        ECC_HIP(hipMemcpyAsync(&kcount, count_dev, 8, hipMemcpyDeviceToHost, s));
        ECC_HIP(hipStreamSynchronize(s));
    }
    if (st != 0) {
        if (st & kStatusNaN) {
            set_error("a float image holds a NaN");
            return ECC_E_NAN;
        }
        set_error("internal error: device status 0x%08x", st);
        return ECC_E_HIP;
    }
    cleanup.armed = false;  // (the status word is clear, the image is read)
    if (steps_only) {  // compact into buffers free after the curve: the second key buffer, the regions
        float *step_keys = (float *)key[1];
        int64_t *step_chi = (int64_t *)nz;
        rc = launch_change_points(out_keys, out_chi, kcount, (uint32_t *)(b + off[kSteps]), sums, step_keys,
                                  step_chi, count2_dev, s);
        if (rc) return rc;
        ECC_HIP(hipMemcpyAsync(&kcount, count2_dev, 8, hipMemcpyDeviceToHost, s));
        ECC_HIP(hipStreamSynchronize(s));
        out_keys = step_keys;
        out_chi = step_chi;
    }
    if (kcount > curve->capacity) {
        curve->count = kcount;
        set_error("curve capacity %lld < %lld output entries", (long long)curve->capacity, (long long)kcount);
        return ECC_E_BUFFER_TOO_SMALL;
    }
    if (!direct) {
        ECC_HIP(hipMemcpyAsync(curve->keys, out_keys, (size_t)kcount * 4, hipMemcpyDefault, s));
        ECC_HIP(hipMemcpyAsync(curve->chi, out_chi, (size_t)kcount * 8, hipMemcpyDefault, s));
        ECC_HIP(hipStreamSynchronize(s));
    }
    curve->count = kcount;
    return ECC_OK;
}

// ws == nullptr: the per-(device, stream) workspace.
int compute_async_ws(const void *image_dev, const ecc_dims *dims, ecc_dtype dtype, int64_t *chi_dev,
                     uint32_t *status_dev, hipStream_t stream, Workspace *ws) {
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image_dev || !chi_dev) {
        set_error("NULL image or chi");
        return ECC_E_ARG;
    }
    if (dtype != ECC_U8 && dtype != ECC_U14 && dtype != ECC_U16) {
        if (dtype == ECC_F32) {
            set_error("ecc_compute_async: dtype %d not available in this library", (int)dtype);
            return ECC_E_UNSUPPORTED;
        }
        set_error("unknown dtype %d", (int)dtype);
        return ECC_E_ARG;
    }
    IntView v{};
    int unsup = 0;
    if (!normalize_int_view(dims, &v, &unsup)) {
        set_error("integer path: shape not supported (4 axes longer than 1, or an extent beyond 2^31)");
        return ECC_E_UNSUPPORTED;
    }
    if (!ws) {
        rc = get_workspace(stream, &ws);
        if (rc) return rc;
    }
    if (dtype == ECC_U16)  // stream-ordered: planned for all values (no host read of the value range)
        return enqueue_u16(image_dev, v, chi_dev, status_dev, stream, ws, 0, 65535);
    return enqueue_int(image_dev, v, dtype, chi_dev, status_dev, stream, ws);
}

}  // namespace ecc

using namespace ecc;

extern "C" {

const char *ecc_last_error(void) { return g_err; }

const char *ecc_version(void) { return "libecc 0.1 (gfx950)"; }

int ecc_threshold_count(ecc_dtype dtype, int64_t *m_out) {
    const int64_t m = threshold_count(dtype);
    if (m < 0 || !m_out) {
        set_error("not an integer dtype or NULL output");
        return ECC_E_ARG;
    }
    *m_out = m;
    return ECC_OK;
}

int ecc_compute_async(const void *image_dev, const ecc_dims *dims, ecc_dtype dtype, int64_t *chi_dev,
                      uint32_t *status_dev, void *stream) {
    g_err[0] = 0;
    return compute_async_ws(image_dev, dims, dtype, chi_dev, status_dev, (hipStream_t)stream, nullptr);
}

int ecc_compute(const void *image, const ecc_dims *dims, ecc_dtype dtype, ecc_curve *curve, void *stream) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image || !curve || !curve->chi) {
        set_error("NULL image, curve or curve->chi");
        return ECC_E_ARG;
    }
    if (dtype == ECC_F32) return compute_float(image, dims, total, curve, (hipStream_t)stream, false);
    return compute_int(image, dims, total, dtype, curve, (hipStream_t)stream, false);
}

int ecc_compute_max_entry(const void *image, const ecc_dims *dims, ecc_dtype dtype, ecc_curve *curve,
                          void *stream) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image || !curve || !curve->chi) {
        set_error("NULL image, curve or curve->chi");
        return ECC_E_ARG;
    }
    if (dtype == ECC_F32) {
        set_error("ecc_compute_max_entry: integer dtypes only");
        return ECC_E_UNSUPPORTED;
    }
    return compute_int(image, dims, total, dtype, curve, (hipStream_t)stream, true);
}

int ecc_compute_change_points(const void *image, const ecc_dims *dims, ecc_dtype dtype, ecc_curve *curve,
                              void *stream) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image || !curve || !curve->chi) {
        set_error("NULL image, curve or curve->chi");
        return ECC_E_ARG;
    }
    if (dtype != ECC_F32) {
        set_error("ecc_compute_change_points: ECC_F32 only");
        return dtype >= ECC_U8 && dtype <= ECC_U16 ? ECC_E_UNSUPPORTED : ECC_E_ARG;
    }
    return compute_float(image, dims, total, curve, (hipStream_t)stream, true);
}

int ecc_compute_quantized(const float *image, const ecc_dims *dims, float lo, float hi, ecc_dtype bins,
                          ecc_curve *curve, void *stream) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image || !curve || !curve->chi) {
        set_error("NULL image, curve or curve->chi");
        return ECC_E_ARG;
    }
    if (bins != ECC_U8 && bins != ECC_U14 && bins != ECC_U16) {
        set_error("ecc_compute_quantized: bins must be ECC_U8, ECC_U14 or ECC_U16");
        return ECC_E_ARG;
    }
    const float width = hi - lo;
    if (!(width > 0.0f) || !(width <= 3.0e38f)) {
        set_error("ecc_compute_quantized: need lo < hi, both finite");
        return ECC_E_ARG;
    }
    const int64_t m = threshold_count(bins);
    if (curve->capacity < m) {
        curve->count = m;
        set_error("curve capacity %lld < %lld", (long long)curve->capacity, (long long)m);
        return ECC_E_BUFFER_TOO_SMALL;
    }
    const Quantizer q{lo, (float)m / width};
    return compute_int(image, dims, total, bins, curve, (hipStream_t)stream, false, &q);
}

int ecc_autotune(const void *image_dev, const ecc_dims *dims, ecc_dtype dtype, void *stream, ecc_tiling *best) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image_dev || !best) {
        set_error("NULL image or output");
        return ECC_E_ARG;
    }
    if (dtype != ECC_U8 && dtype != ECC_U14) {
        set_error("ecc_autotune: U8 or U14 images");
        return (dtype == ECC_U16 || dtype == ECC_F32) ? ECC_E_UNSUPPORTED : ECC_E_ARG;
    }
    if (!is_device_ptr(image_dev)) {
        set_error("ecc_autotune: the image must be device memory");
        return ECC_E_ARG;
    }
    IntView v{};
    int unsup = 0;
    if (!normalize_int_view(dims, &v, &unsup)) {
        set_error("integer path: shape not supported (4 axes longer than 1, or an extent beyond 2^31)");
        return ECC_E_UNSUPPORTED;
    }
    hipStream_t s = (hipStream_t)stream;
    Workspace *ws = nullptr;
    rc = get_workspace(s, &ws);
    if (rc) return rc;
    const int m = (int)threshold_count(dtype);
    rc = ensure_bytes((void **)&ws->vcec, &ws->vcec_bytes, (size_t)m * sizeof(int64_t));
    if (rc) return rc;
    hipEvent_t ev[2] = {nullptr, nullptr};
    hipError_t e = hipEventCreate(&ev[0]);
    if (e == hipSuccess) e = hipEventCreate(&ev[1]);
    if (e != hipSuccess) {
        if (ev[0]) (void)hipEventDestroy(ev[0]);
        return hip_fail(e, "ecc_autotune: events");
    }
    ecc_tiling win{};
    win.ms = 1e30f;
    const ecc_tiling rule = rule_tiling(v, dtype, v.n0);
    float rule_ms = 1e30f;
    IntJob job{};
    job.src.base = (const uint8_t *)image_dev;
    job.src.lo_base = job.src.base;
    job.src.plane_bytes = (int64_t)v.n1 * v.n2 * (int64_t)elem_bytes(dtype);
    job.view = v;
    job.e0 = 0;
    job.e1 = (int32_t)v.n0;
    job.lo_inf = 1;
    job.hi_inf = 1;
    job.dtype = dtype;
    // candidates, timed in rounds over all of them (one warm-up round, then
    // three; each keeps its fastest) so that clock ramps and drift do not
    // favour the ones timed last
    const int rows_c[2] = {2, 4}, tpc_c[3] = {4, 8, 16}, wx_c[2] = {8, 16};
    struct Cand {
        ecc_tiling p;
        IntTiling tl;
        float best;
    };
    std::vector<Cand> cands;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 3; ++b)
            for (int c = 0; c < (v.nin == 2 ? 2 : 1); ++c) {
                Cand x{};
                x.p.rows = rows_c[a];
                x.p.tiles_per_cu = tpc_c[b];
                x.p.waves_x = wx_c[c + (v.nin == 2 ? 0 : 1)];
                x.tl = tiling_from(v, dtype, v.n0, x.p, 0);
                x.best = 1e30f;
                cands.push_back(x);
                if (!rc) rc = ensure_bytes((void **)&ws->partial, &ws->partial_bytes,
                                           (size_t)x.tl.grid * m * sizeof(int32_t));
            }
    for (int round = 0; round < 4 && !rc; ++round)
        for (Cand &x : cands) {
            if ((e = hipEventRecord(ev[0], s)) != hipSuccess) rc = hip_fail(e, "ecc_autotune: event");
            if (!rc) rc = launch_int_partial(job, x.tl, ws->partial, ws->status, nullptr, s);
            if (!rc)
                rc = launch_merge(ws->partial, x.tl.grid, m, ws->vcec, false, false, nullptr, ws->status,
                                  nullptr, s);
            if (!rc && (e = hipEventRecord(ev[1], s)) != hipSuccess) rc = hip_fail(e, "ecc_autotune: event");
            if (!rc && (e = hipEventSynchronize(ev[1])) != hipSuccess) rc = hip_fail(e, "ecc_autotune: sync");
            float ms = 0.0f;
            if (!rc && (e = hipEventElapsedTime(&ms, ev[0], ev[1])) != hipSuccess) rc = hip_fail(e, "ecc_autotune");
            if (!rc && round > 0 && ms < x.best) x.best = ms;
            if (rc) break;
        }
    for (const Cand &x : cands) {
        if (x.p.rows == rule.rows && x.p.tiles_per_cu == rule.tiles_per_cu && x.p.waves_x == rule.waves_x)
            rule_ms = x.best;
        if (x.best < win.ms) {
            win = x.p;
            win.ms = x.best;
        }
    }
    // the rule stays unless a candidate beats it by 2 % (timing noise would
    // otherwise flip between near-equal tilings from run to run)
    if (!rc && win.ms > 0.98f * rule_ms) {
        win = rule;
        win.ms = rule_ms;
    }
    (void)hipEventDestroy(ev[0]);
    (void)hipEventDestroy(ev[1]);
    if (rc) return rc;
    // the status word collects range errors of the timed runs; read and clear it
    uint32_t st = 0;
    ECC_HIP(hipMemcpyAsync(&st, ws->status, 4, hipMemcpyDeviceToHost, s));
    ECC_HIP(hipStreamSynchronize(s));
    rc = launch_zero(ws->status, 8, s);
    if (rc) return rc;
    ECC_HIP(hipStreamSynchronize(s));
    if (st & kStatusRange) {
        set_error("a 14-bit image holds a value >= 16384");
        return ECC_E_RANGE;
    }
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tuned[TuneKey{dtype, v.nin, v.n1, v.n2, v.n0}] = win;
    }
    *best = win;
    return ECC_OK;
}

int ecc_tiling_for(const ecc_dims *dims, ecc_dtype dtype, ecc_tiling *out) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!out) {
        set_error("NULL output");
        return ECC_E_ARG;
    }
    if (dtype != ECC_U8 && dtype != ECC_U14 && dtype != ECC_U16) {
        set_error("ecc_tiling_for: integer dtypes");
        return dtype == ECC_F32 ? ECC_E_UNSUPPORTED : ECC_E_ARG;
    }
    IntView v{};
    int unsup = 0;
    if (!normalize_int_view(dims, &v, &unsup)) {
        set_error("integer path: shape not supported");
        return ECC_E_UNSUPPORTED;
    }
    *out = tiling_params(v, dtype, v.n0);
    out->ms = 0.0f;
    return ECC_OK;
}

void ecc_autotune_reset(void) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned.clear();
}

// The growable scratch of every workspace of the current device is freed, as
// are the blocks kept for its ecc_stream objects
// (the small status block and host word stay, so the workspaces remain
// valid); the next call on a stream grows its buffers again.  Work still in
// flight on the device may use them: it is waited for first.
int ecc_release_workspaces(void) {
    int dev = 0;
    ECC_HIP(hipGetDevice(&dev));
    ECC_HIP(hipDeviceSynchronize());
    hipError_t first = cache_release(dev);
    std::lock_guard<std::mutex> lk(g_ws_mu);
    auto drop = [&](void *p, size_t *cap) {
        if (p) {
            const hipError_t e = hipFree(p);
            if (e != hipSuccess && first == hipSuccess) first = e;
        }
        *cap = 0;
    };
    for (auto &kv : g_ws) {
        Workspace *w = kv.second;
        if (w->device != dev || w->fixed) continue;
        drop(w->partial, &w->partial_bytes);
        w->partial = nullptr;
        drop(w->vcec, &w->vcec_bytes);
        w->vcec = nullptr;
        drop(w->chi_tmp, &w->chi_tmp_bytes);
        w->chi_tmp = nullptr;
        drop(w->img_tmp, &w->img_tmp_bytes);
        w->img_tmp = nullptr;
        drop(w->fbuf, &w->fbuf_bytes);
        w->fbuf = nullptr;
        drop(w->frec, &w->frec_bytes);
        w->frec = nullptr;
        drop(w->fbits, &w->fbits_bytes);
        w->fbits = nullptr;
        drop(w->dual_buf, &w->dual_buf_bytes);
        w->dual_buf = nullptr;
        drop(w->vcec16, &w->vcec16_bytes);
        w->vcec16 = nullptr;
    }
    if (first != hipSuccess) return hip_fail(first, "hipFree(workspace)");
    return ECC_OK;
}

static const char kTuneTag[] = "ecc-tiling-v1";

int ecc_autotune_save(const char *path) {
    g_err[0] = 0;
    if (!path) {
        set_error("ecc_autotune_save: NULL path");
        return ECC_E_ARG;
    }
    std::vector<std::pair<TuneKey, ecc_tiling>> rows;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        rows.assign(g_tuned.begin(), g_tuned.end());
    }
    FILE *f = fopen(path, "w");
    if (!f) {
        set_error("ecc_autotune_save: cannot open %s for writing", path);
        return ECC_E_ARG;
    }
    bool ok = true;
    for (const auto &r : rows)
        ok = ok && fprintf(f, "%s %d %d %d %d %lld %d %d %d %.6g\n", kTuneTag, r.first.dtype, r.first.nin,
                           (int)r.first.n1, (int)r.first.n2, (long long)r.first.planes, (int)r.second.rows,
                           (int)r.second.tiles_per_cu, (int)r.second.waves_x, (double)r.second.ms) > 0;
    ok = (fclose(f) == 0) && ok;
    if (!ok) {
        set_error("ecc_autotune_save: write to %s failed", path);
        return ECC_E_ARG;
    }
    return (int)rows.size();
}

int ecc_autotune_load(const char *path) {
    g_err[0] = 0;
    if (!path) {
        set_error("ecc_autotune_load: NULL path");
        return ECC_E_ARG;
    }
    FILE *f = fopen(path, "r");
    if (!f) {
        set_error("ecc_autotune_load: cannot open %s", path);
        return ECC_E_ARG;
    }
    std::vector<std::pair<TuneKey, ecc_tiling>> rows;
    char line[512];
    int lineno = 0;
    bool ok = true;
    while (ok && fgets(line, sizeof line, f)) {
        ++lineno;
        char tag[32] = {0}, extra[2] = {0};
        int dtype = 0, nin = 0, n1 = 0, n2 = 0, r = 0, tpc = 0, wx = 0;
        long long planes = 0;
        double ms = 0;
        const int got = sscanf(line, "%31s %d %d %d %d %lld %d %d %d %lf %1s", tag, &dtype, &nin, &n1, &n2, &planes, &r,
                               &tpc, &wx, &ms, extra);
        if (got == EOF || (got == 1 && tag[0] == '#')) continue;  // blank line or comment
        ok = got == 10 && strcmp(tag, kTuneTag) == 0 && threshold_count((ecc_dtype)dtype) > 0 &&
             dtype != ECC_F32 && (nin == 1 || nin == 2) && n1 >= 1 && n2 >= 1 && planes >= 1 &&
             (r == 2 || r == 4) && (tpc == 4 || tpc == 8 || tpc == 16) && (wx == 8 || wx == 16) && ms >= 0;
        if (ok) {
            ecc_tiling t{};
            t.rows = r;
            t.tiles_per_cu = tpc;
            t.waves_x = wx;
            t.ms = (float)ms;
            rows.push_back({TuneKey{dtype, nin, n1, n2, (int64_t)planes}, t});
        }
    }
    const bool read_ok = !ferror(f);
    fclose(f);
    if (!ok || !read_ok) {
        if (!ok) set_error("ecc_autotune_load: %s line %d is not a tiling entry", path, lineno);
        else set_error("ecc_autotune_load: reading %s failed", path);
        return ECC_E_ARG;
    }
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (const auto &e : rows) g_tuned[e.first] = e.second;
    return (int)rows.size();
}

// Waits for the scan of a dual curve, reports its status and copies the curve
// to host memory if it belongs there.
static int finish_dual(Workspace *ws, ecc_curve *curve, const int64_t *chi_dev, bool chi_direct, int64_t m,
                       hipStream_t s) {
    ECC_HIP(hipStreamSynchronize(s));
    const uint32_t stv = *ws->host_status;
    if (stv == 0xFFFFFFFFu) {
        set_error("internal error: the scan did not report a status");
        return ECC_E_HIP;
    }
    if (stv & kStatusRange) {
        set_error("a 14-bit image holds a value >= 16384");
        return ECC_E_RANGE;
    }
    if (stv != 0) {
        set_error("internal error: device status 0x%08x", stv);
        return ECC_E_HIP;
    }
    if (!chi_direct) {
        ECC_HIP(hipMemcpyAsync(curve->chi, chi_dev, (size_t)m * sizeof(int64_t), hipMemcpyDefault, s));
        ECC_HIP(hipStreamSynchronize(s));
    }
    curve->count = m;
    return ECC_OK;
}

// Dual complex (voxels as vertices, lower-star filtration).  Its cells are
// the cells of the voxel complex away from the box's outer boundary, with
// dimension d - dim and value the maximum over their voxels, so by
// inclusion-exclusion over the faces F of the box (every axis free, or fixed
// at its first or last index):
//   dual(f)(t) = (-1)^d sum_F (-1)^codim(F) max_entry(f|F)(t).
// The sum is linear, so it is taken over the faces' changes vectors and the
// result is scanned once.  Axes of length 1 are dropped first (a product
// with a point).
int ecc_compute_dual(const void *image, const ecc_dims *dims, ecc_dtype dtype, ecc_curve *curve, void *stream) {
    g_err[0] = 0;
    int64_t total = 0;
    int rc = check_dims(dims, &total);
    if (rc) return rc;
    if (!image || !curve || !curve->chi) {
        set_error("NULL image, curve or curve->chi");
        return ECC_E_ARG;
    }
    if (dtype != ECC_U8 && dtype != ECC_U14) {
        if (dtype == ECC_F32 || dtype == ECC_U16) {
            set_error("ecc_compute_dual: integer dtypes u8 and u14 only");
            return ECC_E_UNSUPPORTED;
        }
        set_error("unknown dtype %d", (int)dtype);
        return ECC_E_ARG;
    }
    const int64_t m = threshold_count(dtype);
    if (curve->capacity < m) {
        curve->count = m;
        set_error("curve capacity %lld < %lld", (long long)curve->capacity, (long long)m);
        return ECC_E_BUFFER_TOO_SMALL;
    }
    int64_t n[4];
    int d = 0;
    for (int k = 0; k < dims->ndim; ++k)
        if (dims->n[k] > 1) n[d++] = dims->n[k];
    // (d <= 4: the full box of a 4-D image goes through the change kernel, its
    // faces of at most three dimensions through the integer kernel)
    hipStream_t s = (hipStream_t)stream;
    Workspace *ws = nullptr;
    rc = get_workspace(s, &ws);
    if (rc) return rc;
    const size_t eb = elem_bytes(dtype);
    const void *img_dev = image;
    if (!is_device_ptr(image)) {
        rc = ensure_bytes(&ws->img_tmp, &ws->img_tmp_bytes, (size_t)total * eb);
        if (rc) return rc;
        ECC_HIP(hipMemcpyAsync(ws->img_tmp, image, (size_t)total * eb, hipMemcpyHostToDevice, s));
        img_dev = ws->img_tmp;
    }
    int nf = 1;
    for (int k = 0; k < d; ++k) nf *= 3;
    const int gsign = (d & 1) ? -1 : 1;
    int64_t st[4] = {1, 1, 1, 1};  // element strides of the kept axes
    for (int k = d - 2; k >= 0; --k) st[k] = st[k + 1] * n[k + 1];
    int64_t face_max = 1;  // the largest face of codimension >= 1
    for (int k = 0; k < d; ++k)
        if (total / n[k] > face_max) face_max = total / n[k];
    // dual_buf: up to three dimensions [m] the signed sum's changes, [m] the
    // curve; for a 4-D image [nf][m] changes vectors of the full box and its
    // faces of three dimensions, [m] the changes of its faces of at most two
    // (all of them, signed), [m] the signed sum, [m] the curve
    const int nvec = d == 4 ? nf + 2 : 1;
    rc = ensure_bytes(&ws->dual_buf, &ws->dual_buf_bytes, (size_t)(nvec + 1) * m * sizeof(int64_t));
    if (rc) return rc;
    int64_t *curves = (int64_t *)ws->dual_buf;
    const bool chi_direct = is_device_ptr(curve->chi);
    int64_t *chi_dev = chi_direct ? curve->chi : curves + (size_t)nvec * m;
    struct Face {
        int nfree, codim;
        int64_t base, n[4], stride[4];
    };
    auto face = [&](int f) {  // axis k of face f: free, or fixed at its first or last index
        Face F{0, 0, 0, {1, 1, 1, 1}, {0, 0, 0, 0}};
        for (int k = 0, r = f; k < d; ++k, r /= 3) {
            if (r % 3 == 0) {
                F.n[F.nfree] = n[k];
                F.stride[F.nfree] = st[k];
                ++F.nfree;
            } else {
                F.base += (r % 3 == 1 ? 0 : n[k] - 1) * st[k];
                ++F.codim;
            }
        }
        return F;
    };
    std::vector<BoxFace> low;
    for (int f = 0; f < nf; ++f) {
        const Face F = face(f);
        if (F.codim == 0 || F.nfree > 2) continue;
        BoxFace B{};
        B.base = F.base;
        B.na = F.nfree == 2 ? F.n[0] : 0;
        B.sa = F.nfree == 2 ? F.stride[0] : 0;
        B.nb = F.nfree ? F.n[F.nfree - 1] : 0;
        B.sb = F.nfree ? F.stride[F.nfree - 1] : 0;
        B.sign = (F.codim & 1) ? -1 : 1;
        low.push_back(B);
    }
    const int cus = device_cu_count();
    const int low_rows = box_face_rows(low.data(), (int)low.size(), cus);
    *ws->host_status = 0xFFFFFFFFu;  // overwritten by the scan
    if (d < 4) {
        // One merge over the count rows of the box and of its faces, all on
        // s: the faces' launch is short (16 us for 400 x 413 x 390, of 115 per
        // curve); beside the volume on a side stream, with a fork, a join and a
        // signed sum, the curve took 168.
        ecc_dims bd{};
        bd.ndim = d > 0 ? d : 1;
        for (int k = 0; k < 4; ++k) bd.n[k] = k < d ? n[k] : 1;
        IntView v{};
        int unsup = 0, rows = 0;
        if (!normalize_int_view(&bd, &v, &unsup)) {
            set_error("ecc_compute_dual: shape not supported");
            return ECC_E_UNSUPPORTED;
        }
        StatusCleanup cleanup{ws, s, true};
        rc = enqueue_max_entry_rows(img_dev, v, dtype, low_rows, &rows, s, ws);
        if (!rc)
            rc = launch_box_faces(img_dev, (int)eb, low.data(), (int)low.size(), cus, ws->partial + (size_t)rows * m, s);
        if (!rc)
            rc = launch_merge(ws->partial, rows + low_rows, (int)m, curves, false, true, chi_dev, ws->status,
                              ws->host_status_dev, s, true, gsign < 0);
        if (rc) return rc;
        cleanup.armed = false;  // (the scan clears the status word)
        return finish_dual(ws, curve, chi_dev, chi_direct, m, s);
    }
    int64_t *lowv = curves + (size_t)nf * m;
    int64_t *result = lowv + m;
    // The full box runs on s; its faces of three dimensions (of a 4-D image)
    // go round-robin to the side streams, each with its own workspace (and
    // gather buffer in its img_tmp), those of at most two in one launch.
    SideStreams *side = nullptr;
    rc = get_side_streams(s, &side);
    if (rc) return rc;
    Workspace *sws[SideStreams::kCount] = {};
    for (int k = 0; k < SideStreams::kCount; ++k) {
        rc = get_workspace(side->s[k], &sws[k]);
        if (rc) return rc;
    }
    bool used[SideStreams::kCount] = {};
    int next_side = 0;
    // after the fork, every return first waits for the side streams (their
    // work uses buffers that a later call may reallocate)
    auto sync_sides = [&]() {
        for (int k = 0; k < SideStreams::kCount; ++k)
            if (used[k]) (void)hipStreamSynchronize(side->s[k]);
    };
    StatusCleanup cleanup{ws, s, true};
    ECC_HIP(hipEventRecord(side->fork, s));  // the image (and its copy, if any) is ready here
    auto fork_to = [&](int k) -> int {
        if (used[k]) return ECC_OK;
        const hipError_t e = hipStreamWaitEvent(side->s[k], side->fork, 0);
        if (e != hipSuccess) return hip_fail(e, "ecc_compute_dual: fork");
        used[k] = true;
        return ECC_OK;
    };
    uint64_t neg[2] = {0, 0}, skip[2] = {0, 0};  // bit f of the pair: face f
    auto set_bit = [](uint64_t *mask, int f) { mask[f >> 6] |= 1ull << (f & 63); };
    // The faces of at most two dimensions on a side stream, summed as one more
    // face (slot nf, which carries their signs already).
    {
        const int k = next_side++ % SideStreams::kCount;
        Workspace *lws = sws[k];
        rc = fork_to(k);
        if (!rc) rc = ensure_bytes((void **)&lws->partial, &lws->partial_bytes, (size_t)low_rows * m * sizeof(int32_t));
        if (!rc) rc = launch_box_faces(img_dev, (int)eb, low.data(), (int)low.size(), cus, lws->partial, side->s[k]);
        if (!rc)
            rc = launch_merge(lws->partial, low_rows, (int)m, lowv, false, false, nullptr, lws->status, nullptr,
                              side->s[k], true);
        if (rc) {
            sync_sides();
            return rc;
        }
    }
    for (int f = 0; f < nf; ++f) {
        const Face F = face(f);
        if (F.nfree <= 2) {
            set_bit(skip, f);
            continue;
        }
        if (F.nfree == 4) {  // the whole 4-D box
            ecc_dims bd{};
            bd.ndim = 4;
            for (int k = 0; k < 4; ++k) bd.n[k] = n[k];
            ChangeJob box{};
            rc = four_d_job(img_dev, &bd, total, dtype, true, &box);
            if (!rc) rc = enqueue_four_d(box, true, nullptr, curves + (size_t)f * m, nullptr, s, ws);
            if (rc) {
                sync_sides();
                return rc;
            }
            continue;
        }
        // a face of three dimensions, gathered into the next side stream's
        // buffer (its faces run in stream order)
        const int k = next_side++ % SideStreams::kCount;
        Workspace *fws = sws[k];
        rc = fork_to(k);
        if (!rc) rc = ensure_bytes(&fws->img_tmp, &fws->img_tmp_bytes, (size_t)face_max * eb);
        if (!rc)
            rc = launch_gather(img_dev, (int)eb, F.base, F.stride[0], F.stride[1], F.stride[2], F.n[0], F.n[1], F.n[2],
                               fws->img_tmp, side->s[k]);
        IntView v{};
        ecc_dims fd{};
        fd.ndim = 3;
        fd.n[3] = 1;
        for (int i = 0; i < 3; ++i) fd.n[i] = F.n[i];
        int unsup = 0, rows = 0;
        if (!rc && !normalize_int_view(&fd, &v, &unsup)) {
            set_error("ecc_compute_dual: face shape not supported");
            rc = ECC_E_UNSUPPORTED;
        }
        if (!rc) rc = enqueue_max_entry_rows(fws->img_tmp, v, dtype, 0, &rows, side->s[k], fws);
        if (!rc)
            rc = launch_merge(fws->partial, rows, (int)m, curves + (size_t)f * m, false, false, nullptr, fws->status,
                              nullptr, side->s[k], true);
        if (rc) {
            sync_sides();
            return rc;
        }
        if (F.codim & 1) set_bit(neg, f);
    }
    // join: s waits for every side stream that took work
    for (int k = 0; k < SideStreams::kCount; ++k) {
        if (!used[k]) continue;
        hipError_t e = hipEventRecord(side->join[k], side->s[k]);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, side->join[k], 0);
        if (e != hipSuccess) {
            sync_sides();
            return hip_fail(e, "ecc_compute_dual: join");
        }
    }
    rc = launch_signed_sum(curves, nf + 1, neg, skip, gsign, (int)m, result, s);
    if (rc) return rc;
    // the scan (its changes are summed already), into the caller's buffer if
    // it is device memory; the status of every launch on the volume or a face
    // of three dimensions (the volume's reads all values) is reported and
    // cleared here, and nothing is written unless it is clear
    rc = launch_merge(nullptr, 0, (int)m, result, true, true, chi_dev, ws->status, ws->host_status_dev, s);
    if (rc) return rc;
    cleanup.armed = false;  // (the scan clears the status word)
    return finish_dual(ws, curve, chi_dev, chi_direct, m, s);
}

}  // extern "C"
