/*
 * Host paths of libecc without a GPU: this program defines the HIP runtime
 * calls that the library makes (its own definitions come before the runtime's
 * for the libraries that it loads), with device memory as addresses that are
 * only counted, and kernels that are only noted.  What a few kernels report to
 * the host is filled in.  argv[1] names the scenario; it prints "key value"
 * lines for the test.
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include "ecc.h"

/* ------------------------------------------------------------ the runtime */

#define DEVICE_LO 0x010000000000ull
#define DEVICE_HI 0x200000000000ull
static uint64_t next_address = DEVICE_LO;
static struct {
    uint64_t p;
    size_t bytes;
} blocks[4096];
static int nblocks;
static size_t used, peak, limit_bytes = (size_t)-1;
static hipError_t last_error;

static struct {
    const void *host;
    const char *name;
} kernels[4096];
static int nkernels;
static long launches;
static int syncs;

static uint32_t status_word;  /* the status word of the one stream that a scenario uses */
static int nan_image;         /* the float image holds a NaN */
static int range_image;       /* the 14-bit image holds a value >= 16384 */
static int stream_waits;      /* for the stream that the scenario gave */
static hipStream_t its_stream;
static int top_bytes = 3;     /* top bytes of the float image's keys */
static long change_launches;  /* of the change kernel */
static long face_launches;    /* of the box faces' kernel */
static unsigned int_grid;     /* workgroups of the last launch of the integer kernel */
static unsigned int_waves;    /* and the waves of each */
static const char *int_kernel = "";

static int is_device(const void *p) { return (uint64_t)p >= DEVICE_LO && (uint64_t)p < DEVICE_HI; }
static hipError_t result(hipError_t e) {
    if (e != hipSuccess) last_error = e;
    return e;
}

hipError_t hipMalloc(void **p, size_t n) {
    if (n > limit_bytes - used) return result(hipErrorOutOfMemory);
    blocks[nblocks].p = next_address;
    blocks[nblocks++].bytes = n;
    *p = (void *)next_address;
    next_address += (n + 0x200000) & ~(uint64_t)0xFFFFF;
    used += n;
    if (used > peak) peak = used;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    for (int i = 0; i < nblocks; ++i)
        if (blocks[i].p == (uint64_t)p) {
            used -= blocks[i].bytes;
            blocks[i] = blocks[--nblocks];
            return hipSuccess;
        }
    printf("bad_free 1\n");
    return result(hipErrorInvalidValue);
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned flags) { *d = h; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    if (!is_device(p)) return result(hipErrorInvalidValue);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipGetLastError(void) {
    hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    ++syncs;
    if (s == its_stream) ++stream_waits;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned f) { *s = (hipStream_t)malloc(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) { *ms = 1.0f; return hipSuccess; }
static int32_t copied[2];  /* the first words of the last copy to the device */
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
    if (is_device(d)) {
        if (!is_device(s) && n >= sizeof copied) memcpy(copied, s, sizeof copied);
        return hipSuccess;
    }
    if (!is_device(s)) memcpy(d, s, n);
    else if (n == 4) memcpy(d, &status_word, 4);
    else memset(d, 0, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { return hipMemcpyAsync(d, s, n, k, 0); }

void **__hipRegisterFatBinary(const void *data) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) {}
void __hipRegisterVar(void **m, void *v, char *hv, char *dv, int e, size_t n, int c, int g) {}
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned n, void *t, void *b, void *bd,
                           void *gd, int *w) {
    kernels[nkernels].host = f;
    kernels[nkernels++].name = name;
}
static dim3 pushed_grid, pushed_block;
static size_t pushed_shared;
static hipStream_t pushed_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, hipStream_t s) {
    pushed_grid = g;
    pushed_block = b;
    pushed_shared = shared;
    pushed_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *s) {
    *g = pushed_grid;
    *b = pushed_block;
    *shared = pushed_shared;
    *s = pushed_stream;
    return hipSuccess;
}
/* argument k of a launch, a pointer to host memory, or NULL */
static uint32_t *host_argument(void **args, int k) {
    void *p = *(void **)args[k];
    return p && !is_device(p) ? (uint32_t *)p : NULL;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t shared, hipStream_t s) {
    const char *name = "";
    for (int i = 0; i < nkernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    ++launches;
    uint32_t *out;
    if (strstr(name, "zero_kernel")) {
        const size_t words = *(size_t *)args[1];
        if (words <= 2 || words == (128 + 1024 * 8 + 128) / 4) status_word = 0;  /* the word, or a new status block */
    } else if (strstr(name, "split_kernel")) {
        if (nan_image) status_word |= 2u;
    } else if (strstr(name, "bucket_totals_kernel")) {
        out = host_argument(args, 4);
        for (int w = 0; w < 8; ++w) out[w] = 0;
        for (int k = 0; k < top_bytes; ++k) out[k / 32] |= 1u << (k % 32);
    } else if (strstr(name, "nz_total_kernel")) {
        memset(host_argument(args, 2), 0, 8);
    } else if (strstr(name, "tile_base_kernel")) {
        *(int64_t *)host_argument(args, 7) = 1;
        *host_argument(args, 9) = status_word;
    } else if (strstr(name, "merge_scan_small_kernel")) {
        if ((out = host_argument(args, 9))) *out = status_word;
        status_word = 0;
    } else if (strstr(name, "11scan_kernel")) {
        if ((out = host_argument(args, 6))) *out = status_word;
        status_word = 0;
    } else if (strstr(name, "box_faces_kernel")) {
        ++face_launches;
    } else if (strstr(name, "int_vcec_kernel")) {
        int_grid = g.x;
        int_waves = b.x / 64;
        int_kernel = name;
    } else if (strstr(name, "change_kernel")) {
        ++change_launches;
        if (range_image) status_word |= 1u;
    }
    return hipSuccess;
}

/* -------------------------------------------------------------- scenarios */

static ecc_dims dims_of(int nd, int64_t a, int64_t b, int64_t c, int64_t d) {
    ecc_dims r = {nd, {a, b, c, d}};
    return r;
}
/* device memory that is an input or output of a call */
static void *device_bytes(size_t n) {
    void *p = (void *)next_address;
    next_address += (n + 0x200000) & ~(uint64_t)0xFFFFF;
    return p;
}

/* A float image with a NaN whose call fails for want of memory at each of its
 * allocations in turn, and a valid 14-bit image on the same stream after it. */
static int float_exits(void) {
    ecc_dims d = dims_of(3, 20, 30, 40, 1);
    void *img = device_bytes(24000 * 4);
    static float keys[24000];
    static int64_t chi[24000];
    for (int k = 0; k < 6; ++k) {
        for (top_bytes = 3; top_bytes <= 40; top_bytes += 37) {
            char num[8];
            void *stream = malloc(8);
            ecc_curve c = {24000, 0, chi, keys};
            nan_image = 0;
            snprintf(num, sizeof num, "%d", k + 1);
            setenv("ECC_FAIL_ALLOC", num, 1);
            const int before = syncs;
            nan_image = 1;
            const int rc = ecc_compute(img, &d, ECC_F32, &c, stream);
            printf("float rc %d waits %d status %u\n", rc, syncs - before, status_word);
            unsetenv("ECC_FAIL_ALLOC");
            ecc_curve v = {16384, 0, chi, NULL};
            printf("next rc %d\n", ecc_compute(img, &d, ECC_U14, &v, stream));
        }
    }
    return 0;
}

/* The dual curve of a 4-D image with a value out of range whose call fails at
 * each of its allocations in turn, and a valid image on the same stream. */
static int dual_exits(void) {
    ecc_dims d = dims_of(4, 6, 7, 8, 9), v = dims_of(2, 20, 30, 1, 1);
    void *img = device_bytes(6 * 7 * 8 * 9 * 2);
    static int64_t chi[16384];
    for (int k = 1; k <= 40; ++k) {
        char num[8];
        its_stream = (hipStream_t)malloc(8);
        ecc_curve c = {16384, 0, chi, NULL};
        snprintf(num, sizeof num, "%d", k);
        setenv("ECC_FAIL_ALLOC", num, 1);
        range_image = 1;
        change_launches = stream_waits = 0;
        const int rc = ecc_compute_dual(img, &d, ECC_U14, &c, its_stream);
        printf("dual rc %d launched %ld waits %d status %u\n", rc, change_launches, stream_waits, status_word);
        range_image = 0;
        unsetenv("ECC_FAIL_ALLOC");
        printf("next rc %d\n", ecc_compute(img, &v, ECC_U14, &c, its_stream));
    }
    return 0;
}

/* Memory enough for a call only without the blocks that a finished stream left. */
static int kept_blocks(void) {
    ecc_dims d = dims_of(3, 64, 2048, 2048, 1), v = dims_of(3, 200, 300, 300, 1);
    void *img = device_bytes(1 << 26);
    static int64_t chi[16384];
    ecc_curve c = {16384, 0, chi, NULL};
    for (int k = 0; k < 100; ++k) {  /* more blocks than are kept, of many sizes */
        ecc_dims small = dims_of(2, 100, 100 + 7000 * k, 1, 1);
        ecc_stream *st[2];
        for (int i = 0; i < 2; ++i) ecc_stream_begin(&small, ECC_U8, NULL, &st[i]);
        for (int i = 0; i < 2; ++i) ecc_stream_abort(st[i]);
    }
    printf("small kept %zu\n", used);
    ecc_stream *st = NULL;
    printf("begin rc %d\n", ecc_stream_begin(&d, ECC_U14, NULL, &st));
    ecc_stream_abort(st);
    printf("large kept %zu\n", used);
    limit_bytes = used + (1 << 20);
    printf("call rc %d\n", ecc_compute(img, &v, ECC_U14, &c, NULL));
    printf("after used %zu\n", used);
    limit_bytes = used;
    printf("none rc %d error %d\n", ecc_compute(img, &d, ECC_U14, &c, NULL), (int)hipGetLastError());
    return 0;
}

/* A float image of a few thousand voxels on a nearly full card. */
static int float_nearly_full(void) {
    ecc_dims d = dims_of(3, 10, 20, 30, 1);
    void *img = device_bytes(6000 * 4);
    static float keys[6000];
    static int64_t chi[6000];
    ecc_curve c = {6000, 0, chi, keys};
    limit_bytes = 1 << 20;
    printf("float rc %d\n", ecc_compute(img, &d, ECC_F32, &c, NULL));
    return 0;
}

/* What a run allocates, against its jobs' footprints less images and curves. */
static void batch_of(const char *name, int n, const ecc_dims *dims, const int *dtypes) {
    ecc_batch *b = NULL;
    ecc_job jobs[64];
    const int64_t extra = 32 << 20;
    int64_t bound = (64 << 10) + 4 * n + 1024;  /* the table and the status words */
    for (int i = 0; i < n; ++i) {
        ecc_job j = {device_bytes(16), dims[i], dtypes[i], (int64_t *)device_bytes(65536 * 8)};
        int64_t foot = 0, bytes = dtypes[i] == ECC_U8 ? 1 : 2;
        ecc_job_footprint(&j, &foot);
        for (int k = 0; k < dims[i].ndim; ++k) bytes *= dims[i].n[k];
        bound += foot - bytes - 8 * (dtypes[i] == ECC_U8 ? 256 : 16384);
        jobs[i] = j;
    }
    ecc_batch_create(NULL, &b);
    const size_t before = used;
    const int rc = ecc_batch_run(b, n, jobs, NULL);
    printf("%s rc %d bytes %zu bound %lld\n", name, rc, used - before, (long long)(bound + extra));
    ecc_batch_destroy(b);
    limit_bytes = used + bound;  /* no more memory than the footprints' */
    ecc_batch_create(NULL, &b);
    const int rc2 = ecc_batch_run(b, n, jobs, NULL);
    printf("short rc %d bytes %zu bound %lld\n", rc2, used - before, (long long)bound);
    ecc_batch_destroy(b);
    limit_bytes = (size_t)-1;
}
static int batch_rows(void) {
    setenv("ECC_BATCH_GRAPH", "0", 1);
    const int u14[1] = {ECC_U14}, u8[1] = {ECC_U8};
    ecc_dims d = dims_of(3, 128, 128, 128, 1);
    batch_of("cube", 1, &d, u14);
    d = dims_of(2, 1 << 30, 2, 1, 1);
    batch_of("columns", 1, &d, u14);
    d = dims_of(2, 2000, 64, 1, 1);
    batch_of("picture", 1, &d, u8);
    unsigned seed = 1;
    for (int n = 2; n <= 64; n *= 2) {
        ecc_dims dims[64];
        int types[64];
        for (int i = 0; i < n; ++i) {
            int64_t r[3];
            for (int k = 0; k < 3; ++k) r[k] = (seed = seed * 1664525u + 1013904223u) >> 8;
            types[i] = r[0] & 1 ? ECC_U8 : ECC_U14;
            if (types[i] == ECC_U8) dims[i] = dims_of(2, 32 + r[1] % 2000, 32 + r[2] % 2000, 1, 1);
            else dims[i] = dims_of(3, 16 + r[0] / 2 % 241, 16 + r[1] % 241, 16 + r[2] % 241, 1);
        }
        batch_of("mix", n, dims, types);
    }
    return 0;
}

/* The tiles of a run (word 1 of its table) after the tuner, every candidate as fast. */
static int batch_tuned(void) {
    setenv("ECC_BATCH_GRAPH", "0", 1);
    const int n0[3] = {256, 2000, 150};
    for (int i = 0; i < 3; ++i) {
        ecc_batch *b = NULL;
        ecc_job j = {device_bytes(16), dims_of(3, n0[i], 32, 64, 1), ECC_U14, (int64_t *)device_bytes(65536 * 8)};
        int32_t min_planes = 0, split = 0;
        float ms = 0;
        ecc_batch_create(NULL, &b);
        const int rc = ecc_batch_autotune(b, 1, &j, &min_planes, &split, &ms);
        ecc_batch_run(b, 1, &j, NULL);
        printf("tuned rc %d n0 %d min_planes %d split %d tiles %d\n", rc, n0[i], min_planes, split, copied[1]);
        ecc_batch_destroy(b);
    }
    return 0;
}

/* The workgroups of a launch by the rule and with tilings loaded from argv[2]. */
static int tilings(const char *path) {
    ecc_dims d = dims_of(3, 200, 300, 300, 1);
    void *img = device_bytes(1 << 26);
    int64_t *chi = device_bytes(16384 * 8);
    ecc_compute_async(img, &d, ECC_U14, chi, NULL, NULL);
    printf("rule grid %u\n", int_grid);
    const char *params[4] = {"2 4 16", "2 16 16", "2 8 8", "4 4 8"};
    for (int i = 0; i < 4; ++i) {
        FILE *f = fopen(path, "w");
        fprintf(f, "ecc-tiling-v1 2 2 300 300 200 %s 0.1\n", params[i]);
        fclose(f);
        const int rc = ecc_autotune_load(path);
        ecc_compute_async(img, &d, ECC_U14, chi, NULL, NULL);
        printf("loaded rc %d grid %u\n", rc, int_grid);
    }
    return 0;
}

/* The launches of 4-D chunks of more than 2^30 values. */
static int stream_4d(void) {
    const int types[3] = {ECC_U8, ECC_U14, ECC_U16};
    for (int i = 0; i < 3; ++i) {
        ecc_dims d = dims_of(4, 10000, 64, 64, 64);
        ecc_stream *st = NULL;
        ecc_stream_begin(&d, types[i], NULL, &st);
        change_launches = 0;
        const int rc = ecc_stream_push_chunk(st, device_bytes((size_t)5000 << 19), 5000);
        printf("push rc %d values %ld launches %ld\n", rc, 4999L << 18, change_launches);
        change_launches = 0;
        const int rc2 = ecc_stream_push_chunk(st, device_bytes((size_t)5000 << 19), 5000);
        printf("push rc %d values %ld launches %ld\n", rc2, 5001L << 18, change_launches);
        ecc_stream_abort(st);
    }
    return 0;
}

/* The dual curve of volumes with faces of many short rows. */
static int dual_long(void) {
    const int64_t n[5][3] = {{0x7FFFFFFFll - 4, 2, 2}, {1500000000, 60, 2}, {2000000000, 2, 2}, {1000, 900, 800}, {2, 2, 2}};
    for (int i = 0; i < 5; ++i) {
        ecc_dims d = dims_of(3, n[i][0], n[i][1], n[i][2], 1);
        static int64_t chi[16384];
        ecc_curve c = {16384, 0, chi, NULL};
        face_launches = 0;
        const int rc = ecc_compute_dual(device_bytes((size_t)n[i][0] * n[i][1] * n[i][2]), &d, ECC_U8, &c, NULL);
        printf("dual rc %d launches %ld\n", rc, face_launches);
    }
    return 0;
}

/* The integer kernel that images take: argv[2] tilings to load ("-": none),
 * argv[3] "min" or "max", then per image its extents as n0xn1xn2 (8 bits). */
static ecc_dims parse_dims(char *p) {
    ecc_dims d = dims_of(1, 1, 1, 1, 1);
    for (d.ndim = 0; *p; ++d.ndim, p += *p == 'x') d.n[d.ndim] = strtoll(p, &p, 10);
    return d;
}
static int kernel_of(int argc, char **argv) {
    if (strcmp(argv[2], "-")) printf("loaded rc %d\n", ecc_autotune_load(argv[2]));
    static int64_t chi[256];
    for (int i = 4; i < argc; ++i) {
        ecc_dims d = parse_dims(argv[i]);
        ecc_curve c = {256, 0, chi, NULL};
        int (*call)(const void *, const ecc_dims *, ecc_dtype, ecc_curve *, void *) =
            strcmp(argv[3], "max") ? ecc_compute : ecc_compute_max_entry;
        const int rc = call(device_bytes(1 << 20), &d, ECC_U8, &c, NULL);
        printf("%s rc %d grid %u waves %u kernel %s\n", argv[i], rc, int_grid, int_waves, int_kernel);
    }
    return 0;
}

/* Device memory of float images of narrow planes. */
static int float_memory(void) {
    const int64_t n[4][4] = {{1 << 22, 2, 2, 1}, {1 << 23, 2, 1, 1}, {1 << 20, 2, 2, 2}, {256, 256, 256, 1}};
    for (int i = 0; i < 4; ++i) {
        ecc_dims d = dims_of(4, n[i][0], n[i][1], n[i][2], n[i][3]);
        const int64_t voxels = n[i][0] * n[i][1] * n[i][2] * n[i][3];
        ecc_curve c = {voxels, 0, device_bytes(voxels * 8), device_bytes(voxels * 4)};
        const size_t before = used;
        const int rc = ecc_compute(device_bytes(voxels * 4), &d, ECC_F32, &c, malloc(8));
        printf("float rc %d bytes %zu voxels %lld\n", rc, used - before, (long long)voxels);
    }
    return 0;
}

/* The workgroups of a 16-bit image's passes, per image. */
static int grids_u16(int argc, char **argv) {
    for (int i = 2; i < argc; ++i) {
        ecc_dims d = parse_dims(argv[i]);
        const int rc = ecc_compute_async(device_bytes(1 << 20), &d, ECC_U16, device_bytes(65536 * 8), NULL, NULL);
        printf("%s rc %d grid %u\n", argv[i], rc, int_grid);
    }
    return 0;
}

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "float_exits")) return float_exits();
    if (!strcmp(what, "dual_exits")) return dual_exits();
    if (!strcmp(what, "kept_blocks")) return kept_blocks();
    if (!strcmp(what, "float_nearly_full")) return float_nearly_full();
    if (!strcmp(what, "batch_rows")) return batch_rows();
    if (!strcmp(what, "batch_tuned")) return batch_tuned();
    if (!strcmp(what, "tilings")) return tilings(argv[2]);
    if (!strcmp(what, "stream_4d")) return stream_4d();
    if (!strcmp(what, "dual_long")) return dual_long();
    if (!strcmp(what, "kernel_of")) return kernel_of(argc, argv);
    if (!strcmp(what, "float_memory")) return float_memory();
    if (!strcmp(what, "grids_u16")) return grids_u16(argc, argv);
    fprintf(stderr, "no scenario %s\n", what);
    return 2;
}
