/* Host-side rules of the launches, without a GPU: this program defines the HIP
 * calls that the library makes (its own definitions go before the runtime's),
 * hands out addresses for device memory, records what would be launched, and
 * refuses launches that HIP refuses.  Nothing runs and nothing reads an image.
 *
 *   c_fake_device SCENARIO    exit status 0: as expected; prints what was not
 */
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "iqa.h"

typedef struct { uint32_t x, y, z; } dim3_t;

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static int mallocs, launches, captured_mallocs;
static size_t malloc_bytes;
static uintptr_t next_address = (uintptr_t)1 << 40;   /* of device memory that does not exist */
static void *capturing;          /* the stream that is being captured */
static uint64_t last_items;      /* work items of the last launch */
static size_t last_lds;
static char scratch[1 << 20];

int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetLastError(void) { return 0; }
int hipMalloc(void **p, size_t n) {
    pthread_mutex_lock(&mu);
    ++mallocs;
    captured_mallocs += capturing != NULL;
    malloc_bytes += n;
    *p = (void *)next_address;
    next_address += (n + 4095) / 4096 * 4096;
    pthread_mutex_unlock(&mu);
    return 0;
}
int hipFree(void *p) { (void)p; return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)p, (void)v, (void)n, (void)s; return 0; }
int hipStreamIsCapturing(void *s, int *st) { *st = s == capturing ? 1 : 0; return 0; }
int hipThreadExchangeStreamCaptureMode(int *m) { (void)m; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = scratch; return 0; }
int hipLaunchKernel(const void *fn, dim3_t grid, dim3_t block, void **args, size_t lds, void *s) {
    (void)fn, (void)args, (void)s;
    const uint64_t items = (uint64_t)grid.x * block.x;
    pthread_mutex_lock(&mu);
    ++launches;
    last_items = items;
    last_lds = lds;
    pthread_mutex_unlock(&mu);
    return items >> 32 ? 9 : 0;   /* hipErrorInvalidConfiguration */
}

#define CHECK(c) do { if (!(c)) { printf("%s:%d: %s\n", __FILE__, __LINE__, #c); return 1; } } while (0)

static const float *const X = (const float *)(uintptr_t)(1 << 20), *const Y = (const float *)(uintptr_t)(2 << 20);
static float *const OUT = (float *)(uintptr_t)(3 << 20), *const OUT2 = (float *)(uintptr_t)(4 << 20);
static void *const PER_THREAD = (void *)(uintptr_t)2;   /* hipStreamPerThread */

static int tiles_at(const float *x, int64_t N, int64_t NT, const iqa_launch_cfg *c, void *s) {
    return iqa_tiles_cfg(x, Y, N, NT, 5e-7f, 1e-6f, 1e-6f, 1e-6f, OUT, OUT2, NULL, c, s);
}

static int tiles(int64_t N, int64_t NT, void *s) { return tiles_at(X, N, NT, NULL, s); }

static int merge(void *s) {
    return iqa_merge_tiles(X, 512, 512, 5e-7f, 1e-6f, 1e-6f, OUT, OUT2, NULL, s);
}

/* ---- hipStreamPerThread is a stream of its own in each host thread ---- */

typedef struct { int which, status, mallocs; } Job;

static int split_call(int which) {
    switch (which) {
        case 0: return merge(PER_THREAD);
        case 1: return tiles(3000, 300, PER_THREAD);   /* split by the built-in rule alone */
        default: return tiles(2048, 256, PER_THREAD);  /* split by the tuned table */
    }
}

static void *thread_main(void *p) {
    Job *j = p;
    const int before = mallocs;
    j->status = split_call(j->which);
    if (j->status == 0) j->status = split_call(j->which);
    j->mallocs = mallocs - before;
    return NULL;
}

static int per_thread(void) {
    for (int which = 0; which < 3; ++which) {
        const int start = mallocs;
        Job mine = {which, 0, 0}, other = {which, 0, 0};
        thread_main(&mine);
        pthread_t t;
        CHECK(pthread_create(&t, NULL, thread_main, &other) == 0);
        pthread_join(t, NULL);
        CHECK(mine.status == 0 && other.status == 0);
        if (which != 1) CHECK(mine.mallocs == 1);      /* 0 and 1 use the same buffer */
        if (which != 1) CHECK(other.mallocs == 1);     /* not the first thread's */
        /* Threads that come and go pass their buffers on. */
        for (int i = 0; i < 20; ++i) {
            CHECK(pthread_create(&t, NULL, thread_main, &other) == 0);
            pthread_join(t, NULL);
            CHECK(other.status == 0);
        }
        CHECK(mallocs - start <= 2);
    }
    return 0;
}

/* ---- streams that come and go: the buffers that no caller asked for end ---- */

static int many_streams(void) {
    for (uintptr_t s = 1 << 12; s < 600 << 12; s += 1 << 12) {
        CHECK(merge((void *)s) == 0);
        CHECK(tiles(3000, 300, (void *)s) == 0);
    }
    CHECK(mallocs <= 128);
    CHECK(malloc_bytes <= 64 << 20);
    CHECK(last_lds > 0);                    /* without a workspace: in LDS */
    const int before = mallocs;
    CHECK(merge((void *)(uintptr_t)(1 << 12)) == 0 && last_lds == 0);   /* the first keeps its own */
    CHECK(tiles(2048, 256, (void *)(uintptr_t)(700 << 12)) == 0);       /* a prepared split always has one */
    CHECK(mallocs == before + 1 && iqa_last_hip_error() == 0);
    return 0;
}

/* ---- iqa_prepare stands for the shape, wherever its images lie ---- */

static int prepared(void) {
    int refused = 0;
    uintptr_t stream = 1 << 12;
    for (int64_t NT = 4; NT <= 4096; ++NT) {
        for (int64_t ns = 1; ns <= 32 && ns * NT <= 16384; ++ns, stream += 1 << 12) {
            void *s = (void *)stream;
            CHECK(iqa_prepare(ns * NT, NT, NULL, s) == 0);
            capturing = s;
            for (int off = 0; off < 4; ++off) {
                const int st = tiles_at(X + off, ns * NT, NT, NULL, s);
                if (st != 0 && refused++ < 5)
                    printf("%d/%d off %d: %s\n", (int)(ns * NT), (int)NT, off, iqa_status_str(st));
            }
            capturing = NULL;
        }
    }
    printf("%d refused\n", refused);
    CHECK(captured_mallocs == 0 && refused == 0);
    return 0;
}

/* ---- every size the library documents can be launched ---- */

static int sizes(void) {
    /* 2^17 pixels a side in the smallest tiles that were ever launched */
    CHECK(tiles(1 << 17, 4, NULL) == 0);
    for (int64_t NT = 6; NT <= 64; ++NT) {
        const int64_t N = (1 << 17) / NT * NT;
        if (NT != 7 && tiles(N, NT, NULL) != 0) {
            printf("%d/%d refused\n", (int)N, (int)NT);
            return 1;
        }
    }
    return 0;
}

/* ---- batches of any number of units ---- */

static int many_units(void) {
    const int64_t units[] = {1, 7, 8, 9, 1 << 20, (1 << 24) - 1, 1 << 24, (1 << 24) + 9, (int64_t)1 << 40};
    for (unsigned i = 0; i < sizeof units / sizeof *units; ++i) {
        CHECK(iqa_odd_tiles_batched(X, 1, units[i], NULL) == 0);
        CHECK(units[i] > 1 << 23 || last_items / 256 == (units[i] < 8 ? units[i] : (units[i] + 7) / 8 * 8));
        CHECK(iqa_tiles_batched(X, 1, units[i], (int64_t)1 << 32, NULL) == 0);
    }
    return 0;
}

/* ---- the default configuration, asked for and passed back ---- */

static int passed_back(void) {
    int splits = 0;
    uintptr_t stream = 1 << 12;
    for (int64_t NT = 100; NT <= 2048; NT += 25) {
        for (int64_t ns = 1; ns <= 16; ++ns, stream += 1 << 12) {
            void *s = (void *)stream;
            iqa_launch_cfg c;
            CHECK(iqa_default_cfg(ns * NT, NT, X, Y, &c) == 0);
            capturing = s;
            const int by_rule = tiles_at(X, ns * NT, NT, NULL, s), before = launches;
            const uint64_t items = last_items;
            const int back = tiles_at(X, ns * NT, NT, &c, s);
            capturing = NULL;
            CHECK(back == by_rule);
            if (by_rule == 0) CHECK(launches == before + 1 && last_items == items);
            splits += c.ksplit > 1 && by_rule == 0;
        }
    }
    CHECK(splits > 100 && captured_mallocs == 0);
    /* Prepared with that configuration it is captured as it is launched. */
    iqa_launch_cfg c;
    void *s = (void *)stream;
    CHECK(iqa_default_cfg(3000, 300, X, Y, &c) == 0 && c.ksplit > 1);
    CHECK(tiles_at(X, 3000, 300, &c, s) == 0 && last_lds == 0);
    const uint64_t split_items = last_items;
    capturing = s;
    CHECK(tiles_at(X, 3000, 300, &c, s) == 0 && last_lds > 0);
    capturing = NULL;
    CHECK(iqa_prepare(3000, 300, &c, s) == 0);
    capturing = s;
    CHECK(tiles_at(X, 3000, 300, &c, s) == 0 && last_lds == 0 && last_items == split_items);
    CHECK(tiles_at(X, 3000, 300, NULL, s) == 0 && last_lds > 0);
    CHECK(iqa_tiles_noalloc(X, Y, 3000, 300, 5e-7f, 1e-6f, 1e-6f, 1e-6f, OUT, OUT2, NULL, &c, s) == 0);
    CHECK(last_lds > 0);
    return 0;
}

/* ---- a pyramid takes the levels that the chain of merges takes ---- */

static int pyramid_sizes(void) {
    float *out[17];
    for (int i = 0; i < 17; ++i) out[i] = OUT;
    for (int64_t ns = 2; ns <= 1 << 17; ns += ns < 90000 ? 2 * (1 + ns / 64) : 2) {
        const int one = iqa_merge_tiles(X, ns, 2, 5e-7f, 1e-6f, 1e-6f, OUT, OUT2, OUT, NULL);
        const int st = iqa_pyramid(X, ns, 1, 5e-7f, 1e-6f, 1e-6f, out, out, out, NULL);
        if (st != one) {
            printf("%d: %s, and %s\n", (int)ns, iqa_status_str(st), iqa_status_str(one));
            return 1;
        }
    }
    CHECK(iqa_pyramid(X, 1 << 17, 17, 5e-7f, 1e-6f, 1e-6f, out, out, out, NULL) == IQA_ERR_SHAPE);
    CHECK(iqa_pyramid(X, 1 << 16, 16, 5e-7f, 1e-6f, 1e-6f, out, out, out, NULL) == IQA_OK);
    return 0;
}

int main(int argc, char **argv) {
    const char *name = argc > 1 ? argv[1] : "";
    if (!strcmp(name, "per_thread")) return per_thread();
    if (!strcmp(name, "many_streams")) return many_streams();
    if (!strcmp(name, "prepared")) return prepared();
    if (!strcmp(name, "sizes")) return sizes();
    if (!strcmp(name, "many_units")) return many_units();
    if (!strcmp(name, "passed_back")) return passed_back();
    if (!strcmp(name, "pyramid_sizes")) return pyramid_sizes();
    printf("no scenario %s\n", name);
    return 2;
}
