/* A HIP runtime without a device, for host-side tests: memory is the host's,
 * copies are immediate, kernels do not run.  Counts device memory and can
 * refuse allocations; keeps the dynamic LDS limits that were set and used. */
#include <pthread.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { OK = 0, NO_MEMORY = 2, NOT_SUPPORTED = 801, MAXP = 1 << 16, MAXL = 1 << 12 };
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static void* ptr[MAXP];
static size_t len[MAXP], live, peak;
static size_t limit = SIZE_MAX; /* allocations that would pass it are refused */
static int sync_us;
typedef struct { const void* func; int64_t set, used; } lds_t;
static lds_t lds[MAXL];
static int nlds;

size_t fake_live(void) { return live; }
size_t fake_peak(void) { return peak; }
void fake_reset_peak(void) { peak = live; }
void fake_limit(size_t bytes) { limit = bytes; }
void fake_sync_us(int us) { sync_us = us; }
int fake_lds(int i, const void** func, int64_t* set, int64_t* used) {
    if (i >= nlds) return 0;
    *func = lds[i].func, *set = lds[i].set, *used = lds[i].used;
    return 1;
}

int hipMalloc(void** p, size_t n) {
    int i = 0, rc = NO_MEMORY;
    pthread_mutex_lock(&mu);
    *p = NULL;
    if (live + n <= limit) {
        while (i < MAXP && ptr[i]) i++;
        void* q = i < MAXP ? aligned_alloc(256, (n + 256) / 256 * 256) : NULL;
        if (q) {
            memset(q, 0, n);
            ptr[i] = *p = q, len[i] = n, live += n, rc = OK;
            if (live > peak) peak = live;
        }
    }
    pthread_mutex_unlock(&mu);
    return rc;
}
int hipFree(void* p) {
    pthread_mutex_lock(&mu);
    for (int i = 0; p && i < MAXP; i++)
        if (ptr[i] == p) {
            live -= len[i], ptr[i] = NULL;
            break;
        }
    pthread_mutex_unlock(&mu);
    free(p);
    return OK;
}
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return (*p = calloc(1, n)) ? OK : NO_MEMORY; }
int hipHostFree(void* p) { free(p); return OK; }
int hipHostGetDevicePointer(void** d, void* h, unsigned f) { (void)f; *d = h; return OK; }
int hipGetSymbolAddress(void** p, const void* s) { static char* z; (void)s; if (!z) z = calloc(1, 64 << 20); *p = z; return OK; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memmove(d, s, n); return OK; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)k, (void)st; memmove(d, s, n); return OK; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; memset(d, v, n); return OK; }
int hipMemGetInfo(size_t* f, size_t* t) { *f = *t = (size_t)64 << 30; return OK; }
int hipGetDeviceCount(int* n) { *n = 1; return OK; }
int hipGetDevice(int* d) { *d = 0; return OK; }
int hipSetDevice(int d) { (void)d; return OK; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a, (void)d; *v = 100000; return OK; }
int hipGetLastError(void) { return OK; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = malloc(1); return OK; }
int hipStreamDestroy(void* s) { free(s); return OK; }
int hipStreamSynchronize(void* s) { (void)s; if (sync_us) usleep((useconds_t)sync_us); return OK; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s, (void)e, (void)f; return OK; }
int hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; return NOT_SUPPORTED; }
int hipEventCreate(void** e) { *e = malloc(1); return OK; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = malloc(1); return OK; }
int hipEventDestroy(void* e) { free(e); return OK; }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return OK; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a, (void)b; *ms = 0; return OK; }

static __thread struct { dim3_t g, b; size_t shmem; void* st; } call;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t shmem, void* st) {
    call.g = g, call.b = b, call.shmem = shmem, call.st = st;
    return OK;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* shmem, void** st) {
    *g = call.g, *b = call.b, *shmem = call.shmem, *st = call.st;
    return OK;
}
static void note(const void* f, int64_t set, int64_t used) {
    pthread_mutex_lock(&mu);
    if (nlds < MAXL) lds[nlds++] = (lds_t){f, set, used};
    pthread_mutex_unlock(&mu);
}
int hipFuncSetAttribute(const void* f, int a, int v) { (void)a; note(f, v, -1); return OK; }
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t shmem, void* st) {
    (void)g, (void)b, (void)args, (void)st;
    if (shmem > 65536) note(f, -1, (int64_t)shmem);
    return OK;
}
