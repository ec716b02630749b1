/* A HIP runtime without a device, for tests of the library's host code on the
 * CPU: loaded with RTLD_GLOBAL before liblanczos_topk.so, its definitions take
 * the place of the runtime's.  Kernels do nothing, copies to the host deliver
 * zeros, and allocations are counted against fake_capacity bytes:
 *   - a block freed stream-ordered into a pool is idle until its stream is
 *     waited for ("pending") and stays the pool's until the pool is trimmed;
 *     the default pool gives a block back as soon as it is idle and waited for;
 *   - idle blocks of a pool serve that pool alone, whole, and pending ones
 *     their own stream alone. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <pthread.h>

enum { OK = 0, INVALID = 1, NOMEM = 2 };
enum { BLOCKS = 4096, POOLS = 8, RANGES = 16 };

typedef struct { int device; } Pool;
typedef struct { void* p; size_t bytes; int pool; int idle; void* pending; } Block;     /* pool -1: default, -2: hipMalloc */

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static Block blocks[BLOCKS];
static Pool pools[POOLS];
static int npools, current_device, last_error, capturing;
static size_t capacity = (size_t)1 << 40, used, lagging;
static int lag, lag_left;
static struct { char* base; size_t bytes; } pinned[RANGES];
static int npinned;
static long count_host_malloc, count_host_live, count_h2d_pinned, count_launch, count_pool_alloc_other_device;

void fake_capacity(size_t bytes) { capacity = bytes; }
/* Trimmed memory comes free only after this many further failed allocations. */
void fake_lag(int attempts) { lag = attempts; }
size_t fake_used(void) { return used; }
size_t fake_idle(void) {
    size_t s = 0;
    for (int i = 0; i < BLOCKS; ++i)
        if (blocks[i].p && blocks[i].idle) s += blocks[i].bytes;
    return s;
}
void fake_device(int d) { current_device = d; }
void fake_capturing(int on) { capturing = on; }
void fake_pin(void* base, size_t bytes) { pinned[npinned].base = base; pinned[npinned++].bytes = bytes; }
long fake_count(int what) {
    return what == 0   ? count_host_malloc
           : what == 1 ? count_host_live
           : what == 2 ? count_h2d_pinned
           : what == 3 ? count_launch
                       : count_pool_alloc_other_device;
}

/* A stream is null, hipStreamLegacy (1) or hipStreamPerThread (2), the current
 * device's, or has 1 + its device in the low byte. */
static int stream_device(void* s) { return (uintptr_t)s > 2 ? (int)((uintptr_t)s & 255) - 1 : current_device; }
static int fail(int e) { return last_error = e; }
static void drop(Block* b) {
    used -= b->bytes;
    free(b->p);
    memset(b, 0, sizeof(*b));
}
static int take(void** out, size_t bytes, int pool, void* stream) {
    pthread_mutex_lock(&mu);
    Block* slot = NULL;
    for (int i = 0; i < BLOCKS; ++i) {
        Block* b = &blocks[i];
        if (b->p && b->idle && b->pool == pool && b->bytes >= bytes &&
            (!b->pending || b->pending == (stream ? stream : (void*)-1))) {
            b->idle = 0;
            b->pending = NULL;
            *out = b->p;
            pthread_mutex_unlock(&mu);
            return OK;
        }
        if (!b->p && !slot) slot = b;
    }
    int rc = OK;
    if (lagging && lag_left == 0) lagging = 0;
    if (!slot || used + lagging + bytes > capacity) {
        if (lagging) --lag_left;
        rc = fail(NOMEM);
    } else {
        used += bytes;
        slot->p = malloc(1);
        slot->bytes = bytes;
        slot->pool = pool;
        slot->idle = 0;
        *out = slot->p;
    }
    pthread_mutex_unlock(&mu);
    return rc;
}
static Block* find(void* p) {
    for (int i = 0; i < BLOCKS; ++i)
        if (p && blocks[i].p == p) return &blocks[i];
    return NULL;
}

int hipGetDevice(int* d) { *d = current_device; return OK; }
int hipSetDevice(int d) { current_device = d; return OK; }
int hipGetStreamDeviceId(void* s) {
    if ((uintptr_t)s == 1 || (uintptr_t)s == 2) abort();   /* as the runtime, which follows the handle */
    return stream_device(s);
}
int hipGetLastError(void) { int e = last_error; last_error = OK; return e; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = capturing; return OK; }
int hipMalloc(void** p, size_t bytes) { return take(p, bytes, -2, NULL); }
int hipFree(void* p) {
    pthread_mutex_lock(&mu);
    Block* b = find(p);
    if (b) drop(b);
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipMallocAsync(void** p, size_t bytes, void* s) { return take(p, bytes, -1, s); }
int hipMemPoolCreate(void** pool, const int* props) {      /* props: type, handle types, location type, id */
    pools[npools].device = props[3];
    *pool = &pools[npools++];
    return OK;
}
int hipMemPoolSetAttribute(void* pool, int attr, void* value) { (void)pool; (void)attr; (void)value; return OK; }
int hipMemPoolGetAttribute(void* pool, int attr, void* value) {
    uint64_t s = 0;
    pthread_mutex_lock(&mu);
    for (int i = 0; i < BLOCKS; ++i)
        if (blocks[i].p && blocks[i].pool == (int)((Pool*)pool - pools)) s += blocks[i].bytes;
    pthread_mutex_unlock(&mu);
    *(uint64_t*)value = s;
    return attr == 5 ? OK : fail(INVALID);                 /* hipMemPoolAttrReservedMemCurrent */
}
int hipMemPoolDestroy(void* pool) { (void)pool; return OK; }
int hipMallocFromPoolAsync(void** p, size_t bytes, void* pool, void* s) {
    if (((Pool*)pool)->device != stream_device(s)) ++count_pool_alloc_other_device;
    return take(p, bytes, (int)((Pool*)pool - pools), s);
}
int hipFreeAsync(void* p, void* s) {
    pthread_mutex_lock(&mu);
    Block* b = find(p);
    if (b) {
        b->idle = 1;
        b->pending = s ? s : (void*)-1;
    }
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipStreamSynchronize(void* s) {
    pthread_mutex_lock(&mu);
    for (int i = 0; i < BLOCKS; ++i) {
        Block* b = &blocks[i];
        if (!b->p || !b->idle || b->pending != (s ? s : (void*)-1)) continue;
        b->pending = NULL;
        if (b->pool == -1) drop(b);
    }
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipMemPoolTrimTo(void* pool, size_t keep) {
    (void)keep;
    pthread_mutex_lock(&mu);
    for (int i = 0; i < BLOCKS; ++i) {
        Block* b = &blocks[i];
        if (!b->p || !b->idle || b->pending || b->pool != (int)((Pool*)pool - pools)) continue;
        if (lag) {
            lagging += b->bytes;
            lag_left = lag;
        }
        drop(b);
    }
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
    (void)flags;
    pthread_mutex_lock(&mu);
    ++count_host_malloc;
    ++count_host_live;
    pthread_mutex_unlock(&mu);
    *p = calloc(1, bytes);
    return OK;
}
int hipHostFree(void* p) {
    pthread_mutex_lock(&mu);
    --count_host_live;
    pthread_mutex_unlock(&mu);
    free(p);
    return OK;
}
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int kind, void* s) {
    (void)s;
    if (kind == 2) memset(dst, 0, bytes);
    if (kind == 1)
        for (int i = 0; i < npinned; ++i)
            if ((const char*)src >= pinned[i].base && (const char*)src < pinned[i].base + pinned[i].bytes) {
                ++count_h2d_pinned;
                if ((const char*)src + bytes > pinned[i].base + pinned[i].bytes) return fail(INVALID);
            }
    return OK;
}
int hipMemcpyWithStream(void* dst, const void* src, size_t bytes, int kind, void* s) {
    return hipMemcpyAsync(dst, src, bytes, kind, s);
}
/* Pinned host memory: addressed by the device where the host addresses it. */
int hipHostGetDevicePointer(void** d, void* h, unsigned flags) { (void)flags; *d = h; return OK; }
int hipMemGetAddressRange(void** base, size_t* bytes, void* p) {
    for (int i = 0; i < npinned; ++i)
        if ((char*)p >= pinned[i].base && (char*)p < pinned[i].base + pinned[i].bytes) {
            *base = pinned[i].base;
            *bytes = pinned[i].bytes;
            return OK;
        }
    return fail(INVALID);
}
int hipPointerGetAttributes(int* at, const void* p) {
    void* base;
    size_t bytes;
    if (hipMemGetAddressRange(&base, &bytes, (void*)p) != OK) return INVALID;
    at[0] = 1;                                             /* hipMemoryTypeHost */
    return OK;
}
int hipLaunchKernel(const void* f, uint64_t a, uint32_t b, uint64_t c, uint32_t d, void** args, size_t lds, void* s) {
    (void)f; (void)a; (void)b; (void)c; (void)d; (void)args; (void)lds; (void)s;
    pthread_mutex_lock(&mu);
    ++count_launch;
    pthread_mutex_unlock(&mu);
    return OK;
}
int __hipPushCallConfiguration(uint64_t a, uint32_t b, uint64_t c, uint32_t d, size_t lds, void* s) {
    (void)a; (void)b; (void)c; (void)d; (void)lds; (void)s;
    return OK;
}
int __hipPopCallConfiguration(void* g, void* b, size_t* lds, void** s) { (void)g; (void)b; *lds = 0; *s = NULL; return OK; }
int hipStreamCreateWithFlags(void** s, unsigned f) {
    (void)f;
    static uintptr_t next;
    *s = (void*)((++next << 8) + 1 + (uintptr_t)current_device);
    return OK;
}
int hipStreamDestroy(void* s) { (void)s; return OK; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return OK; }
int hipEventCreate(void** e) { *e = (void*)1; return OK; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = (void*)1; return OK; }
int hipEventDestroy(void* e) { (void)e; return OK; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return OK; }
int hipEventSynchronize(void* e) { (void)e; return OK; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.0f; return OK; }
