/* hipMalloc and hipFree with failures on demand and a limit on the live bytes,
 * a count of calls from threads that chose no device, and failures of events, for tests/test_gpu_memory.py: loaded with RTLD_GLOBAL before libtc.so, so that
 * the library's calls come here first.  Every call that is not refused goes to
 * the HIP runtime. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <pthread.h>
#include <stddef.h>
#include <stdint.h>

enum { kOutOfMemory = 2 }; /* hipErrorOutOfMemory */
enum { kMax = 1 << 16 };

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static struct { void* p; size_t bytes; } live_blocks[kMax];
static int blocks;
static uint64_t live, peak, limit = UINT64_MAX;
static long fail_from = -1, calls, refused;

static void count_unchosen(void);

static void* real(const char* name) {
    void* h = dlopen("libamdhip64.so.7", RTLD_NOW);
    return h ? dlsym(h, name) : NULL;
}

int hipMalloc(void** out, size_t bytes) {
    int (*f)(void**, size_t) = (int (*)(void**, size_t))real("hipMalloc");
    count_unchosen();
    pthread_mutex_lock(&mu);
    int rc = kOutOfMemory;
    const long k = calls++;
    if (f && !(fail_from >= 0 && k >= fail_from) && live + bytes <= limit && blocks < kMax) rc = f(out, bytes);
    else ++refused;
    if (rc == 0) {
        live_blocks[blocks].p = *out;
        live_blocks[blocks++].bytes = bytes;
        live += bytes;
        if (live > peak) peak = live;
    }
    pthread_mutex_unlock(&mu);
    return rc;
}

int hipFree(void* p) {
    int (*f)(void*) = (int (*)(void*))real("hipFree");
    pthread_mutex_lock(&mu);
    for (int k = 0; k < blocks; ++k)
        if (live_blocks[k].p == p) {
            live -= live_blocks[k].bytes;
            live_blocks[k] = live_blocks[--blocks];
            break;
        }
    pthread_mutex_unlock(&mu);
    return f ? f(p) : 1;
}

/* Calls that the device of the calling thread decides, from threads that never chose one. */
static __thread int chosen;
static long unchosen;

static void count_unchosen(void) {
    if (!chosen) __atomic_add_fetch(&unchosen, 1, __ATOMIC_SEQ_CST);
}

int hipSetDevice(int device) {
    int (*f)(int) = (int (*)(int))real("hipSetDevice");
    chosen = 1;
    return f ? f(device) : 1;
}

int hipStreamCreateWithFlags(void** out, unsigned flags) {
    int (*f)(void**, unsigned) = (int (*)(void**, unsigned))real("hipStreamCreateWithFlags");
    count_unchosen();
    return f ? f(out, flags) : 1;
}

long shim_unchosen(void) { return __atomic_load_n(&unchosen, __ATOMIC_SEQ_CST); }

/* Event records and waits: those from the k-th on fail (k < 0: none), and the
 * stream synchronisations since the first that failed are counted. */
static long fail_event = -1, event_calls, event_failed, syncs;

static int event_fails(void) {
    pthread_mutex_lock(&mu);
    const int f = fail_event >= 0 && event_calls++ >= fail_event;
    event_failed += f;
    pthread_mutex_unlock(&mu);
    return f;
}
int hipEventRecord(void* ev, void* stream) {
    int (*f)(void*, void*) = (int (*)(void*, void*))real("hipEventRecord");
    return !f || event_fails() ? 1 : f(ev, stream);
}
int hipStreamWaitEvent(void* stream, void* ev, unsigned flags) {
    int (*f)(void*, void*, unsigned) = (int (*)(void*, void*, unsigned))real("hipStreamWaitEvent");
    return !f || event_fails() ? 1 : f(stream, ev, flags);
}
int hipStreamSynchronize(void* stream) {
    int (*f)(void*) = (int (*)(void*))real("hipStreamSynchronize");
    pthread_mutex_lock(&mu);
    syncs += event_failed != 0;
    pthread_mutex_unlock(&mu);
    return f ? f(stream) : 1;
}
void shim_fail_events(long k) {
    pthread_mutex_lock(&mu);
    fail_event = k;
    event_calls = event_failed = syncs = 0;
    pthread_mutex_unlock(&mu);
}
long shim_events_failed(void) { return event_failed; }
long shim_syncs(void) { return syncs; }

/* The k-th call from now (0: the next) and all after it fail; k < 0: none. */
void shim_fail_from(long k) {
    pthread_mutex_lock(&mu);
    calls = 0;
    refused = 0;
    fail_from = k;
    pthread_mutex_unlock(&mu);
}
void shim_set_limit(uint64_t bytes) {
    pthread_mutex_lock(&mu);
    limit = bytes;
    refused = 0;
    pthread_mutex_unlock(&mu);
}
uint64_t shim_live(void) { return live; }
/* The most live bytes since the last call. */
uint64_t shim_peak(void) {
    pthread_mutex_lock(&mu);
    const uint64_t p = peak;
    peak = live;
    pthread_mutex_unlock(&mu);
    return p;
}
long shim_refused(void) { return refused; }
/* hipMalloc calls since the last shim_fail_from. */
long shim_calls(void) { return calls; }
