/* A device that does nothing, for tests of the library's host side: device
 * memory is host memory, copies are memcpy, kernels are not run, every event
 * has fired.  Preloaded in front of the HIP runtime.  FAKEHIP_FAIL=name:k makes
 * the k-th call of a function fail; fakehip_calls(name) counts its calls. */
#include <pthread.h>
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

enum { OK = 0, E_MEMORY = 2, E_UNKNOWN = 999 };

static struct { const char* name; int calls; } table[32];
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;

static int* counter(const char* name)
{
    for (int k = 0; k < 32; ++k) {
        if (!table[k].name)
            table[k].name = name;
        if (!strcmp(table[k].name, name))
            return &table[k].calls;
    }
    return NULL;
}

int fakehip_calls(const char* name)
{
    pthread_mutex_lock(&mu);
    const int k = *counter(strdup(name));
    pthread_mutex_unlock(&mu);
    return k;
}

static int call(const char* name)
{
    pthread_mutex_lock(&mu);
    const int k = ++*counter(name);
    pthread_mutex_unlock(&mu);
    const char* fail = getenv("FAKEHIP_FAIL");
    const size_t n = strlen(name);
    return fail && !strncmp(fail, name, n) && fail[n] == ':' && atoi(fail + n + 1) == k ? E_UNKNOWN : OK;
}

static int give(const char* name, void** p, size_t n)
{
    const int e = call(name);
    *p = e ? NULL : malloc(n);
    return e ? e : *p ? OK : E_MEMORY;
}

int hipGetDevice(int* d) { *d = 0; return call("hipGetDevice"); }
int hipSetDevice(int d) { (void)d; return call("hipSetDevice"); }
int hipMemGetInfo(size_t* f, size_t* t) { *f = *t = (size_t)1 << 40; return call("hipMemGetInfo"); }
int hipMalloc(void** p, size_t n) { return give("hipMalloc", p, n); }
int hipFree(void* p) { free(p); return call("hipFree"); }
int hipHostMalloc(void** p, size_t n, unsigned flags) { (void)flags; return give("hipHostMalloc", p, n); }
int hipHostFree(void* p) { free(p); return call("hipHostFree"); }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return call("hipMemcpy"); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st)
{
    (void)kind, (void)st;
    memcpy(d, s, n);
    return call("hipMemcpyAsync");
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; memset(d, v, n); return call("hipMemsetAsync"); }
int hipStreamCreateWithFlags(void** s, unsigned flags) { (void)flags; return give("hipStreamCreateWithFlags", s, 1); }
int hipStreamDestroy(void* s) { free(s); return call("hipStreamDestroy"); }
int hipStreamSynchronize(void* s) { (void)s; return call("hipStreamSynchronize"); }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) { (void)s, (void)e, (void)flags; return call("hipStreamWaitEvent"); }
int hipEventCreate(void** e) { return give("hipEventCreate", e, 1); }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; return give("hipEventCreateWithFlags", e, 1); }
int hipEventDestroy(void* e) { free(e); return call("hipEventDestroy"); }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return call("hipEventRecord"); }
int hipEventQuery(void* e) { (void)e; return call("hipEventQuery"); }
int hipEventSynchronize(void* e) { (void)e; return call("hipEventSynchronize"); }
int hipLaunchKernel(void) { return call("hipLaunchKernel"); }
int hipGetLastError(void) { return OK; }
