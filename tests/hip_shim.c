/* Stands between libcpic and the HIP runtime in a test's own process (loaded before
 * both, globally): counts some calls, fails chosen ones from the host, and
 * answers elapsed times and the current device from a script.  No call is made that the library did
 * not make, and no failed call reaches the GPU. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>

enum { MALLOC, HOST_MALLOC, GRAPH_LAUNCH, KERNEL, ELAPSED, N_CALLS };
static long calls[N_CALLS], fail_from[N_CALLS], fail_to[N_CALLS];
static size_t fail_bytes;          /* allocations below this many bytes succeed */
static float ms_before, ms_after;  /* elapsed times, before and from call ms_turn on */
static long ms_turn = -1;

/* calls number first .. last - 1 of a kind, counted from now, fail */
void shim_fail(int kind, long first, long last, size_t bytes)
{
    fail_from[kind] = calls[kind] + first;
    fail_to[kind] = calls[kind] + last;
    fail_bytes = bytes;
}
void shim_elapsed(float before, long turn, float after)
{
    ms_before = before;
    ms_turn = calls[ELAPSED] + turn;
    ms_after = after;
}
long shim_calls(int kind) { return calls[kind]; }
/* the device that hipGetDevice names, and the allocations made while it was not 0 */
static int device;
static long elsewhere;
void shim_set_device(int d) { device = d; }
int shim_device(void) { return device; }
long shim_elsewhere(void) { return elsewhere; }

static void* real(const char* name)
{
    static void* lib;
    if (!lib) lib = dlopen("libamdhip64.so.7", RTLD_LAZY);
    return lib ? dlsym(lib, name) : NULL;
}
static int failing(int kind)
{
    const long k = calls[kind]++;
    return k >= fail_from[kind] && k < fail_to[kind];
}

int hipGetDevice(int* d)
{
    *d = device;
    return 0;
}
int hipSetDevice(int d)
{
    device = d;
    return 0;
}
int hipMalloc(void** p, size_t bytes)
{
    if (device) elsewhere++;
    static int (*f)(void**, size_t);
    if (!f) f = (int (*)(void**, size_t))real("hipMalloc");
    if (bytes >= fail_bytes && failing(MALLOC)) return 2; /* hipErrorOutOfMemory */
    return f(p, bytes);
}
int hipHostMalloc(void** p, size_t bytes, unsigned flags)
{
    if (device) elsewhere++;
    static int (*f)(void**, size_t, unsigned);
    if (!f) f = (int (*)(void**, size_t, unsigned))real("hipHostMalloc");
    if (bytes >= fail_bytes && failing(HOST_MALLOC)) return 2;
    return f(p, bytes, flags);
}
int hipGraphLaunch(void* g, void* st)
{
    static int (*f)(void*, void*);
    if (!f) f = (int (*)(void*, void*))real("hipGraphLaunch");
    if (failing(GRAPH_LAUNCH)) return 999; /* hipErrorUnknown */
    return f(g, st);
}
typedef struct { unsigned x, y, z; } dim3_;
int hipLaunchKernel(const void* k, dim3_ grid, dim3_ block, void** args, size_t lds, void* st)
{
    static int (*f)(const void*, dim3_, dim3_, void**, size_t, void*);
    if (!f) f = (int (*)(const void*, dim3_, dim3_, void**, size_t, void*))real("hipLaunchKernel");
    calls[KERNEL]++;
    return f(k, grid, block, args, lds, st);
}
int hipEventElapsedTime(float* ms, void* a, void* b)
{
    static int (*f)(float*, void*, void*);
    if (!f) f = (int (*)(float*, void*, void*))real("hipEventElapsedTime");
    const int s = f(ms, a, b);
    const long k = calls[ELAPSED]++;
    if (s == 0 && ms_turn >= 0) *ms = k < ms_turn ? ms_before : ms_after;
    return s;
}
