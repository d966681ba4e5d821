// pool.hip -- memory that a call needs only while it runs (the initial condition's
// spectral planes), kept for the next call of any context instead of being
// allocated and released each time.
//
// Allocating fresh device memory costs more than the allocation itself (the first
// pass over new pages): with a block of its own per call the initial condition and
// read-back of a 144^2 event took 1345 us against 1263 with the block kept, a 384^2
// one 6.69 ms against 6.30.  What is kept does not grow with the number of contexts: two
// idle blocks of at most 64 MiB, released with the last context.  Calls that run
// at the same time on several threads get blocks of their own.
#include <mutex>

#include "internal.h"

namespace cpic {
namespace {

constexpr int kIdle = 2;
struct Idle {
    PoolBlock b;
    int device = 0;
};
std::mutex g_lock;
Idle g_idle[kIdle];
int64_t g_users = 0;

}  // namespace

hipError_t pool_take(int device, size_t bytes, PoolBlock* out)
{
    {
        std::lock_guard<std::mutex> hold(g_lock);
        Idle* fit = nullptr;
        for (Idle& i : g_idle)
            if (i.b.p && i.device == device && i.b.bytes >= bytes && (!fit || i.b.bytes < fit->b.bytes)) fit = &i;
        if (fit) {
            *out = fit->b;
            *fit = Idle{};
            return hipSuccess;
        }
    }
    *out = PoolBlock{};
    const hipError_t e = hipMalloc(&out->p, bytes);
    if (e == hipSuccess) {
        out->bytes = bytes;
    } else {
        (void)hipGetLastError();  // reported by the caller, not by the next launch
        out->p = nullptr;
    }
    return e;
}

void pool_give(int device, PoolBlock b)
{
    if (!b.p) return;
    if (b.bytes <= kPoolBlockBytes) {
        std::lock_guard<std::mutex> hold(g_lock);
        // the larger blocks stay
        Idle* at = &g_idle[0];
        for (Idle& i : g_idle)
            if (i.b.bytes < at->b.bytes) at = &i;
        if (g_users > 0 && at->b.bytes < b.bytes) {
            const Idle gone = *at;
            *at = Idle{b, device};
            b = gone.b;
        }
    }
    (void)hipFree(b.p);
}

void pool_enter()
{
    std::lock_guard<std::mutex> hold(g_lock);
    g_users++;
}
void pool_leave()
{
    Idle gone[kIdle];
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (--g_users > 0) return;
        for (int k = 0; k < kIdle; k++) {
            gone[k] = g_idle[k];
            g_idle[k] = Idle{};
        }
    }
    for (const Idle& i : gone) (void)hipFree(i.b.p);
}

}  // namespace cpic
