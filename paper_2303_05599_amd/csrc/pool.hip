// pool.hip -- memory that a call needs only while it runs (the initial condition's
// spectral planes, the state exchange's pinned chunks), kept for the next call of
// any context instead of being allocated and released each time.
//
// Allocating fresh device memory costs more than the allocation itself (the first
// pass over new pages): with a block of its own per call the initial condition and
// read-back of a 144^2 event took 1345 us against 1263 with the block kept, a 384^2
// one 6.69 ms against 6.30.  One block serves a call: releasing one takes about 0.3 ms,
// whatever its size (four of 36 MiB: 0.82 ms, one of 144: 0.34).  What is kept does not
// grow with the number of contexts: two idle blocks of 256 MiB together and two idle
// pairs of pinned chunks (of 8 MiB at most), released with the last context.  Calls
// that run at the same time on several threads get memory of their own.
#include <mutex>
#include <utility>

#include "internal.h"

namespace cpic {
namespace {

constexpr int kIdle = 2;
template <typename B> struct Idle {
    B b;
    int device = 0;
};
std::mutex g_lock;
Idle<PoolBlock> g_idle[kIdle];
Idle<PoolPins> g_pins[kIdle];
int64_t g_users = 0;

// the smallest idle one that is large enough (under the lock)
template <typename B> bool find(Idle<B> (&idle)[kIdle], int device, size_t bytes, B* out)
{
    Idle<B>* fit = nullptr;
    for (Idle<B>& i : idle)
        if (i.b.bytes >= bytes && i.b.bytes > 0 && i.device == device && (!fit || i.b.bytes < fit->b.bytes)) fit = &i;
    if (!fit) return false;
    *out = fit->b;
    *fit = Idle<B>{};
    return true;
}
// the larger ones stay, up to `most` bytes together; returns what is to be released
template <typename B> B keep(Idle<B> (&idle)[kIdle], int device, const B& b, size_t most)
{
    std::lock_guard<std::mutex> hold(g_lock);
    Idle<B>* at = &idle[0];
    size_t others = 0;
    for (Idle<B>& i : idle) {
        others += i.b.bytes;
        if (i.b.bytes < at->b.bytes) at = &i;
    }
    if (g_users <= 0 || at->b.bytes >= b.bytes || others - at->b.bytes + b.bytes > most) return b;
    const B gone = at->b;
    *at = Idle<B>{b, device};
    return gone;
}
void release(const PoolPins& p)
{
    for (int k = 0; k < 2; k++) {
        if (p.pin[k]) (void)hipHostFree(p.pin[k]);
        if (p.ev[k]) (void)hipEventDestroy(p.ev[k]);
    }
}

}  // namespace

hipError_t pool_take(int device, size_t bytes, PoolBlock* out)
{
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (find(g_idle, device, bytes, out)) return hipSuccess;
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
    if (b.p) b = keep(g_idle, device, b, kPoolBytes);
    (void)hipFree(b.p);
}

hipError_t pool_take_pins(int device, size_t bytes, PoolPins* out)
{
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (find(g_pins, device, bytes, out)) return hipSuccess;
    }
    PoolPins p{};
    p.bytes = (bytes + 65535) / 65536 * 65536;
    hipError_t e = hipSuccess;
    for (int k = 0; k < 2 && e == hipSuccess; k++) {
        e = hipHostMalloc(&p.pin[k], p.bytes);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&p.ev[k], hipEventDisableTiming);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        release(p);
        p = PoolPins{};
    }
    *out = p;
    return e;
}
void pool_give_pins(int device, const PoolPins& p)
{
    release(keep(g_pins, device, p, SIZE_MAX));
}

void pool_enter()
{
    std::lock_guard<std::mutex> hold(g_lock);
    g_users++;
}
void pool_leave()
{
    Idle<PoolBlock> gone[kIdle];
    Idle<PoolPins> pins[kIdle];
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (--g_users > 0) return;
        std::swap(gone, g_idle);
        std::swap(pins, g_pins);
    }
    for (const auto& i : gone) (void)hipFree(i.b.p);
    for (const auto& i : pins) release(i.b);
}

}  // namespace cpic
