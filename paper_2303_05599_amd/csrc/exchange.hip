// exchange.hip -- state exchange with caller host memory (cpic_get_state,
// cpic_set_state): the double-precision site-major interchange layout against
// the structure-of-arrays buffers of the device.
//
// The layouts are converted on the device, in chunks that pass through pinned
// host memory: a kernel gathers a chunk into interchange order, a copy brings
// it to a pinned buffer, and the host copies it to the caller's memory (or the
// other way round) while the next chunk is on its way.  The device's chunks lie in
// memory that is idle between steps (the field buffer set that does not hold the
// state, the scratch records), the pinned ones are shared by all contexts.  The caller's memory is
// pageable and often untouched, so its page faults bound a single host thread
// (about 12 GB/s); a few threads share the host copies.
// Measured (384^2, FP64, all four fields, 80 MB): get 23.0 -> 4.6 ms, of which the page
// faults of the caller's fresh arrays take most; set (216^2, 25 MB) 2.6 -> 1.2 ms.
// The conversion loops ran on one host thread over strided arrays before.  Chunks
// of 2 or 4 MB and eight threads were slower or equal.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <thread>

#include "ctx.h"
#include "internal.h"

using namespace cpic;

namespace {

constexpr size_t kChunkBytes = (size_t)8 << 20;
constexpr int kCopyThreads = 4;
constexpr size_t kThreadBytes = (size_t)1 << 20;  // least share of a copying thread
// up to this size the kernels reach the pinned memory themselves: one launch
// and one wait instead of a copy command between (64 KB get: 38 -> 21 us)
constexpr size_t kDirectBytes = (size_t)512 << 10;

// What a part of the state looks like: `width` doubles per element in the
// interchange layout, elements e = 0 .. count - 1.
enum Kind { kLinks3, kLinks2, kAlgebra, kSites, kRecords, kPtau };
struct Part {
    Kind kind;
    int width;       // doubles per element
    size_t count;    // elements
    int V;           // sites, or records
    int comps;       // kAlgebra: components
    const int* cell; // kRecords: [2][np]
    const int* inv;  // kRecords, kPtau: the record of every row
    double t, mhat;  // kPtau: the constraint at the current time
};

// interchange particle columns: x y eta px py peta Q1..Q8 cx cy deta ux0 uy0 pt0
// (-1, -2: the cell)
__device__ const int kRecordColumn[20] = {PX_, PY_, PETA_, PPX, PPY, PPETA, PQ0, PQ0 + 1, PQ0 + 2, PQ0 + 3, PQ0 + 4,
                                          PQ0 + 5, PQ0 + 6, PQ0 + 7, -1, -2, PDETA, PUX0, PUY0, PPT0};

// p^tau from the constraint, evaluated without contraction
__device__ __forceinline__ double ptau_of(double px, double py, double pe, double t, double mhat)
{
#pragma clang fp contract(off)
    const double a = px * px, b = py * py, c = (t * pe) * (t * pe), d = mhat * mhat;
    return sqrt(a + b + c + d);
}

// entry k of the third row of a link from its first two (interchange order:
// entries 0..11 the rows r1, r2 as re, im), conj(r1 x r2), without contraction
template <typename T> __device__ __forceinline__ double third_row(const T* u, size_t V, size_t s, int k)
{
#pragma clang fp contract(off)
    const int j = (k - 12) / 2, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
    auto at = [&](int c) { return (double)u[(size_t)c * V + s]; };
    const double are = at(2 * j1), aim = at(2 * j1 + 1), bre = at(6 + 2 * j2), bim = at(7 + 2 * j2);
    const double ere = at(2 * j2), eim = at(2 * j2 + 1), fre = at(6 + 2 * j1), fim = at(7 + 2 * j1);
    if (((k - 12) & 1) == 0) {
        const double p = are * bre - aim * bim, q = ere * fre - eim * fim;
        return p - q;
    }
    const double p = are * bim + aim * bre, q = ere * fim + eim * fre;
    return q - p;
}

// entry k of element e in interchange order
template <typename T> __device__ __forceinline__ double interchange(const Part& p, const T* src, size_t e, int k)
{
    const size_t V = p.V;
    switch (p.kind) {
    case kLinks3: {
        const size_t i = e / V, s = e - i * V;
        const T* u = src + i * 18 * V;
        return k < 12 ? (double)u[(size_t)k * V + s] : third_row(u, V, s, k);
    }
    case kLinks2: {
        // quaternion (w, a1, a2, a3) as [[w + i a3, a2 + i a1], [-a2 + i a1, w - i a3]]
        const size_t i = e / V, s = e - i * V;
        const int c = k == 0 || k == 6 ? 0 : (k == 3 || k == 5 ? 1 : (k == 2 || k == 4 ? 2 : 3));
        const double v = (double)src[(i * 4 + c) * V + s];
        return k == 4 || k == 7 ? -v : v;
    }
    case kAlgebra: {
        const size_t i = e / V, s = e - i * V;
        return (double)src[(i * p.comps + k) * V + s];
    }
    case kSites: return (double)src[(size_t)k * V + e];
    case kRecords: {
        const size_t r = p.inv[e];
        const int col = kRecordColumn[k];
        return col >= 0 ? (double)src[(size_t)col * V + r] : (double)p.cell[(size_t)(-col - 1) * V + r];
    }
    default: {
        const size_t r = p.inv[e];
        if (k == 1) return (double)src[(size_t)PPTAU * V + r];
        return ptau_of(src[(size_t)PPX * V + r], src[(size_t)PPY * V + r], src[(size_t)PPETA * V + r], p.t, p.mhat);
    }
    }
}
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(Part p, const T* __restrict__ src, double* __restrict__ dst,
                                                   size_t first, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * p.width) return;
    const size_t e = i / p.width;
    dst[i] = interchange(p, src, first + e, (int)(i - e * p.width));
}

// elements first .. first + n - 1 from interchange order; the threads of a
// wavefront take neighbouring elements (coalesced stores)
template <typename T>
__global__ __launch_bounds__(256) void unpack_kernel(Part p, const double* __restrict__ src, T* __restrict__ dst,
                                                     int* __restrict__ cell, size_t first, size_t n, int comps)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * comps) return;
    const size_t k = i / n, j = i - k * n, e = first + j, V = p.V;
    const double* h = src + j * p.width;
    switch (p.kind) {
    case kLinks3: dst[(e / V * 18 + k) * V + e % V] = (T)h[k]; break;
    case kLinks2: dst[(e / V * 4 + k) * V + e % V] = (T)h[k == 0 ? 0 : (k == 1 ? 3 : (k == 2 ? 2 : 1))]; break;
    case kAlgebra: dst[(e / V * p.comps + k) * V + e % V] = (T)h[k]; break;
    default:
        if (k == 20) {
            dst[(size_t)PPTAU * V + e] = (T)ptau_of(h[3], h[4], h[5], p.t, p.mhat);
        } else {
            const int col = kRecordColumn[k];
            if (col >= 0) dst[(size_t)col * V + e] = (T)h[k];
            else cell[(size_t)(-col - 1) * V + e] = (int)h[k];
        }
    }
}

__global__ void invert_kernel(const int* __restrict__ pid, int n, int* __restrict__ inv)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && pid[i] >= 0 && pid[i] < n) inv[pid[i]] = i;
}

// memcpy by a few threads; never throws (a thread that cannot be started does
// its share here)
void host_copy(void* dst, const void* src, size_t bytes)
{
    const size_t hw = std::max(1u, std::thread::hardware_concurrency());
    const size_t nt = std::max<size_t>(1, std::min<size_t>({(size_t)kCopyThreads, hw, bytes / kThreadBytes}));
    std::thread th[kCopyThreads];
    const size_t share = (bytes / nt + 4095) / 4096 * 4096;
    auto part = [=](size_t k) {
        const size_t a = std::min(bytes, k * share), b = k + 1 == nt ? bytes : std::min(bytes, (k + 1) * share);
        if (b > a) std::memcpy(static_cast<char*>(dst) + a, static_cast<const char*>(src) + a, b - a);
    };
    for (size_t k = 1; k < nt; k++) {
        try {
            th[k] = std::thread(part, k);
        } catch (...) {
            part(k);
        }
    }
    part(0);
    for (size_t k = 1; k < nt; k++)
        if (th[k].joinable()) th[k].join();
}

// the part's description, its array on the device, and the components an unpack writes
template <typename T> bool describe(const cpic_ctx* c, int which, Part* p, T** array, int* comps)
{
    const size_t V = c->V;
    const bool su2 = c->nc == 2;
    T* f = static_cast<T*>(c->fbuf[c->cur]);
    *p = Part{};
    p->V = c->V;
    p->t = c->n * c->sc.dt;
    p->mhat = c->mhat;
    auto algebra = [&](size_t at, int blocks) {
        p->kind = kAlgebra;
        p->comps = p->width = *comps = su2 ? 3 : 8;
        p->count = blocks * V;
        *array = f + at * V;
    };
    switch (which) {
    case CPIC_STATE_U:
        p->kind = su2 ? kLinks2 : kLinks3;
        p->width = su2 ? 8 : 18;
        *comps = su2 ? 4 : 18;
        p->count = 2 * V;
        *array = f;
        return true;
    case CPIC_STATE_PHI: algebra(su2 ? 8 : 36, 1); return true;
    case CPIC_STATE_E: algebra(su2 ? 11 : 44, 2); return true;
    case CPIC_STATE_PI: algebra(su2 ? 17 : 60, 1); return true;
    case CPIC_STATE_JET_W:
    case CPIC_STATE_JET_F:
        p->kind = kSites;
        p->width = which == CPIC_STATE_JET_W ? 18 : 24;
        p->count = V;
        *array = static_cast<T*>(which == CPIC_STATE_JET_W ? c->jW : c->jF);
        return true;
    case CPIC_STATE_PARTICLES:
    case CPIC_STATE_PTAU:
        p->kind = which == CPIC_STATE_PTAU ? kPtau : kRecords;
        p->width = which == CPIC_STATE_PTAU ? 2 : 20;
        *comps = 21;  // and p^tau
        p->count = (size_t)c->np;
        p->V = (int)c->np;
        p->cell = c->pcell;
        p->inv = c->sb.perm;
        *array = static_cast<T*>(c->pr);
        return true;
    default: return false;
    }
}

// The chunks of one call, two on each side: on the device in the buffer set that does
// not hold the state or, for particles, in the scratch records where those are
// larger (both idle between steps); pinned from the pool.
struct Staging {
    cpic_ctx* c;
    OnDevice on;
    PoolPins pins{};
    double* dev[2] = {nullptr, nullptr};
    size_t bytes = 0;
    bool done = false;  // the stream is idle
    explicit Staging(cpic_ctx* ctx) : c(ctx), on(ctx) {}
    Staging(const Staging&) = delete;
    hipError_t open(bool particles, size_t total)
    {
        char* base = static_cast<char*>(c->fbuf[next_buffer(c->cur)]);
        size_t room = (size_t)c->rps * c->V * c->tsz;
        const size_t records = (size_t)kPartReals * (size_t)c->np * c->tsz;
        if (particles && records > room) {
            base = static_cast<char*>(c->sb.r2);
            room = records;
        }
        // (half of it on a 256-byte boundary; up to kDirectBytes no device chunk is used)
        bytes = std::min(total, kChunkBytes);
        if (total > kDirectBytes) bytes = std::min(bytes, room / 512 * 256);
        dev[0] = reinterpret_cast<double*>(base);
        dev[1] = reinterpret_cast<double*>(base + room / 512 * 256);
        return pool_take_pins(c->device, bytes, &pins);
    }
    hipError_t finish()
    {
        const hipError_t e = hipStreamSynchronize(c->st);
        done = e == hipSuccess;
        return done ? hipGetLastError() : e;
    }
    ~Staging()
    {
        // after an error part way a chunk may be in flight; pinned memory that cannot be waited for is left
        if (pins.bytes && (done || hipStreamSynchronize(c->st) == hipSuccess)) pool_give_pins(c->device, pins);
    }
};

template <typename T> hipError_t get_part(cpic_ctx* c, int which, double* host)
{
    Part p;
    T* src = nullptr;
    int comps = 0;
    if (!describe<T>(c, which, &p, &src, &comps)) return hipErrorInvalidValue;
    if (p.kind == kRecords || p.kind == kPtau)
        hipLaunchKernelGGL(invert_kernel, dim3((p.V + 255) / 256), dim3(256), 0, c->st, c->pid, p.V, c->sb.perm);
    const size_t total = p.count * p.width * sizeof(double);
    Staging x(c);
    hipError_t e = x.open(p.kind == kRecords || p.kind == kPtau, total);
    if (e != hipSuccess) return e;
    if (total <= kDirectBytes) {
        hipLaunchKernelGGL(pack_kernel<T>, dim3((unsigned)((p.count * p.width + 255) / 256)), dim3(256), 0, c->st, p, src,
                           static_cast<double*>(x.pins.pin[0]), (size_t)0, p.count);
        e = x.finish();
        if (e == hipSuccess) std::memcpy(host, x.pins.pin[0], total);
        return e;
    }
    const size_t per = std::max<size_t>(1, x.bytes / (p.width * sizeof(double)));
    const size_t chunks = (p.count + per - 1) / per;
    auto range = [&](size_t k, size_t* first, size_t* n) {
        *first = k * per;
        *n = std::min(per, p.count - k * per);
    };
    size_t first, n;
    for (size_t k = 0; k <= chunks; k++) {
        if (k < chunks) {
            // chunk k on its way (the pinned buffer's last chunk, k - 2, has been copied out)
            range(k, &first, &n);
            const int b = (int)(k & 1);
            hipLaunchKernelGGL(pack_kernel<T>, dim3((unsigned)((n * p.width + 255) / 256)), dim3(256), 0, c->st, p, src,
                               x.dev[b], first, n);
            e = hipMemcpyAsync(x.pins.pin[b], x.dev[b], n * p.width * sizeof(double), hipMemcpyDeviceToHost, c->st);
            if (e == hipSuccess) e = hipEventRecord(x.pins.ev[b], c->st);
            if (e != hipSuccess) return e;
        }
        if (k > 0) {
            range(k - 1, &first, &n);
            const int b = (int)((k - 1) & 1);
            e = hipEventSynchronize(x.pins.ev[b]);
            if (e != hipSuccess) return e;
            host_copy(host + first * p.width, x.pins.pin[b], n * p.width * sizeof(double));
        }
    }
    x.done = true;  // the last chunk's event was the stream's last work
    return hipGetLastError();
}

template <typename T> hipError_t set_part(cpic_ctx* c, int which, const double* host)
{
    Part p;
    T* dst = nullptr;
    int comps = 0;
    if (!describe<T>(c, which, &p, &dst, &comps)) return hipErrorInvalidValue;
    const size_t total = p.count * p.width * sizeof(double);
    Staging x(c);
    hipError_t e = x.open(p.kind == kRecords || p.kind == kPtau, total);
    if (e != hipSuccess) return e;
    if (total <= kDirectBytes) {
        std::memcpy(x.pins.pin[0], host, total);
        hipLaunchKernelGGL(unpack_kernel<T>, dim3((unsigned)((p.count * comps + 255) / 256)), dim3(256), 0, c->st, p,
                           static_cast<const double*>(x.pins.pin[0]), dst, c->pcell, (size_t)0, p.count, comps);
        return x.finish();
    }
    const size_t per = std::max<size_t>(1, x.bytes / (p.width * sizeof(double)));
    for (size_t k = 0, first = 0; first < p.count; k++, first += per) {
        const size_t n = std::min(per, p.count - first);
        const int b = (int)(k & 1);
        // (the copy that last read this pinned buffer, two chunks ago, is over)
        if (k >= 2) e = hipEventSynchronize(x.pins.ev[b]);
        if (e != hipSuccess) return e;
        host_copy(x.pins.pin[b], host + first * p.width, n * p.width * sizeof(double));
        e = hipMemcpyAsync(x.dev[b], x.pins.pin[b], n * p.width * sizeof(double), hipMemcpyHostToDevice, c->st);
        if (e == hipSuccess) e = hipEventRecord(x.pins.ev[b], c->st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(unpack_kernel<T>, dim3((unsigned)((n * comps + 255) / 256)), dim3(256), 0, c->st, p,
                           x.dev[b], dst, c->pcell, first, n, comps);
    }
    return x.finish();
}

}  // namespace

hipError_t cpic::exchange_get(cpic_ctx* c, int which, double* host)
{
    return c->prec == CPIC_FP64 ? get_part<double>(c, which, host) : get_part<float>(c, which, host);
}
hipError_t cpic::exchange_set(cpic_ctx* c, int which, const double* host)
{
    return c->prec == CPIC_FP64 ? set_part<double>(c, which, host) : set_part<float>(c, which, host);
}
