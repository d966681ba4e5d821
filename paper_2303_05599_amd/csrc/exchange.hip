// exchange.hip -- state exchange with caller host memory (cpic_get_state,
// cpic_set_state): the double-precision site-major interchange layout against
// the structure-of-arrays buffers of the device.
//
// A part passes through pinned host memory in chunks, and the host moves a chunk
// between there and the caller's memory while the next one is on its way.  The
// caller's memory is pageable and often untouched, so its page faults bound a
// single host thread (about 12 GB/s); a few threads share the host's work.  The layouts
// are converted on the side where that moves less:
//   rows     the device's component arrays cross the link as they are, and the host
//            converts while it copies: the algebra elements, the quaternions, the
//            light-like paths, and (reading) the links of single-precision runs, half or
//            a quarter of whose interchange form they are;
//   packed   a kernel converts and reaches the pinned memory itself: the links in
//            double precision, whose third rows it rebuilds, the particle records,
//            which come in another order, and what else fills several chunks in double
//            precision (E of 512^2, set: 810 us, by rows 910).
// One launch or copy command and one wait for a part of one chunk: what small parts cost.
// Measured into and out of memory in use, one host thread over pageable copies -> every part
// packed -> this: phi of 48^2 in FP64, set 16 -> 35 -> 13 us; pi of 96^2 in FP32, get 29 -> 54 -> 22,
// set 26 -> 43 -> 21; links of 48^2 in FP32, get 36 -> 58 -> 33; SU(2) links of 128^2 in FP32, get 53
// -> 146 -> 42, set 45 -> 99 -> 39; links of 384^2 in FP64 (42 MB), get 11.7 -> 1.08 -> 0.99 ms, set 19.8
// -> 1.10 -> 0.99; 18662 records, get 790 -> 184 -> 140 us, set 324 -> 248 -> 211.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <thread>
#include <type_traits>

#include "ctx.h"
#include "internal.h"

using namespace cpic;

namespace {

constexpr size_t kChunkBytes = (size_t)8 << 20;  // (2 or 4 MB, and eight threads, were slower or equal)
// a copy command and its wait take 8 us from here on, 12 up to 16 KiB, a kernel's launch and wait 12
constexpr size_t kCopyBytes = ((size_t)16 << 10) + 1;
// links installed by rows up to this size of their interchange form (16^2, FP64: 13 us, by a
// kernel 19; 27^2: equal)
constexpr size_t kFewLinks = (size_t)192 << 10;
constexpr int kCopyThreads = 4;
constexpr size_t kThreadBytes = (size_t)1 << 20;  // least share of a copying thread

// What a part of the state looks like: `width` doubles per element in the
// interchange layout, elements e = 0 .. count - 1.
enum Kind { kLinks3, kLinks2, kAlgebra, kSites, kRecords, kPtau };
struct Part {
    Kind kind;
    int width;       // doubles per element
    size_t count;    // elements
    int V;           // sites, or records
    int blocks;      // times V elements (directions, or 1)
    int stride;      // components per block on the device
    int comps;       // of them in the interchange form
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

// entry k of the third row of a link from the entries 0..11 of its first two (rows r1, r2
// as re, im): conj(r1 x r2), without contraction, the same bits on either side
template <typename At> __host__ __device__ __forceinline__ double third_row(int k, At at)
{
#pragma clang fp contract(off)
    const int j = (k - 12) / 2, j1 = (j + 1) % 3, j2 = (j + 2) % 3;
    const double are = at(2 * j1), aim = at(2 * j1 + 1), bre = at(6 + 2 * j2), bim = at(7 + 2 * j2);
    const double ere = at(2 * j2), eim = at(2 * j2 + 1), fre = at(6 + 2 * j1), fim = at(7 + 2 * j1);
    if (((k - 12) & 1) == 0) {
        const double p = are * bre - aim * bim, q = ere * fre - eim * fim;
        return p - q;
    }
    const double p = are * bim + aim * bre, q = ere * fim + eim * fre;
    return q - p;
}

// ---- packed parts (all but kLinks2)
// entry k of element e in interchange order
template <typename T> __device__ __forceinline__ double interchange(const Part& p, const T* src, size_t e, int k)
{
    const size_t V = p.V;
    if (p.kind == kLinks3) {
        const size_t i = e / V, s = e - i * V;
        const T* u = src + i * 18 * V + s;
        return k < 12 ? (double)u[(size_t)k * V] : third_row(k, [&](int c) { return (double)u[(size_t)c * V]; });
    }
    if (p.kind == kAlgebra || p.kind == kSites) {
        const size_t i = e / V, s = e - i * V;
        return (double)src[(i * p.stride + k) * V + s];
    }
    const size_t r = p.inv[e];
    if (p.kind == kRecords) {
        const int col = kRecordColumn[k];
        return col >= 0 ? (double)src[(size_t)col * V + r] : (double)p.cell[(size_t)(-col - 1) * V + r];
    }
    if (k == 1) return (double)src[(size_t)PPTAU * V + r];
    return ptau_of(src[(size_t)PPX * V + r], src[(size_t)PPY * V + r], src[(size_t)PPETA * V + r], p.t, p.mhat);
}
// dst: pinned
template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(Part p, const T* __restrict__ src, double* __restrict__ dst,
                                                   size_t first, size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * p.width) return;
    const size_t e = i / p.width;
    dst[i] = interchange(p, src, first + e, (int)(i - e * p.width));
}

// Elements first .. first + n - 1 from interchange order in pinned memory (kLinks3,
// kAlgebra, kRecords): a workgroup reads 64 elements whole, each line of the link once, and
// writes them component by component out of LDS.
constexpr int kUnpackWidth = 20;
template <typename T>
__global__ __launch_bounds__(256) void unpack_kernel(Part p, const double* __restrict__ src, T* __restrict__ dst,
                                                     int* __restrict__ cell, size_t first, size_t n)
{
    __shared__ double lds[64 * (kUnpackWidth + 1)];
    const size_t e0 = (size_t)blockIdx.x * 64, V = p.V;
    const int W = p.width, ne = (int)min((size_t)64, n - e0);
    for (int i = threadIdx.x; i < ne * W; i += 256) lds[i / W * (W + 1) + i % W] = src[e0 * W + i];
    __syncthreads();
    const int j = (int)threadIdx.x & 63;
    if (j >= ne) return;
    const size_t e = first + e0 + j;
    const double* h = lds + j * (W + 1);
    if (p.kind != kRecords) {
        T* const u = dst + e / V * p.stride * V + e % V;
        for (int k = (int)threadIdx.x >> 6; k < p.stride; k += 4) u[(size_t)k * V] = (T)h[k];
        return;
    }
    for (int k = (int)threadIdx.x >> 6; k < 21; k += 4) {
        if (k == 20) {
            dst[(size_t)PPTAU * V + e] = (T)ptau_of(h[3], h[4], h[5], p.t, p.mhat);
        } else {
            const int col = kRecordColumn[k];
            if (col >= 0) dst[(size_t)col * V + e] = (T)h[k];
            else cell[(size_t)(-col - 1) * V + e] = (int)h[k];
        }
    }
}

// ---- parts by rows
// Sites first .. first + n - 1 of every row (block, component) between the device's
// arrays and rows of `ld` entries in pinned memory.
template <typename T, bool GET>
__global__ __launch_bounds__(256) void rows_kernel(T* dev, T* pin, int V, int rows, int comps, int stride, int first,
                                                   int n, int ld)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)rows * n) return;
    const int r = (int)(i / n), s = (int)(i - (size_t)r * n);
    T* const d = dev + ((size_t)(r / comps) * stride + r % comps) * V + first + s;
    T* const h = pin + (size_t)r * ld + s;
    if (GET) *h = *d;
    else *d = *h;
}
// sites a .. b - 1 of one block: rows d (of ld entries) to interchange order at h, and back
template <typename T, int C> void algebra_to_host(const T* d, size_t ld, double* h, size_t a, size_t b)
{
    for (size_t s = a; s < b; s++)
#pragma unroll
        for (int k = 0; k < C; k++) h[s * C + k] = (double)d[k * ld + s];
}
template <typename T, int C> void algebra_from_host(T* d, size_t ld, const double* h, size_t a, size_t b)
{
    for (size_t s = a; s < b; s++)
#pragma unroll
        for (int k = 0; k < C; k++) d[k * ld + s] = (T)h[s * C + k];
}
template <typename T> void rows_to_host(const Part& p, const T* d, size_t ld, double* h, size_t a, size_t b)
{
    switch (p.kind) {
    case kAlgebra:
        if (p.comps == 8) algebra_to_host<T, 8>(d, ld, h, a, b);
        else algebra_to_host<T, 3>(d, ld, h, a, b);
        break;
    case kLinks2:  // quaternion (w, x, y, z) as [[w + i z, y + i x], [-y + i x, w - i z]]
        for (size_t s = a; s < b; s++) {
            const double w = d[s], x = d[ld + s], y = d[2 * ld + s], z = d[3 * ld + s];
            double* const o = h + 8 * s;
            o[0] = w; o[1] = z; o[2] = y; o[3] = x;
            o[4] = -y; o[5] = x; o[6] = w; o[7] = -z;
        }
        break;
    case kLinks3:
        for (size_t s = a; s < b; s++) {
            double* const u = h + 18 * s;
#pragma unroll
            for (int k = 0; k < 12; k++) u[k] = (double)d[k * ld + s];
            auto entry = [&](auto k) { u[decltype(k)::value] = third_row(decltype(k)::value, [&](int c) { return u[c]; }); };
            entry(std::integral_constant<int, 12>{}); entry(std::integral_constant<int, 13>{});
            entry(std::integral_constant<int, 14>{}); entry(std::integral_constant<int, 15>{});
            entry(std::integral_constant<int, 16>{}); entry(std::integral_constant<int, 17>{});
        }
        break;
    default:
        if (p.comps == 18) algebra_to_host<T, 18>(d, ld, h, a, b);
        else algebra_to_host<T, 24>(d, ld, h, a, b);
    }
}
template <typename T> void rows_from_host(const Part& p, T* d, size_t ld, const double* h, size_t a, size_t b)
{
    if (p.kind == kLinks2) {
        for (size_t s = a; s < b; s++) {
            const double* const o = h + 8 * s;
            d[s] = (T)o[0];
            d[ld + s] = (T)o[3];
            d[2 * ld + s] = (T)o[2];
            d[3 * ld + s] = (T)o[1];
        }
    } else if (p.comps == 8) {
        algebra_from_host<T, 8>(d, ld, h, a, b);
    } else if (p.comps == 18) {
        algebra_from_host<T, 18>(d, ld, h, a, b);
    } else {
        algebra_from_host<T, 3>(d, ld, h, a, b);
    }
}

__global__ void invert_kernel(const int* __restrict__ pid, int n, int* __restrict__ inv)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && pid[i] >= 0 && pid[i] < n) inv[pid[i]] = i;
}

// f(begin, end) over 0 .. n - 1 by a few threads, a share of at least kThreadBytes of
// `bytes` each, in multiples of `unit`; never throws (a thread that cannot be started does its share here)
template <typename F> void shared_work(size_t n, size_t bytes, size_t unit, F f)
{
    size_t nt = std::min((size_t)kCopyThreads, bytes / kThreadBytes);
    if (nt <= 1) return f((size_t)0, n);
    nt = std::min<size_t>(nt, std::max(1u, std::thread::hardware_concurrency()));  // (reads a file: 2 us)
    std::thread th[kCopyThreads];
    const size_t share = (n / nt + unit) / unit * unit;
    auto part = [=](size_t k) {
        const size_t a = std::min(n, k * share), b = std::min(n, (k + 1) * share);
        if (b > a) f(a, b);
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
void host_copy(void* dst, const void* src, size_t bytes)
{
    shared_work(bytes, bytes, 4096, [=](size_t a, size_t b) {
        std::memcpy(static_cast<char*>(dst) + a, static_cast<const char*>(src) + a, b - a);
    });
}

// the part's description and its array on the device
template <typename T> bool describe(const cpic_ctx* c, int which, Part* p, T** array)
{
    const size_t V = c->V;
    const bool su2 = c->nc == 2;
    T* f = static_cast<T*>(c->fbuf[c->cur]);
    *p = Part{};
    p->V = c->V;
    p->t = c->n * c->sc.dt;
    p->mhat = c->mhat;
    auto sites = [&](Kind kind, T* at, int blocks, int stride, int comps, int width) {
        p->kind = kind;
        p->blocks = blocks;
        p->stride = stride;
        p->comps = comps;
        p->width = width;
        p->count = blocks * V;
        *array = at;
        return true;
    };
    const int A = su2 ? 3 : 8;
    switch (which) {
    case CPIC_STATE_U: return su2 ? sites(kLinks2, f, 2, 4, 4, 8) : sites(kLinks3, f, 2, 18, 12, 18);
    case CPIC_STATE_PHI: return sites(kAlgebra, f + (su2 ? 8 : 36) * V, 1, A, A, A);
    case CPIC_STATE_E: return sites(kAlgebra, f + (su2 ? 11 : 44) * V, 2, A, A, A);
    case CPIC_STATE_PI: return sites(kAlgebra, f + (su2 ? 17 : 60) * V, 1, A, A, A);
    case CPIC_STATE_JET_W: return sites(kSites, static_cast<T*>(c->jW), 1, 18, 18, 18);
    case CPIC_STATE_JET_F: return sites(kSites, static_cast<T*>(c->jF), 1, 24, 24, 24);
    case CPIC_STATE_PARTICLES:
    case CPIC_STATE_PTAU:
        p->kind = which == CPIC_STATE_PTAU ? kPtau : kRecords;
        p->width = which == CPIC_STATE_PTAU ? 2 : 20;
        p->count = (size_t)c->np;
        p->V = (int)c->np;
        p->cell = c->pcell;
        p->inv = c->sb.perm;
        *array = static_cast<T*>(c->pr);
        return true;
    default: return false;
    }
}

// the pinned chunks of one call
struct Staging {
    cpic_ctx* c;
    OnDevice on;
    PoolPins pins{};
    bool done = false;  // the stream is idle
    explicit Staging(cpic_ctx* ctx) : c(ctx), on(ctx) {}
    Staging(const Staging&) = delete;
    hipError_t open(size_t total) { return pool_take_pins(c->device, std::min(total, kChunkBytes), &pins); }
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

// A part of `count` elements in chunks of `per`: device(k, b, first, n) enqueues chunk k's
// device work on pinned buffer b, host(b, first, n) is the host's share of it.  Reading, the
// host's share comes after the device's, and the device is a chunk ahead; installing, before.
template <typename D, typename H> hipError_t read_chunks(Staging& x, size_t count, size_t per, D device, H host)
{
    const size_t chunks = (count + per - 1) / per;
    for (size_t k = 0; k <= chunks; k++) {
        if (k < chunks) {
            // (the pinned buffer's last chunk, k - 2, has been copied out)
            const int b = (int)(k & 1);
            hipError_t e = device(b, k * per, std::min(per, count - k * per));
            if (e == hipSuccess && chunks > 1) e = hipEventRecord(x.pins.ev[b], x.c->st);
            if (e != hipSuccess) return e;
        }
        if (k > 0) {
            const int b = (int)((k - 1) & 1);
            const hipError_t e = chunks > 1 ? hipEventSynchronize(x.pins.ev[b]) : x.finish();
            if (e != hipSuccess) return e;
            host(b, (k - 1) * per, std::min(per, count - (k - 1) * per));
        }
    }
    x.done = true;  // the last chunk was the stream's last work
    return hipGetLastError();
}
template <typename D, typename H> hipError_t install_chunks(Staging& x, size_t count, size_t per, D device, H host)
{
    for (size_t k = 0; k * per < count; k++) {
        const int b = (int)(k & 1);
        const size_t first = k * per, n = std::min(per, count - first);
        // (the work that last read this pinned buffer, two chunks ago, is over)
        hipError_t e = k >= 2 ? hipEventSynchronize(x.pins.ev[b]) : hipSuccess;
        if (e != hipSuccess) return e;
        host(b, first, n);
        e = device(b, first, n);
        if (e == hipSuccess && first + n < count) e = hipEventRecord(x.pins.ev[b], x.c->st);
        if (e != hipSuccess) return e;
    }
    return x.finish();
}

// Parts by rows: chunks of sites, all rows of a chunk side by side.  A part of one
// chunk lies in the pinned memory as on the device and goes by one copy command
// (the smallest by a kernel, and components a multiple of a page apart).  Not by the
// synchronous copy, which fails while another thread of the process captures a stream.
template <typename T, bool GET, typename H> hipError_t row_part(cpic_ctx* c, const Part& p, T* dev, H* host)
{
    const int rows = p.blocks * p.comps;
    const size_t V = p.V, all = ((size_t)(p.blocks - 1) * p.stride + p.comps) * V * sizeof(T);
    // (not where many rows of a copy would share the sets of the host's caches)
    const bool one = all <= kChunkBytes - ((size_t)64 << 10);
    const bool copied = one && all >= kCopyBytes && (p.comps <= 8 || V * sizeof(T) % 4096 != 0);
    Staging x(c);
    // rows of a chunk start 64 bytes further into their page than the one before: equal
    // offsets would share the sets of the host's caches
    const size_t pad = 64 / sizeof(T), per = one ? V : (kChunkBytes / rows / sizeof(T) - pad) / 1024 * 1024;
    const size_t ld = copied ? V : per + pad, block = (copied ? p.stride : p.comps) * ld;
    const hipError_t e = x.open(copied ? all : rows * ld * sizeof(T));
    if (e != hipSuccess) return e;
    auto device = [&](int b, size_t first, size_t n) {
        T* const pin = static_cast<T*>(x.pins.pin[b]);
        if (copied)
            return GET ? hipMemcpyAsync(pin, dev, all, hipMemcpyDeviceToHost, c->st)
                       : hipMemcpyAsync(dev, pin, all, hipMemcpyHostToDevice, c->st);
        hipLaunchKernelGGL((rows_kernel<T, GET>), dim3((unsigned)((rows * n + 255) / 256)), dim3(256), 0, c->st, dev,
                           pin, p.V, rows, p.comps, p.stride, (int)first, (int)n, (int)ld);
        return hipSuccess;
    };
    auto convert = [&](int b, size_t first, size_t n) {
        T* const pin = static_cast<T*>(x.pins.pin[b]);
        // the sites of all blocks in one go, a thread's share from one or two of them
        // (reading takes fewer threads: they may all be touching the caller's pages first)
        const size_t bytes = p.blocks * n * p.comps * (GET ? 5 : 8);
        shared_work(p.blocks * n, bytes, 64, [=, &p](size_t begin, size_t end) {
            for (size_t i = begin / n; i * n < end; i++) {
                const size_t s0 = std::max(begin, i * n) - i * n, s1 = std::min(end, (i + 1) * n) - i * n;
                H* const h = host + (i * V + first) * p.width;
                if constexpr (GET) rows_to_host<T>(p, pin + i * block, ld, h, s0, s1);
                else rows_from_host<T>(p, pin + i * block, ld, h, s0, s1);
            }
        });
    };
    return GET ? read_chunks(x, V, per, device, convert) : install_chunks(x, V, per, device, convert);
}

// whether a part crosses by rows (links when they are read)
template <typename T> bool by_rows(const Part& p)
{
    switch (p.kind) {
    case kRecords: case kPtau: return false;
    case kLinks3: return sizeof(T) == 4;
    case kLinks2: return true;
    default: return sizeof(T) == 4 || p.count * p.width * sizeof(double) <= kChunkBytes;
    }
}

template <typename T> hipError_t get_part(cpic_ctx* c, int which, double* host)
{
    Part p;
    T* src = nullptr;
    if (!describe<T>(c, which, &p, &src)) return hipErrorInvalidValue;
    if (by_rows<T>(p)) return row_part<T, true>(c, p, src, host);
    if (p.kind == kRecords || p.kind == kPtau)
        hipLaunchKernelGGL(invert_kernel, dim3((p.V + 255) / 256), dim3(256), 0, c->st, c->pid, p.V, c->sb.perm);
    const size_t element = p.width * sizeof(double);
    Staging x(c);
    const hipError_t e = x.open(p.count * element);
    if (e != hipSuccess) return e;
    return read_chunks(
        x, p.count, std::max<size_t>(1, kChunkBytes / element),
        [&](int b, size_t first, size_t n) {
            hipLaunchKernelGGL(pack_kernel<T>, dim3((unsigned)((n * p.width + 255) / 256)), dim3(256), 0, c->st, p, src,
                               static_cast<double*>(x.pins.pin[b]), first, n);
            return hipSuccess;
        },
        [&](int b, size_t first, size_t n) { host_copy(host + first * p.width, x.pins.pin[b], n * element); });
}

template <typename T> hipError_t set_part(cpic_ctx* c, int which, const double* host)
{
    Part p;
    T* dst = nullptr;
    if (!describe<T>(c, which, &p, &dst)) return hipErrorInvalidValue;
    const size_t element = p.width * sizeof(double);
    if (p.kind == kLinks3 && p.count * element <= kFewLinks) {
        p.comps = p.stride;  // the third rows too
        return row_part<T, false>(c, p, dst, host);
    }
    if (p.kind != kLinks3 && by_rows<T>(p)) return row_part<T, false>(c, p, dst, host);
    Staging x(c);
    const hipError_t e = x.open(p.count * element);
    if (e != hipSuccess) return e;
    return install_chunks(
        x, p.count, std::max<size_t>(1, kChunkBytes / element),
        [&](int b, size_t first, size_t n) {
            hipLaunchKernelGGL(unpack_kernel<T>, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, c->st, p,
                               static_cast<const double*>(x.pins.pin[b]), dst, c->pcell, first, n);
            return hipSuccess;
        },
        [&](int b, size_t first, size_t n) { host_copy(x.pins.pin[b], host + first * p.width, n * element); });
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
