// ic.hip -- MV-model initial condition on the GPU (Sec. II, II.A) and the
// test-particle initial conditions (Sec. III.B, IV.B).  Always double
// precision; a float run rounds the finished values.
//
//   rows      Gaussian colour charges per sheet from Philox4x64-10 and their
//             transform along x, of which only the columns below the UV cut
//             are stored
//   columns   transform along y, times 1/(khat^2 + m^2) with the zero mode and
//             the modes above the UV cut removed, and back along y
//   Wilson    the inverse transform along x and, without storing alpha,
//             V^+(x) <- V^+(x) exp(-i alpha_n(x)), sheets in order
//   links     U^X_i(x) = V(x) V(x+i)^+, then the tau = 0 Glasma links from the
//             lattice initial condition, solved per link by Newton's method
//   pi(0)     from U, U^A, U^B
// The transforms are mixed-radix (8, 4, 2, 3) Stockham FFTs in LDS.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "philox.h"
#include "su2.h"
#include "su3.h"

namespace cpic {

using d2 = double2;

// ------------------------------------------------------------------ FFT
// Stages of a length-N transform, largest radix first.
struct Radices {
    int n;
    int r[10];
};
static Radices radices_of(int N)
{
    Radices R{};
    while (N % 8 == 0) { R.r[R.n++] = 8; N /= 8; }
    while (N % 4 == 0) { R.r[R.n++] = 4; N /= 4; }
    while (N % 2 == 0) { R.r[R.n++] = 2; N /= 2; }
    while (N % 3 == 0) { R.r[R.n++] = 3; N /= 3; }
    if (N != 1) R.n = -1;
    return R;
}
constexpr int kMaxFFT = 1024;

__device__ __forceinline__ d2 cm(d2 a, d2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ d2 ad(d2 a, d2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ d2 sb(d2 a, d2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ d2 mul_i(d2 a, double sg) { return make_double2(-sg * a.y, sg * a.x); }  // (sg i) a

// The radices packed four bits each, first stage lowest: the kernels read them
// from one register instead of indexing an array.
static unsigned radix_code(const Radices& R)
{
    unsigned c = 0;
    for (int s = R.n - 1; s >= 0; s--) c = (c << 4) | (unsigned)R.r[s];
    return c;
}
__device__ __forceinline__ int stage_radix(unsigned code, int stg) { return (int)((code >> (4 * stg)) & 15u); }

// One transform as the kernels take it: its stages and the twiddle table of
// its direction.  inv_r[s] = 1 / (N / R), inv_ns[s] = 1 / Ns of stage s, for the
// divisions of small integers by floating-point products.
struct Fft {
    const d2* tw;
    unsigned code;
    int n;
    float inv_r[7], inv_ns[7];
};
static Fft make_fft(const d2* tw, int N, const Radices& R)
{
    Fft f{};
    f.tw = tw;
    f.code = radix_code(R);
    f.n = R.n;
    int Ns = 1;
    for (int s = 0; s < R.n; s++) {
        f.inv_r[s] = 1.0f / (float)(N / R.r[s]);
        f.inv_ns[s] = 1.0f / (float)Ns;
        Ns *= R.r[s];
    }
    return f;
}
// LDS place of entry i: one entry of padding per eight.  The first stage's
// outputs lie R entries (R = 8: 128 bytes, all the banks once) apart from lane to
// lane; unpadded, every lane of a store would use the same banks.
__host__ __device__ constexpr int lds_at(int i) { return i + (i >> 3); }
// a / b for 0 <= a < 2^16 and inv = 1 / b in single precision: (a + 1/2) / b is
// at least 1 / (2 b) away from an integer, above the product's rounding error
__device__ __forceinline__ int small_div(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// The twiddle factors of every stage (R, Ns) of the Stockham FFT below,
// tw[(Ns - 1) + (q - 1) Ns + k] = exp(sign 2 pi i k q / (Ns R)) for k < Ns and
// 1 <= q < R: k fastest, so that the butterflies of a wavefront read
// consecutive entries.  The stages' entries follow one another without gaps,
// since the Ns of a stage is the product of the radices before it: N - 1 in all.
// Made once per initial condition, so that the butterflies read their factors
// instead of evaluating a sine and a cosine each.  Block 0 makes the table of
// the forward transforms and block 1 that of the inverse ones in the same stage
// order, block 2 that of the inverse in the opposite order.
__global__ void twiddle_kernel(d2* tw, int N, int nstages, unsigned rcode, unsigned rcode_back)
{
    const unsigned code = blockIdx.x == 2 ? rcode_back : rcode;
    const int sign = blockIdx.x == 0 ? -1 : 1;
    tw += (size_t)blockIdx.x * N;
    int Ns = 1;
    for (int stg = 0; stg < nstages; stg++) {
        const int R = stage_radix(code, stg);
        for (int t = threadIdx.x; t < Ns * (R - 1); t += blockDim.x) {
            const int k = t % Ns, q = t / Ns + 1;
            double sn, cs;
            sincospi((double)sign * 2.0 * (double)(k * q) / (double)(Ns * R), &sn, &cs);
            tw[Ns - 1 + t] = make_double2(cs, sn);
        }
        Ns *= R;
    }
}

// DFT of R values, sign sg
template <int R> __device__ __forceinline__ void dft(d2 (&v)[R], double sg)
{
    if constexpr (R == 2) {
        const d2 t = v[0];
        v[0] = ad(t, v[1]);
        v[1] = sb(t, v[1]);
    } else if constexpr (R == 3) {
        const d2 t = ad(v[1], v[2]);
        const d2 m = make_double2(v[0].x - 0.5 * t.x, v[0].y - 0.5 * t.y);
        const d2 dd = sb(v[1], v[2]);
        const d2 d = mul_i(make_double2(0.86602540378443864676 * dd.x, 0.86602540378443864676 * dd.y), sg);
        v[0] = ad(v[0], t);
        v[1] = ad(m, d);
        v[2] = sb(m, d);
    } else if constexpr (R == 4) {
        const d2 a = ad(v[0], v[2]), b = sb(v[0], v[2]), c = ad(v[1], v[3]), d = mul_i(sb(v[1], v[3]), sg);
        v[0] = ad(a, c);
        v[1] = ad(b, d);
        v[2] = sb(a, c);
        v[3] = sb(b, d);
    } else {
        static_assert(R == 8, "radix 2, 3, 4 or 8");
        d2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft<4>(e, sg);
        dft<4>(o, sg);
        constexpr double h = 0.70710678118654752440;
        // times exp(sg i pi q / 4)
        o[1] = make_double2(h * (o[1].x - sg * o[1].y), h * (o[1].y + sg * o[1].x));
        o[2] = mul_i(o[2], sg);
        o[3] = make_double2(h * (-o[3].x - sg * o[3].y), h * (-o[3].y + sg * o[3].x));
#pragma unroll
        for (int q = 0; q < 4; q++) {
            v[q] = ad(e[q], o[q]);
            v[q + 4] = sb(e[q], o[q]);
        }
    }
}

// One radix-R stage of the Stockham FFT on nb transforms: butterfly j < N / R
// takes the inputs j + q N / R, multiplies them by the twiddles of its k = j mod
// Ns, and writes the R outputs to (j - k) R + k + q Ns.  load(b, i) and
// store(b, i, value) reach entry i of transform b.  The threads take the
// butterflies with j fastest, or, with BFAST, the transform fastest (nb = 1 << bsh).
// A thread holds all its butterflies (about VALS values; nb N <= VALS blockDim)
// across a barrier between its loads and its stores, so one LDS buffer serves
// both; with VALS = 0 the stage goes from one buffer to another instead, which
// keeps fewer registers.  The stage ends with a barrier: every thread of the
// workgroup calls it.
template <int R, bool BFAST, int VALS, typename L, typename S, typename P>
__device__ __forceinline__ void fft_stage(int nb, int bsh, int N, int Ns, float inv_r, float inv_ns, double sg,
                                          const d2* __restrict__ tw, L load, S store, P mid)
{
    constexpr int M = VALS > 0 ? (VALS + R - 1) / R : 1;
    const int NR = N / R, total = nb * NR;
    if constexpr (VALS == 0) {
        for (int i = threadIdx.x; i < total; i += blockDim.x) {
            const int b = BFAST ? i & (nb - 1) : small_div(i, inv_r), j = BFAST ? i >> bsh : i - b * NR;
            const int k = Ns > 1 ? j - Ns * small_div(j, inv_ns) : 0;
            d2 v[R];
#pragma unroll
            for (int q = 0; q < R; q++) v[q] = load(b, j + q * NR);
            if (Ns > 1) {
                const d2* w = tw + (Ns - 1) + k;
#pragma unroll
                for (int q = 1; q < R; q++) v[q] = cm(v[q], w[(q - 1) * Ns]);
            }
            dft<R>(v, sg);
            const int base = (j - k) * R + k;
#pragma unroll
            for (int q = 0; q < R; q++) store(b, base + q * Ns, v[q]);
        }
        __syncthreads();
        return;
    }
    d2 v[M][R];
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int i = (int)threadIdx.x + m * (int)blockDim.x;
        if (i >= total) break;
        const int b = BFAST ? i & (nb - 1) : small_div(i, inv_r), j = BFAST ? i >> bsh : i - b * NR;
#pragma unroll
        for (int q = 0; q < R; q++) v[m][q] = load(b, j + q * NR);
        if (Ns > 1) {
            const d2* w = tw + (Ns - 1) + (j - Ns * small_div(j, inv_ns));
#pragma unroll
            for (int q = 1; q < R; q++) v[m][q] = cm(v[m][q], w[(q - 1) * Ns]);
        }
        dft<R>(v[m], sg);
        mid(b, j, v[m]);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; m++) {
        const int i = (int)threadIdx.x + m * (int)blockDim.x;
        if (i >= total) break;
        const int b = BFAST ? i & (nb - 1) : small_div(i, inv_r), j = BFAST ? i >> bsh : i - b * NR;
        const int k = Ns > 1 ? j - Ns * small_div(j, inv_ns) : 0, base = (j - k) * R + k;
#pragma unroll
        for (int q = 0; q < R; q++) store(b, base + q * Ns, v[m][q]);
    }
    __syncthreads();
}
template <bool BFAST = false, int VALS = 8, typename L, typename S>
__device__ __forceinline__ void fft_any(int R, int nb, int bsh, int N, int Ns, float inv_r, float inv_ns, double sg,
                                        const d2* __restrict__ tw, L load, S store)
{
    auto none = [](int, int, auto&) {};
    if (R == 8) fft_stage<8, BFAST, VALS>(nb, bsh, N, Ns, inv_r, inv_ns, sg, tw, load, store, none);
    else if (R == 4) fft_stage<4, BFAST, VALS>(nb, bsh, N, Ns, inv_r, inv_ns, sg, tw, load, store, none);
    else if (R == 2) fft_stage<2, BFAST, VALS>(nb, bsh, N, Ns, inv_r, inv_ns, sg, tw, load, store, none);
    else fft_stage<3, BFAST, VALS>(nb, bsh, N, Ns, inv_r, inv_ns, sg, tw, load, store, none);
}

// ------------------------------------------------------------------ Poisson
// The modes along x that the UV cut leaves: |k~| <= kc, nk = 2 kc + 1 columns
// (all N where nothing is cut), column c < nk holding k = c for c <= kc and
// k = N - nk + c above.  Spectral planes are [plane][y][nk].
struct Band {
    int nk, kc;
};
static Band band_of(int N, double uvhat)
{
    int kc = N / 2;
    if (uvhat > 0)
        while (kc > 0 && (2.0 * M_PI / N) * kc > uvhat) kc--;
    if (2 * kc + 1 >= N) return {N, N};
    return {2 * kc + 1, kc};
}
__host__ __device__ inline int column_mode(int c, int N, int nk, int kc) { return c <= kc ? c : N - nk + c; }

// K[c][k2] = 1/(khat^2 + m^2), khat^2 = 4 sum_i sin^2(pi k_i/N), of the stored columns;
// K = 0 at k = 0 and where the continuum |k| = (2 pi/N) |k~| exceeds the UV cut (k~ signed)
__global__ void poisson_kernel(double* K, int N, int nk, int kc, double mhat, double uvhat)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nk * N) return;
    const int k1 = column_mode(i / N, N, nk, kc), k2 = i % N;
    const double s1 = sinpi((double)k1 / N), s2 = sinpi((double)k2 / N);
    double v = 1.0 / (4.0 * (s1 * s1 + s2 * s2) + mhat * mhat);
    if (k1 == 0 && k2 == 0) v = 0.0;
    if (uvhat > 0) {
        const double q1 = k1 > N / 2 ? k1 - N : k1, q2 = k2 > N / 2 ? k2 - N : k2;
        if ((2.0 * M_PI / N) * sqrt(q1 * q1 + q2 * q2) > uvhat) v = 0.0;
    }
    K[i] = v;
}

// Charges and their transform along x.  Colours are paired: plane
// sheet * pairs + pair holds rho^{2 pair} + i rho^{2 pair + 1} of sheet sheet0 +
// sheet of nucleus `nucleus`; stream key (seed, 1 + nucleus), counter (s, sheet,
// block, 0), Philox block b giving the four normals of pairs 2b and 2b + 1
// (SU(3): blocks 0, 1; SU(2): block 0, whose fourth normal is unused).  A
// workgroup makes both pairs of one Philox block on RB rows in LDS and
// transforms the 2 RB rows there; only the kept columns go to memory.
// Bound: arithmetic (Philox, Box-Muller).  36 KB of LDS (RB N <= 1024 sites),
// four workgroups per CU.
__global__ __launch_bounds__(256) void rows_forward_kernel(d2* __restrict__ out, int N, int nk, int kc, uint64_t seed,
                                                           int nucleus, int sheet0, double sigma, int pairs, int RB,
                                                           Fft f)
{
    __shared__ d2 lds[lds_at(2 * 1024)];
    const int blocks = pairs / 2, sheet = (int)blockIdx.y / blocks, pb = (int)blockIdx.y - sheet * blocks;
    const int y0 = (int)blockIdx.x * RB, rows = min(RB, N - y0);
    for (int i = threadIdx.x; i < rows * N; i += blockDim.x) {
        const u64x4 r = philox4x64((uint64_t)(y0 * N + i), (uint64_t)(sheet0 + sheet), (uint64_t)pb, 0, seed,
                                   1 + (uint64_t)nucleus);
        double z[4];
        box_muller(r.v[0], r.v[1], z[0], z[1]);
        box_muller(r.v[2], r.v[3], z[2], z[3]);
        lds[lds_at(i)] = make_double2(sigma * z[0], sigma * z[1]);             // transforms 0 .. rows - 1: pair 2 pb
        lds[lds_at(rows * N + i)] = make_double2(sigma * z[2], sigma * z[3]);  // rows .. 2 rows - 1: pair 2 pb + 1
    }
    __syncthreads();
    d2* const plane = out + (size_t)(sheet * pairs + 2 * pb) * N * nk + (size_t)y0 * nk;
    int Ns = 1;
    auto load = [&](int t, int i) { return lds[lds_at(t * N + i)]; };
    auto keep = [&](int t, int i, d2 v) { lds[lds_at(t * N + i)] = v; };
    auto emit = [&](int t, int i, d2 v) {
        if (i > kc && i < N - nk + kc + 1) return;  // cut
        const int second = t >= rows, c = i <= kc ? i : i - (N - nk);
        plane[(size_t)second * N * nk + (size_t)(t - second * rows) * nk + c] = v;
    };
    for (int s = 0; s < f.n; s++) {
        const int R = stage_radix(f.code, s);
        if (s + 1 < f.n) fft_any(R, 2 * rows, 0, N, Ns, f.inv_r[s], f.inv_ns[s], -1.0, f.tw, load, keep);
        else fft_any(R, 2 * rows, 0, N, Ns, f.inv_r[s], f.inv_ns[s], -1.0, f.tw, load, emit);
        Ns *= R;
    }
}

// Transform along y, times K, and back, in place, for nb = 1 << bsh columns of
// one plane per workgroup (the columns past nk repeat the last one and store
// nothing).  The inverse runs its stages in the opposite order: its first stage
// takes the same R modes as the last forward stage produces, so the two and the
// multiplication between them need no exchange.  Memory is one read and one
// write of the kept columns.  f: the forward transform; g: the inverse.
template <int NT>
__global__ __launch_bounds__(NT) void columns_kernel(d2* __restrict__ data, int N, int nk, int bsh,
                                                     const double* __restrict__ Ktab, double scale, Fft f, Fft g)
{
    // nb N <= 8 NT entries, one of padding per column
    __shared__ d2 lds[lds_at(8 * NT + 32)];
    const int nb = 1 << bsh, ngroups = (nk + nb - 1) >> bsh;
    // consecutive column groups share lines: keep them on one XCD
    const int per = (ngroups + 7) / 8, grp = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (grp >= ngroups) return;
    const int c0 = grp << bsh, P = N + 1;
    d2* const plane = data + (size_t)blockIdx.y * N * nk + c0;
    const int last = nk - 1 - c0;  // the last column of the plane, from c0
    auto gload = [&](int b, int i) { return plane[(size_t)i * nk + min(b, last)]; };
    auto gstore = [&](int b, int i, d2 v) {
        if (b <= last) plane[(size_t)i * nk + b] = v;
    };
    auto lload = [&](int b, int i) { return lds[lds_at(b * P + i)]; };
    auto lstore = [&](int b, int i, d2 v) { lds[lds_at(b * P + i)] = v; };
    int Ns = 1;
    for (int s = 0; s + 1 < f.n; s++) {
        const int R = stage_radix(f.code, s);
        if (s == 0) fft_any<true>(R, nb, bsh, N, Ns, f.inv_r[s], f.inv_ns[s], -1.0, f.tw, gload, lstore);
        else fft_any<true>(R, nb, bsh, N, Ns, f.inv_r[s], f.inv_ns[s], -1.0, f.tw, lload, lstore);
        Ns *= R;
    }
    {
        // the last forward stage (k = j), K, and the first inverse stage, whose
        // output q of butterfly j is entry j R + q
        const int R = stage_radix(f.code, f.n - 1), s = f.n - 1;
        auto turn = [&](auto ld, auto st) {
            auto solve = [&](int b, int j, auto& v) {
                constexpr int RR = sizeof(v) / sizeof(d2);
                const double* K = Ktab + (size_t)(c0 + min(b, last)) * N + j;
#pragma unroll
                for (int q = 0; q < RR; q++) {
                    const double k = K[q * (N / RR)];
                    v[q] = make_double2(v[q].x * k * scale, v[q].y * k * scale);
                }
                dft<RR>(v, 1.0);
            };
            // outputs come as (j - k) R + k + q Ns = j + q Ns: back to j R + q
            auto flip = [&](auto RC) {
                constexpr int RR = decltype(RC)::value;
                auto st2 = [&](int b, int i, d2 v) {
                    const int q = small_div(i, f.inv_r[s]);
                    st(b, (i - q * (N / RR)) * RR + q, v);
                };
                fft_stage<RR, true, 8>(nb, bsh, N, Ns, f.inv_r[s], f.inv_ns[s], -1.0, f.tw, ld, st2, solve);
            };
            if (R == 8) flip(std::integral_constant<int, 8>{});
            else if (R == 4) flip(std::integral_constant<int, 4>{});
            else if (R == 2) flip(std::integral_constant<int, 2>{});
            else flip(std::integral_constant<int, 3>{});
        };
        if (f.n == 1) {
            turn(gload, gstore);  // N of one stage: every butterfly is a whole column
            return;
        }
        turn(lload, lstore);
        Ns = R;
    }
    for (int s = 1; s < g.n; s++) {
        const int R = stage_radix(g.code, s);
        if (s + 1 < g.n) fft_any<true>(R, nb, bsh, N, Ns, g.inv_r[s], g.inv_ns[s], 1.0, g.tw, lload, lstore);
        else fft_any<true>(R, nb, bsh, N, Ns, g.inv_r[s], g.inv_ns[s], 1.0, g.tw, lload, gstore);
        Ns *= R;
    }
}

// ------------------------------------------------------------------ Wilson lines
__device__ __forceinline__ m3<double> ldM(const double* p, int s, int V)
{
    m3<double> m;
    for (int c = 0; c < 9; c++) m.e[c] = {p[(size_t)(2 * c) * V + s], p[(size_t)(2 * c + 1) * V + s]};
    return m;
}
__device__ __forceinline__ void stM(double* p, int s, int V, const m3<double>& m)
{
    for (int c = 0; c < 9; c++) {
        p[(size_t)(2 * c) * V + s] = m.e[c].re;
        p[(size_t)(2 * c + 1) * V + s] = m.e[c].im;
    }
}

// SU(2): V^+ as quaternions [4][V]
__device__ __forceinline__ q4<double> ldQ(const double* p, int s, int V)
{
    return {p[s], p[(size_t)V + s], p[2 * (size_t)V + s], p[3 * (size_t)V + s]};
}
__device__ __forceinline__ void stQ(double* p, int s, int V, const q4<double>& q)
{
    p[s] = q.w;
    p[(size_t)V + s] = q.x;
    p[2 * (size_t)V + s] = q.y;
    p[3 * (size_t)V + s] = q.z;
}

struct Segments {
    double* p[kMaxSegments];
};

// The inverse transform along x and the Wilson lines: a workgroup owns RB whole
// rows (one thread per site, SPT where a row is longer than the workgroup) and
// takes the sheets of its segment (blockIdx.y) in order.  Per sheet it reads the
// kept columns of the planes, transforms them in LDS, and every thread
// multiplies V^+(x) <- V^+(x) exp(-i alpha_n(x)), kept in registers.  segs.p[segment]
// receives the product of the segment's sheets.  Bound: the FP64 arithmetic of
// the exponentials and the LDS traffic of the transforms, about equal.
template <int NC, int SITES>
__global__ __launch_bounds__(SITES > 512 ? 512 : SITES, SITES > 512 ? 2 : 4) void rows_wilson_kernel(
    const d2* __restrict__ spec, int N, int nk, int kc, int RB, int nsh, int seg_len, Segments segs, Fft f)
{
    constexpr int PAIRS = NC == 2 ? 2 : 4, SPT = SITES > 512 ? 2 : 1;
    __shared__ d2 lds[2][PAIRS * SITES];
    const int V = N * N, y0 = (int)blockIdx.x * RB, rows = min(RB, N - y0), ns = rows * N;
    const int first = (int)blockIdx.y * seg_len, last = min(nsh, first + seg_len);
    m3<double> v[SPT];
    q4<double> w[SPT];
#pragma unroll
    for (int k = 0; k < SPT; k++) {
        v[k] = identity<double>();
        w[k] = qone<double>();
    }
    // transform b = pair * rows + row
    const float inv_rows = 1.0f / (float)rows;
    for (int sh = first; sh < last; sh++) {
        const d2* const plane = spec + (size_t)sh * PAIRS * N * nk + (size_t)y0 * nk;
        auto gload = [&](int b, int i) {
            if (i > kc && i < N - nk + kc + 1) return make_double2(0.0, 0.0);
            const int p = small_div(b, inv_rows), c = i <= kc ? i : i - (N - nk);
            return plane[(size_t)p * N * nk + (size_t)(b - p * rows) * nk + c];
        };
        int Ns = 1;
        for (int s = 0; s < f.n; s++) {
            const int R = stage_radix(f.code, s);
            const d2* a = lds[(s & 1) ^ 1];
            d2* b = lds[s & 1];
            auto lload = [&](int t, int i) { return a[t * N + i]; };
            auto lstore = [&](int t, int i, d2 x) { b[t * N + i] = x; };
            if (s == 0) fft_any<false, 0>(R, PAIRS * rows, 0, N, Ns, f.inv_r[s], f.inv_ns[s], 1.0, f.tw, gload, lstore);
            else fft_any<false, 0>(R, PAIRS * rows, 0, N, Ns, f.inv_r[s], f.inv_ns[s], 1.0, f.tw, lload, lstore);
            Ns *= R;
        }
        const d2* const alpha = lds[(f.n - 1) & 1];
#pragma unroll
        for (int k = 0; k < SPT; k++) {
            const int t = (int)threadIdx.x + k * (int)blockDim.x;
            if (t >= ns) continue;
            if constexpr (NC == 2) {
                const d2 w0 = alpha[t], w1 = alpha[ns + t];
                w[k] = qmul(w[k], qexpi(v3<double>{{w0.x, w0.y, w1.x}}, -1.0));
            } else {
                a8<double> x;
#pragma unroll
                for (int p = 0; p < PAIRS; p++) {
                    const d2 z = alpha[p * ns + t];
                    x.v[2 * p] = z.x;
                    x.v[2 * p + 1] = z.y;
                }
                v[k] = mul(v[k], expi(x, -1.0));
            }
        }
        __syncthreads();  // the next sheet's first stage overwrites a buffer
    }
    double* const out = segs.p[blockIdx.y];
#pragma unroll
    for (int k = 0; k < SPT; k++) {
        const int t = (int)threadIdx.x + k * (int)blockDim.x;
        if (t >= ns) continue;
        if constexpr (NC == 2) stQ(out, y0 * N + t, V, w[k]);
        else stM(out, y0 * N + t, V, v[k]);
    }
}

// Vdag <- [Vdag] seg_0 seg_1 ... (with Vdag in front unless `fresh`)
template <int NC>
__global__ void join_segments_kernel(Segments seg, int nseg, int V, int fresh, double* Vdag)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    if constexpr (NC == 2) {
        q4<double> q = ldQ(fresh ? seg.p[0] : Vdag, s, V);
        for (int k = fresh ? 1 : 0; k < nseg; k++) q = qmul(q, ldQ(seg.p[k], s, V));
        stQ(Vdag, s, V, q);
    } else {
        m3<double> m = ldM(fresh ? seg.p[0] : Vdag, s, V);
        for (int k = fresh ? 1 : 0; k < nseg; k++) m = mul(m, ldM(seg.p[k], s, V));
        stM(Vdag, s, V, m);
    }
}

// the double-precision links along x and y
struct Links {
    double *x, *y;
};

// the pure-gauge link U^X_i(x) = V(x) V(x+i)^+ = (V^+(x))^+ V^+(x+i) of sites s and s+i
__device__ __forceinline__ m3<double> pure_link(const double* Vdag, int s, int si, int V)
{
    return adj_mul(ldM(Vdag, s, V), ldM(Vdag, si, V));
}
__device__ __forceinline__ q4<double> pure_link2(const double* Vdag, int s, int si, int V)
{
    return qmul(qadj(ldQ(Vdag, s, V)), ldQ(Vdag, si, V));
}
// the neighbours of site s at +i and -i
__device__ __forceinline__ int site_up(int s, int i, int N)
{
    const int x = s % N, y = s / N;
    return i == 0 ? y * N + (x + 1 == N ? 0 : x + 1) : (y + 1 == N ? 0 : y + 1) * N + x;
}
__device__ __forceinline__ int site_down(int s, int i, int N)
{
    const int x = s % N, y = s / N;
    return i == 0 ? y * N + (x == 0 ? N - 1 : x - 1) : (y == 0 ? N - 1 : y - 1) * N + x;
}

// Gaussian elimination with partial pivoting, unrolled so that J stays in
// registers: the pivot (the first largest |J[r][c]|, r >= c) is brought up by
// conditional swaps instead of an indexed row exchange.
__device__ __forceinline__ int solve8(double (&J)[8][8], double (&b)[8], double (&x)[8])
{
#pragma unroll
    for (int c = 0; c < 8; c++) {
#pragma unroll
        for (int r = c + 1; r < 8; r++) {
            const bool sw = fabs(J[r][c]) > fabs(J[c][c]);
#pragma unroll
            for (int k = c; k < 8; k++) {
                const double t = J[c][k];
                J[c][k] = sw ? J[r][k] : t;
                J[r][k] = sw ? t : J[r][k];
            }
            const double t = b[c];
            b[c] = sw ? b[r] : t;
            b[r] = sw ? t : b[r];
        }
        if (J[c][c] == 0.0) return -1;
#pragma unroll
        for (int r = c + 1; r < 8; r++) {
            const double f = J[r][c] / J[c][c];
#pragma unroll
            for (int k = c; k < 8; k++) J[r][k] -= f * J[c][k];
            b[r] -= f * b[c];
        }
    }
#pragma unroll
    for (int r = 7; r >= 0; r--) {
        double acc = b[r];
#pragma unroll
        for (int k = r + 1; k < 8; k++) acc -= J[r][k] * x[k];
        x[r] = acc / J[r][r];
    }
    return 0;
}

// The same without pivoting: false where an element is eliminated with a factor
// above 8 (then x is not to be used).
__device__ __forceinline__ bool solve8_plain(double (&J)[8][8], double (&b)[8], double (&x)[8])
{
    bool good = true;
    double inv[8];
#pragma unroll
    for (int c = 0; c < 8; c++) {
        inv[c] = 1.0 / J[c][c];
#pragma unroll
        for (int r = c + 1; r < 8; r++) {
            const double f = J[r][c] * inv[c];
            good = good && fabs(f) <= 8.0;
#pragma unroll
            for (int k = c + 1; k < 8; k++) J[r][k] = fma(-f, J[c][k], J[r][k]);
            b[r] = fma(-f, b[c], b[r]);
        }
    }
#pragma unroll
    for (int r = 7; r >= 0; r--) {
        double acc = b[r];
#pragma unroll
        for (int k = r + 1; k < 8; k++) acc = fma(-J[r][k], x[k], acc);
        x[r] = acc * inv[r];
        good = good && fabs(x[r]) < 1e300;  // also a vanishing last pivot
    }
    return good;
}

// column b of the Jacobian, Proj[-i Z] for Z = M T^b with the columns z0, z1, z2
// (NULL: zero)
__device__ __forceinline__ void jacobian_column(double (&J)[8][8], int b, const cx<double>* z0, const cx<double>* z1,
                                                const cx<double>* z2)
{
    auto re = [](const cx<double>* z, int r) { return z ? z[r].re : 0.0; };
    auto im = [](const cx<double>* z, int r) { return z ? z[r].im : 0.0; };
    J[0][b] = -(re(z0, 1) + re(z1, 0));
    J[1][b] = im(z1, 0) - im(z0, 1);
    J[2][b] = re(z1, 1) - re(z0, 0);
    J[3][b] = -(re(z0, 2) + re(z2, 0));
    J[4][b] = im(z2, 0) - im(z0, 2);
    J[5][b] = -(re(z1, 2) + re(z2, 1));
    J[6][b] = im(z2, 1) - im(z1, 2);
    J[7][b] = (2.0 * re(z2, 2) - re(z0, 0) - re(z1, 1)) * kInvSqrt3<double>;
}
__device__ __forceinline__ void jacobian(const m3<double>& M, double (&J)[8][8])
{
    // the columns of M by 1/2, i/2 and -i/2
    cx<double> h[3][3], p[3][3], m[3][3];
#pragma unroll
    for (int c = 0; c < 3; c++)
#pragma unroll
        for (int r = 0; r < 3; r++) {
            const cx<double> z = {0.5 * M.e[3 * r + c].re, 0.5 * M.e[3 * r + c].im};
            h[c][r] = z;
            p[c][r] = {-z.im, z.re};
            m[c][r] = {z.im, -z.re};
        }
    jacobian_column(J, 0, h[1], h[0], nullptr);
    jacobian_column(J, 1, p[1], m[0], nullptr);
    jacobian_column(J, 3, h[2], nullptr, h[0]);
    jacobian_column(J, 4, p[2], nullptr, m[0]);
    jacobian_column(J, 5, nullptr, h[2], h[1]);
    jacobian_column(J, 6, nullptr, p[2], m[1]);
    cx<double> a[3], b[3], c[3];
#pragma unroll
    for (int r = 0; r < 3; r++) a[r] = {-h[1][r].re, -h[1][r].im};
    jacobian_column(J, 2, h[0], a, nullptr);
#pragma unroll
    for (int r = 0; r < 3; r++) {
        a[r] = {kInvSqrt3<double> * h[0][r].re, kInvSqrt3<double> * h[0][r].im};
        b[r] = {kInvSqrt3<double> * h[1][r].re, kInvSqrt3<double> * h[1][r].im};
        c[r] = {-2.0 * kInvSqrt3<double> * h[2][r].re, -2.0 * kInvSqrt3<double> * h[2][r].im};
    }
    jacobian_column(J, 7, a, b, c);
}

// tau = 0 links: Newton on Proj[(U^A + U^B)(1 + U^+)] = 0 in the coordinates of
// U = exp(iX) U_0, Jacobian columns Proj[-i W U^+ T^b] (W = U^A + U^B), start at
// the row-projected W; stop at |F|_inf < tol or when the step is at rounding level.
// A chain of a few iterations per link, bound by its length on small lattices and by
// instruction issue on large ones: the generators are used by their two or three
// entries, and the elimination pivots only where it has to (smooth fields have
// M ~ 2, a dominant diagonal).  Eight general products and a pivoted elimination ->
// this: 32^2 37.8 -> 22.0 us, 96^2 28.2 -> 15.8, 384^2 123 -> 78, 1024^2 764 -> 470.
__global__ __launch_bounds__(128) void links_kernel(const double* __restrict__ VA, const double* __restrict__ VB, int N, double tol,
                             int maxit, Links U, int* fails)
{
    const int V = N * N;
    const int id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= 2 * V) return;
    const int i = id / V, s = id % V, si = site_up(s, i, N);
    const m3<double> A = pure_link(VA, s, si, V), B = pure_link(VB, s, si, V);
    m3<double> W;
    for (int c = 0; c < 9; c++) W.e[c] = {A.e[c].re + B.e[c].re, A.e[c].im + B.e[c].im};
    m3<double> u = reunitarize(W);
    bool ok = false;
    for (int it = 0; it < maxit; it++) {
        const m3<double> WUd = mul_adj(W, u);
        m3<double> M = WUd;
        for (int c = 0; c < 9; c++) { M.e[c].re += W.e[c].re; M.e[c].im += W.e[c].im; }
        const a8<double> F = proj(M);
        double fmax = 0;
        for (int a = 0; a < 8; a++) fmax = fmax > fabs(F.v[a]) ? fmax : fabs(F.v[a]);
        if (fmax < tol) { ok = true; break; }
        double J[8][8], rhs[8], X[8];
        jacobian(WUd, J);
        for (int a = 0; a < 8; a++) rhs[a] = -F.v[a];
        if (!solve8_plain(J, rhs, X)) {
            jacobian(WUd, J);
            for (int a = 0; a < 8; a++) rhs[a] = -F.v[a];
            if (solve8(J, rhs, X)) break;
        }
        a8<double> xa;
        double xmax = 0;
        for (int a = 0; a < 8; a++) { xa.v[a] = X[a]; xmax = xmax > fabs(X[a]) ? xmax : fabs(X[a]); }
        u = mul(expi(xa, 1.0), u);
        if (xmax < 1e-15) { ok = true; break; }
    }
    if (!ok) atomicAdd(fails, 1);
    stM(i == 0 ? U.x : U.y, s, V, u);
}

// pi(x) = (1/2) sum_i Proj[(U_i(x)-1)(U^B_i(x)^+ - U^A_i(x)^+) + (U_i(x-i)^+ - 1)(U^B_i(x-i) - U^A_i(x-i))]
template <typename T>
__global__ __launch_bounds__(128) void pi0_kernel(const double* __restrict__ VA, const double* __restrict__ VB,
                                                  Links U, int N, T* pi)
{
    const int V = N * N;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    m3<double> acc;
    for (int c = 0; c < 9; c++) acc.e[c] = {0, 0};
    for (int i = 0; i < 2; i++) {
        const int sm = site_down(s, i, N), sp = site_up(s, i, N);
        const double* const Ui = i == 0 ? U.x : U.y;
        m3<double> u = ldM(Ui, s, V), a = pure_link(VA, s, sp, V), b = pure_link(VB, s, sp, V);
        m3<double> L = u, R;
        L.e[0].re -= 1; L.e[4].re -= 1; L.e[8].re -= 1;
        for (int c = 0; c < 9; c++) {  // U^B^+ - U^A^+
            const int tr = 3 * (c % 3) + c / 3;
            R.e[c] = {b.e[tr].re - a.e[tr].re, -(b.e[tr].im - a.e[tr].im)};
        }
        m3<double> P1 = mul(L, R);
        u = ldM(Ui, sm, V); a = pure_link(VA, sm, s, V); b = pure_link(VB, sm, s, V);
        L = adj(u);
        L.e[0].re -= 1; L.e[4].re -= 1; L.e[8].re -= 1;
        for (int c = 0; c < 9; c++) R.e[c] = {b.e[c].re - a.e[c].re, b.e[c].im - a.e[c].im};
        m3<double> P2 = mul(L, R);
        for (int c = 0; c < 9; c++) {
            acc.e[c].re += P1.e[c].re + P2.e[c].re;
            acc.e[c].im += P1.e[c].im + P2.e[c].im;
        }
    }
    const a8<double> p = proj(acc);
    for (int a = 0; a < 8; a++) pi[(size_t)a * V + s] = (T)(0.5 * p.v[a]);
}

template <typename T> __global__ void zero_kernel(T* p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = T(0);
}

// ------------------------------------------------------------------ particles
// key (seed, 3), counter (p, block, 0, 0).  Block 0: x, y, azimuth, p_T.
// Blocks 1..5: normals; the 3x3 complex Ginibre matrix Z takes entry (r,c)
// from normals 2(3r+c), 2(3r+c)+1; its columns orthonormalised by modified
// Gram-Schmidt give a Haar unitary (positive R diagonal), Q = U Q0 U^+.
template <typename T> __global__ void particles_kernel(PartICArgs a, T* r, int* cell)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int np = a.np, N = a.N;
    if (p >= np) return;
    const uint64_t seed = a.seed;
    const u64x4 w = philox4x64((uint64_t)p, 0, 0, 0, seed, 3);
    const double x = N * u01_co(w.v[0]), y = N * u01_co(w.v[1]);
    const double phi0 = a.azimuth_uniform ? 2.0 * M_PI * u01_co(w.v[2]) : 0.0;
    const double pt = a.pt_min + (a.pt_max - a.pt_min) * u01_co(w.v[3]);
    double z[20];
    for (int b = 1; b <= 5; b++) {
        const u64x4 q = philox4x64((uint64_t)p, (uint64_t)b, 0, 0, seed, 3);
        box_muller(q.v[0], q.v[1], z[4 * (b - 1)], z[4 * (b - 1) + 1]);
        box_muller(q.v[2], q.v[3], z[4 * (b - 1) + 2], z[4 * (b - 1) + 3]);
    }
    m3<double> G;
    for (int rr = 0; rr < 3; rr++)
        for (int cc = 0; cc < 3; cc++) G.e[3 * rr + cc] = {z[2 * (3 * rr + cc)], z[2 * (3 * rr + cc) + 1]};
    for (int k = 0; k < 3; k++) {
        cx<double> v[3] = {G.e[k], G.e[3 + k], G.e[6 + k]};
        for (int j = 0; j < k; j++) {
            cx<double> ip = {0, 0};
            for (int rr = 0; rr < 3; rr++) {
                const cx<double> q = ccmul(G.e[3 * rr + j], v[rr]);
                ip.re += q.re; ip.im += q.im;
            }
            for (int rr = 0; rr < 3; rr++) {
                const cx<double> q = cmul(ip, G.e[3 * rr + j]);
                v[rr].re -= q.re; v[rr].im -= q.im;
            }
        }
        double nn = 0;
        for (int rr = 0; rr < 3; rr++) nn += v[rr].re * v[rr].re + v[rr].im * v[rr].im;
        nn = sqrt(nn);
        for (int rr = 0; rr < 3; rr++) G.e[3 * rr + k] = {v[rr].re / nn, v[rr].im / nn};
    }
    a8<double> q0;
    for (int c = 0; c < 8; c++) q0.v[c] = a.q0[c];
    const a8<double> Q = transport(G, q0);
    const double cph = cos(phi0), sph = sin(phi0);
    auto col = [&](int c) -> T& { return r[(size_t)c * np + p]; };
    col(PX_) = T(x); col(PY_) = T(y); col(PETA_) = T(0);
    col(PPX) = T(pt * cph); col(PPY) = T(pt * sph); col(PPETA) = T(0); col(PDETA) = T(0);
    col(PUX0) = T(cph); col(PUY0) = T(sph); col(PPT0) = T(pt);
    col(PPTAU) = T(0.0);  // set by the push at the formation step
    for (int c = 0; c < 8; c++) col(PQ0 + c) = T(Q.v[c]);
    int nx = (int)floor(x + 0.5), ny = (int)floor(y + 0.5);
    cell[p] = nx >= N ? nx - N : nx;
    cell[np + p] = ny >= N ? ny - N : ny;
}

// the links of both directions, n reals each, rounded
__global__ void convert_kernel(const double* __restrict__ x, const double* __restrict__ y, float* __restrict__ d, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 2 * n) d[i] = (float)(i < n ? x[i] : y[i - n]);
}

// ------------------------------------------------------------------ drivers
static hipError_t convert_to_float(const double* x, const double* y, float* dst, size_t n, hipStream_t st)
{
    hipLaunchKernelGGL(convert_kernel, dim3((unsigned)((2 * n + 255) / 256)), dim3(256), 0, st, x, y, dst, n);
    return hipGetLastError();
}

#define CK(x)                                \
    do {                                     \
        hipError_t e_ = (x);                 \
        if (e_ != hipSuccess) return e_;     \
    } while (0)

// Spectral planes are made, solved and consumed in chunks of sheets of at most
// this much memory: a chunk then stays in the last-level cache from one kernel
// to the next.
constexpr size_t kChunkBytes = (size_t)64 << 20;

static size_t padded(size_t bytes) { return (bytes + 255) / 256 * 256; }
void ICScratch::lend(void* base, size_t bytes, unsigned spans)
{
    if (base) ranges[nranges++] = {static_cast<char*>(base), bytes, spans};
}
int ICScratch::want(size_t bytes, Span span)
{
    Part& p = parts[nparts++];
    p = {bytes, span, nullptr};
    for (int k = 0; k < nranges && !p.at; k++) {
        Range& r = ranges[k];
        if (bytes > r.left || !(r.spans & only(span))) continue;
        p.at = r.base;
        r.base += std::min(padded(bytes), r.left);
        r.left -= std::min(padded(bytes), r.left);
    }
    return nparts - 1;
}
int ICScratch::room(size_t bytes, Span span) const
{
    int n = 0;
    for (int k = 0; k < nranges; k++)
        if (ranges[k].spans & only(span)) n += (int)(ranges[k].left / padded(bytes));
    return n;
}
hipError_t ICScratch::make()
{
    // what is needed before the links and what is from then on share their memory
    size_t sum[3] = {0, 0, 0};
    for (int k = 0; k < nparts; k++)
        if (!parts[k].at) sum[parts[k].span] += padded(parts[k].bytes);
    const size_t total = sum[kThroughout] + std::max(sum[kBefore], sum[kAfter]);
    if (!total) return hipSuccess;
    CK(pool_take(device, total, &block));
    char* at[3];
    at[kThroughout] = static_cast<char*>(block.p);
    at[kBefore] = at[kAfter] = at[kThroughout] + sum[kThroughout];
    for (int k = 0; k < nparts; k++)
        if (!parts[k].at) {
            parts[k].at = at[parts[k].span];
            at[parts[k].span] += padded(parts[k].bytes);
        }
    return hipSuccess;
}
ICScratch::~ICScratch() { pool_give(device, block); }

hipError_t ic_reserve(const ICArgs& a, int n_colors, bool double_links, ICScratch& mem, ICWork* w)
{
    const int pairs = n_colors == 2 ? 2 : 4, MW = n_colors == 2 ? 4 : 18, N = a.N;
    const size_t V = (size_t)N * N;
    if (N > kMaxFFT || N < 4 || radices_of(N).n < 0) return hipErrorInvalidValue;
    *w = ICWork{};
    const Band bd = band_of(N, a.uvhat);
    const size_t per_sheet = (size_t)pairs * N * bd.nk * sizeof(d2);
    // (and of at most 16383 sheets: four planes each in a grid dimension of 65535)
    const int chunk = (int)std::max<size_t>(1, std::min<size_t>(std::min(a.n_sheets, 16383), kChunkBytes / per_sheet));
    // Wilson lines: workgroups of whole rows, 256 sites where a row is
    // shorter.  The sheets of a chunk are split into up to 16 segments (joined
    // afterwards) so that the workgroups fill the chip in whole rounds: the
    // register file holds 16 of their wavefronts per CU.  The cost is counted in
    // sheets: the rounds times a segment's sheets and its start and end, and the
    // joining.  (384^2: four segments 37 sheets long instead of one of 50.)  Segments
    // whose products fit neither the lent ranges nor, beside the planes, what the pool
    // keeps are not considered.
    const size_t mw = sizeof(double) * MW * V;
    const int va = mem.want(mw, ICScratch::kThroughout), vb = mem.want(mw, ICScratch::kThroughout);
    const int in_range = mem.room(mw, ICScratch::kBefore);
    const size_t spare = std::max(kPoolBytes, double_links ? 2 * mw : 0) - std::min(per_sheet * chunk, kPoolBytes);
    const int RB = std::max(1, 256 / N), groups = (N + RB - 1) / RB;
    const int sites = RB * N, wt = std::min(512, (sites + 63) / 64 * 64), slots = 256 * (16 / (wt / 64));
    int seg_len = chunk;
    for (double best = 1e300, k = 1; k <= std::min(chunk, kMaxSegments); k++) {
        const int len = (chunk + (int)k - 1) / (int)k, nseg = (chunk + len - 1) / len;
        if (nseg > 1 && nseg > in_range && (nseg - in_range) * mw > spare) continue;
        const double cost = ((groups * nseg + slots - 1) / slots) * (len + 0.7) + 0.1 * nseg;
        if (cost < best) {
            best = cost;
            seg_len = len;
        }
    }
    const int nseg = (chunk + seg_len - 1) / seg_len;
    w->chunk = chunk;
    w->seg_len = seg_len;
    w->direct = nseg == 1 && chunk >= a.n_sheets;  // one segment: no joining
    int seg[kMaxSegments];
    for (int k = 0; k < nseg && !w->direct; k++) seg[k] = mem.want(mw, ICScratch::kBefore);
    const int K = mem.want(sizeof(double) * bd.nk * N, ICScratch::kBefore);
    const int tw = mem.want(sizeof(d2) * 3 * N, ICScratch::kBefore), spec = mem.want(per_sheet * chunk, ICScratch::kBefore);
    const int ux = double_links ? mem.want(mw, ICScratch::kAfter) : -1, uy = double_links ? mem.want(mw, ICScratch::kAfter) : -1;
    CK(mem.make());
    w->VA = mem.at<double>(va);
    w->VB = mem.at<double>(vb);
    if (double_links) {
        w->U[0] = mem.at<double>(ux);
        w->U[1] = mem.at<double>(uy);
    }
    for (int k = 0; k < nseg && !w->direct; k++) w->seg[k] = mem.at<double>(seg[k]);
    w->K = mem.at<double>(K);
    w->tw = mem.at<d2>(tw);
    w->spec = mem.at<d2>(spec);
    return hipSuccess;
}

// The Wilson lines V^+ of both nuclei (SU(3): [18][V] matrices; SU(2): [4][V]
// quaternions).
template <int NC> static hipError_t wilson_lines(const ICArgs& a, const ICWork& w, hipStream_t st)
{
    constexpr int pairs = NC == 2 ? 2 : 4;
    const int N = a.N, V = N * N, chunk = w.chunk, seg_len = w.seg_len;
    const Radices R = radices_of(N);
    Radices B = R;  // the opposite order
    for (int s = 0; s < R.n; s++) B.r[s] = R.r[R.n - 1 - s];
    const Band bd = band_of(N, a.uvhat);
    const int RB = std::max(1, 256 / N), groups = (N + RB - 1) / RB;
    const int sites = RB * N, wt = std::min(512, (sites + 63) / 64 * 64);
    hipLaunchKernelGGL(twiddle_kernel, dim3(3), dim3(256), 0, st, w.tw, N, R.n, radix_code(R), radix_code(B));
    hipLaunchKernelGGL(poisson_kernel, dim3((bd.nk * N + 255) / 256), dim3(256), 0, st, w.K, N, bd.nk, bd.kc, a.mhat,
                       a.uvhat);
    const Fft fwd = make_fft(w.tw, N, R), inv = make_fft(w.tw + N, N, R), back = make_fft(w.tw + 2 * N, N, B);
    const double sigma = a.g2mua / sqrt((double)a.n_sheets), scale = 1.0 / ((double)N * N);
    const int rb = std::max(1, 1024 / N), row_groups = (N + rb - 1) / rb;
    int bsh = 0;  // columns per workgroup: 2048 entries (4096 above 512)
    while (bsh < 5 && (2 << bsh) * N <= (N > 512 ? 4096 : 2048)) bsh++;
    const int col_groups = 8 * ((((bd.nk + (1 << bsh) - 1) >> bsh) + 7) / 8);
    for (int nucleus = 0; nucleus < 2; nucleus++) {
        double* Vdag = nucleus == 0 ? w.VA : w.VB;
        for (int s0 = 0; s0 < a.n_sheets; s0 += chunk) {
            const int nsh = std::min(chunk, a.n_sheets - s0), nseg = (nsh + seg_len - 1) / seg_len;
            hipLaunchKernelGGL(rows_forward_kernel, dim3(row_groups, nsh * (pairs / 2)), dim3(256), 0, st, w.spec, N,
                               bd.nk, bd.kc, a.seed, nucleus, s0, sigma, pairs, rb, fwd);
            const dim3 cg(col_groups, nsh * pairs);
            if (N > 512) hipLaunchKernelGGL(columns_kernel<512>, cg, dim3(512), 0, st, w.spec, N, bd.nk, bsh, w.K, scale, fwd, back);
            else hipLaunchKernelGGL(columns_kernel<256>, cg, dim3(256), 0, st, w.spec, N, bd.nk, bsh, w.K, scale, fwd, back);
            Segments dst{};
            for (int k = 0; k < nseg; k++) dst.p[k] = w.direct ? Vdag : w.seg[k];
            const dim3 wg(groups, nseg);
            if (sites <= 256) hipLaunchKernelGGL((rows_wilson_kernel<NC, 256>), wg, dim3(wt), 0, st, w.spec, N, bd.nk, bd.kc, RB, nsh, seg_len, dst, inv);
            else if (sites <= 512) hipLaunchKernelGGL((rows_wilson_kernel<NC, 512>), wg, dim3(wt), 0, st, w.spec, N, bd.nk, bd.kc, RB, nsh, seg_len, dst, inv);
            else hipLaunchKernelGGL((rows_wilson_kernel<NC, 1024>), wg, dim3(wt), 0, st, w.spec, N, bd.nk, bd.kc, RB, nsh, seg_len, dst, inv);
            if (!w.direct)
                hipLaunchKernelGGL(join_segments_kernel<NC>, dim3((V + 255) / 256), dim3(256), 0, st, dst, nseg, V,
                                   s0 == 0 ? 1 : 0, Vdag);
            CK(hipGetLastError());
        }
    }
    return hipSuccess;
}

template <typename T>
hipError_t ic_glasma(const ICArgs& a, const ICWork& w, const Fields<T>& out, int* d_fails, hipStream_t st)
{
    constexpr bool own = std::is_same<T, double>::value;  // the links are solved in place
    const int N = a.N, V = N * N;
    CK(wilson_lines<3>(a, w, st));
    Links U = {w.U[0], w.U[1]};
    if constexpr (own) U = {out.U, out.U + (size_t)18 * V};
    hipLaunchKernelGGL(links_kernel, dim3((2 * V + 127) / 128), dim3(128), 0, st, w.VA, w.VB, N, a.tol, a.maxit, U,
                       d_fails);
    hipLaunchKernelGGL(pi0_kernel<T>, dim3((V + 127) / 128), dim3(128), 0, st, w.VA, w.VB, U, N, out.pi);
    const size_t nz = (size_t)24 * V;  // phi (8V) and E (16V) are adjacent
    hipLaunchKernelGGL(zero_kernel<T>, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, st, out.phi, nz);
    if constexpr (!own) CK(convert_to_float(U.x, U.y, out.U, (size_t)18 * V, st));
    return hipGetLastError();
}
template hipError_t ic_glasma<double>(const ICArgs&, const ICWork&, const Fields<double>&, int*, hipStream_t);
template hipError_t ic_glasma<float>(const ICArgs&, const ICWork&, const Fields<float>&, int*, hipStream_t);

// ------------------------------------------------------------------ SU(2)
// tau = 0 links: W = U^A + U^B is a real multiple of an SU(2) element S, and
// U = S^2 = W W / |W|^2 solves Proj[W (1 + U^+)] = 0 (W (1 + U^+) = W + W^+ |W|^0
// is then a multiple of 1)
__global__ void links2_kernel(const double* __restrict__ VA, const double* __restrict__ VB, int N, Links U)
{
    const int V = N * N;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= 2 * V) return;
    const int i = k / V, s = k - i * V, si = site_up(s, i, N);
    const q4<double> W = qadd(pure_link2(VA, s, si, V), pure_link2(VB, s, si, V));
    const double n2 = W.w * W.w + W.x * W.x + W.y * W.y + W.z * W.z;
    const q4<double> S2 = qmul(W, W);
    stQ(i == 0 ? U.x : U.y, s, V, {S2.w / n2, S2.x / n2, S2.y / n2, S2.z / n2});
}
// pi(0) of the SU(3) kernel on quaternions
template <typename T>
__global__ void pi02_kernel(const double* __restrict__ VA, const double* __restrict__ VB, Links U, int N, T* pi)
{
    const int V = N * N;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= V) return;
    q4<double> acc = {0, 0, 0, 0};
    for (int i = 0; i < 2; i++) {
        const int sm = site_down(s, i, N), sp = site_up(s, i, N);
        const double* const Ui = i == 0 ? U.x : U.y;
        const q4<double> P1 = qmul(qsub(ldQ(Ui, s, V), qone<double>()),
                                   qsub(qadj(pure_link2(VB, s, sp, V)), qadj(pure_link2(VA, s, sp, V))));
        const q4<double> P2 = qmul(qsub(qadj(ldQ(Ui, sm, V)), qone<double>()),
                                   qsub(pure_link2(VB, sm, s, V), pure_link2(VA, sm, s, V)));
        acc = qadd(acc, qadd(P1, P2));
    }
    const v3<double> p = qproj(acc);
    for (int a = 0; a < 3; a++) pi[(size_t)a * V + s] = (T)(0.5 * p.v[a]);
}

template <typename T>
hipError_t ic_glasma2(const ICArgs& a, const ICWork& w, const Fields2<T>& out, hipStream_t st)
{
    constexpr bool own = std::is_same<T, double>::value;
    const int N = a.N, V = N * N;
    CK(wilson_lines<2>(a, w, st));
    Links U = {w.U[0], w.U[1]};
    if constexpr (own) U = {out.U, out.U + (size_t)4 * V};
    hipLaunchKernelGGL(links2_kernel, dim3((2 * V + 255) / 256), dim3(256), 0, st, w.VA, w.VB, N, U);
    hipLaunchKernelGGL(pi02_kernel<T>, dim3((V + 255) / 256), dim3(256), 0, st, w.VA, w.VB, U, N, out.pi);
    const size_t nz = (size_t)9 * V;  // phi (3V) and E (6V) are adjacent
    hipLaunchKernelGGL(zero_kernel<T>, dim3((unsigned)((nz + 255) / 256)), dim3(256), 0, st, out.phi, nz);
    if constexpr (!own) CK(convert_to_float(U.x, U.y, out.U, (size_t)4 * V, st));
    return hipGetLastError();
}
template hipError_t ic_glasma2<double>(const ICArgs&, const ICWork&, const Fields2<double>&, hipStream_t);
template hipError_t ic_glasma2<float>(const ICArgs&, const ICWork&, const Fields2<float>&, hipStream_t);

// SU(2) particles: block 0 as for SU(3); the charge from the Darboux
// parametrisation (Sec. IV.A) with J^2 = q2: words 0, 1 of block 1 give
// phi = 2 pi u and xi = J (2 u' - 1), Q = (cos phi rho, sin phi rho, xi),
// rho = sqrt(J^2 - xi^2).  Records keep the SU(3) layout (Q^4..Q^8 = 0).
template <typename T> __global__ void particles2_kernel(PartICArgs a, double J, T* r, int* cell)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int np = a.np, N = a.N;
    if (p >= np) return;
    const u64x4 w = philox4x64((uint64_t)p, 0, 0, 0, a.seed, 3);
    const u64x4 v = philox4x64((uint64_t)p, 1, 0, 0, a.seed, 3);
    const double x = N * u01_co(w.v[0]), y = N * u01_co(w.v[1]);
    const double phi0 = a.azimuth_uniform ? 2.0 * M_PI * u01_co(w.v[2]) : 0.0;
    const double pt = a.pt_min + (a.pt_max - a.pt_min) * u01_co(w.v[3]);
    const double ph = 2.0 * M_PI * u01_co(v.v[0]), xi = J * (2.0 * u01_co(v.v[1]) - 1.0);
    const double rho = sqrt(J * J - xi * xi);
    const double cph = cos(phi0), sph = sin(phi0);
    auto col = [&](int c) -> T& { return r[(size_t)c * np + p]; };
    col(PX_) = T(x); col(PY_) = T(y); col(PETA_) = T(0);
    col(PPX) = T(pt * cph); col(PPY) = T(pt * sph); col(PPETA) = T(0); col(PDETA) = T(0);
    col(PUX0) = T(cph); col(PUY0) = T(sph); col(PPT0) = T(pt);
    col(PPTAU) = T(0.0);  // set by the push at the formation step
    col(PQ0) = T(cos(ph) * rho); col(PQ0 + 1) = T(sin(ph) * rho); col(PQ0 + 2) = T(xi);
    for (int c = 3; c < 8; c++) col(PQ0 + c) = T(0.0);
    int nx = (int)floor(x + 0.5), ny = (int)floor(y + 0.5);
    cell[p] = nx >= N ? nx - N : nx;
    cell[np + p] = ny >= N ? ny - N : ny;
}

template <typename T>
hipError_t ic_particles2(const PartICArgs& a, double q2, T* r, int* cell, hipStream_t st)
{
    if (a.np <= 0) return hipSuccess;
    hipLaunchKernelGGL(particles2_kernel<T>, dim3((a.np + 127) / 128), dim3(128), 0, st, a, sqrt(q2), r, cell);
    return hipGetLastError();
}
template hipError_t ic_particles2<double>(const PartICArgs&, double, double*, int*, hipStream_t);
template hipError_t ic_particles2<float>(const PartICArgs&, double, float*, int*, hipStream_t);

template <typename T> hipError_t ic_particles(const PartICArgs& a, T* r, int* cell, hipStream_t st)
{
    if (a.np <= 0) return hipSuccess;
    hipLaunchKernelGGL(particles_kernel<T>, dim3((a.np + 127) / 128), dim3(128), 0, st, a, r, cell);
    return hipGetLastError();
}
template hipError_t ic_particles<double>(const PartICArgs&, double*, int*, hipStream_t);
template hipError_t ic_particles<float>(const PartICArgs&, float*, int*, hipStream_t);

}  // namespace cpic
