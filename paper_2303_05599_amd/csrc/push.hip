// push.hip -- the Wong / CPIC particle push (Sec. III.B) and the momentum
// broadening sums [eq:mombroad].
//
// One thread owns one test particle (structure-of-arrays records).  At time
// t_n it (1) rotates its colour charge with the links it crossed since t_{n-1}
// and with the rapidity Wilson line, (2) reads the colour-electric and
// -magnetic fields at its nearest grid point from U(n), phi(n), E(n +- 1/2),
// pi(n +- 1/2), (3) takes one explicit Euler step.  On recording steps the
// block writes double-precision partial sums of the broadening; a second
// small kernel adds the block partials in a fixed order.
#include "pushbody.h"

namespace cpic {


// The field update of step n copies n into d_step[1]; the push reads it there
// and its first block advances d_step[0] to n + 1 (no other kernel of the
// push reads d_step[0], and the next field update starts after the push).
// off: the push of a later step of a pipelined stretch (step.hip).
__device__ __forceinline__ int push_step(int* d_step, int blk, int off = 0)
{
    const int n = d_step[1] + off;
    if (blk == 0 && threadIdx.x == 0) d_step[0] = n + 1;
    return n;
}

// At least two waves per SIMD for blocks of 256 threads (FP64: 176 VGPRs,
// two blocks per CU), four (128 VGPRs: two blocks per CU) for the 512-thread
// blocks of eight waves per group.  A third block per CU (168 VGPRs, 12 of
// them spilled) puts more lines in flight than the L2 keeps for the
// wavefronts that share them: the FP64 step was 2.4 % slower.  The logarithm
// variant also takes two (FP64: 254 VGPRs, 8 spilled): with one wave per SIMD
// and no spills its FP64 step took 0.180 ms against 0.132 ms.
template <typename T, int TPP, bool LOGQ = false>
__global__ __launch_bounds__(push_block_threads(TPP), (TPP == 8 && !LOGQ) ? 4 : 2) void push_kernel(
    Fields<T> Af, Fields<T> Bf, const T* gpl, Parts<T> P, PushArgs a, int* d_step, int off, double* partials, int* err)
{
    __shared__ T shF[kPushRows<TPP, LOGQ>][64];
    const int nblocks = (a.np + kPushPPB<TPP> - 1) / kPushPPB<TPP>;
    const int blk = xcd_block(nblocks);
    if (blk >= nblocks) return;
    const int n = push_step(d_step, blk, off);
    push_body<T, TPP, LOGQ>(Af, Bf, gpl, P, a, n, partials, err, blk, shF);
}

// one wavefront per group of 64 particles, fields from the force table
template <typename T>
__global__ __launch_bounds__(256) void push_table_kernel(Fields<T> Af, Fields<T> Bf, const T* table, Parts<T> P,
                                                         PushArgs a, int* d_step, int off, double* partials, int* err)
{
    const int nblocks = (a.np + 255) / 256;
    const int blk = xcd_block(nblocks);
    if (blk >= nblocks) return;
    const int n = push_step(d_step, blk, off);
    push_body<T, 1, false, true>(Af, Bf, nullptr, P, a, n, partials, err, blk, nullptr, table);
}

// The six field vectors (E_x, E_y, E_eta, B_x, B_y, B_eta, 8 components
// each, [48][V]) at every site at t_n, from the same per-site arithmetic
// the push applies at a particle's cell.  Runs between the field update
// (which provides n in d_step[1]) and the table push or the light-like
// paths, which read the table at their cells.
template <typename T>
__global__ __launch_bounds__(256) void force_table_kernel(Fields<T> Af, Fields<T> Bf, const T* gpl, T* table, int N,
                                                          Schedule sc, bool electric_only, const int* d_step,
                                                          int off)
{
    const int V = N * N, nb = (V + 255) / 256;
    const int blk = xcd_block(nb);
    if (blk >= nb) return;
    const int n = d_step[1] + off;
    if (n < sc.n_form || n >= sc.n_max) return;
    const int s = blk * 256 + (int)threadIdx.x;
    if (s >= V) return;
    const View<T> A = make_view<T>(Af.U, kRealsPerSite, V), B = make_view<T>(Bf.U, kRealsPerSite, V);
    const View<T> TB = make_view<T>(table, 48, V), Gv = make_view<T>(gpl, kPlaqReals, V);
    const Cell cell = make_cell<T>(s % N, s / N, N);
    const T t = T(n * sc.dt);
#pragma unroll 1
    for (int j = 0; j < kJobs; j++) {
        a8<T> F = azero<T>();
        if (job_active(j, n, electric_only)) F = job_field<T>(j, A, B, Gv, cell, n, t);
        vA_st(TB, (uint32_t)s * (uint32_t)sizeof(T), 8 * (uint32_t)j, F);
        CPIC_PHASE();
    }
}

// batched events: logical block g works on particle block map[g].y of event map[g].x
// (at least two waves per SIMD, as push_kernel: the FP64 batch of 64 uneven
// events ran 2.3 % faster than with three and 12 registers spilled)
template <typename T, int TPP>
__global__ __launch_bounds__(256, 2) void batch_push_kernel(const EventDesc* __restrict__ ev, const int2* __restrict__ map,
                                                         int total)
{
    __shared__ T shF[kPushRows<TPP>][64];
    const int g = xcd_block(total);
    if (g >= total) return;
    // the work item is uniform over the workgroup: keep it (and every address
    // derived from it) in scalar registers
    const int2 m = map[g];
    const int e = __builtin_amdgcn_readfirstlane(m.x), blk = __builtin_amdgcn_readfirstlane(m.y);
    const EventDesc& d = ev[e];
    const int n = __builtin_amdgcn_readfirstlane(push_step(d.d_step, blk));
    if (d.pa.np == 0) return;  // an event without particles only advances its step
    const int V = d.N * d.N, parity = (n & 1) ^ d.flip;
    push_body<T, TPP, false>(fields_at<T>(d.f[parity], V), fields_at<T>(d.f[parity ^ 1], V),
                             static_cast<const T*>(d.gpl), Parts<T>{static_cast<T*>(d.pr), d.cell}, d.pa, n,
                             d.partials, d.d_err, blk, shF);
}

template <typename T>
hipError_t launch_batch_push(const EventDesc* ev, const int2* map, int total_blocks, int tpp, hipStream_t st)
{
    if (total_blocks <= 0) return hipSuccess;
    const dim3 g(8 * ((total_blocks + 7) / 8)), b(256);
    switch (tpp) {
    case 2: hipLaunchKernelGGL((batch_push_kernel<T, 2>), g, b, 0, st, ev, map, total_blocks); break;
    case 4: hipLaunchKernelGGL((batch_push_kernel<T, 4>), g, b, 0, st, ev, map, total_blocks); break;
    default: hipLaunchKernelGGL((batch_push_kernel<T, 1>), g, b, 0, st, ev, map, total_blocks);
    }
    return hipGetLastError();
}
template hipError_t launch_batch_push<double>(const EventDesc*, const int2*, int, int, hipStream_t);
template hipError_t launch_batch_push<float>(const EventDesc*, const int2*, int, int, hipStream_t);

int push_blocks(int np, int tpp) { return push_blocks_d(np, tpp); }

template <typename T>
hipError_t launch_force_table(const Fields<T>& A, const Fields<T>& B, const T* gpl, T* table, int N,
                              const Schedule& sc, bool electric_only, const int* d_step, hipStream_t st,
                              const KTimer& tm, int off)
{
    if (!table || !gpl || N <= 0) return hipErrorInvalidValue;
    const int nbt = (N * N + 255) / 256;
    klaunch(tm, force_table_kernel<T>, dim3(8 * ((nbt + 7) / 8)), dim3(256), st, A, B, gpl, table, N, sc,
            electric_only, d_step, off);
    return hipGetLastError();
}
template hipError_t launch_force_table<double>(const Fields<double>&, const Fields<double>&, const double*, double*,
                                               int, const Schedule&, bool, const int*, hipStream_t, const KTimer&, int);
template hipError_t launch_force_table<float>(const Fields<float>&, const Fields<float>&, const float*, float*, int,
                                              const Schedule&, bool, const int*, hipStream_t, const KTimer&, int);

template <typename T>
hipError_t launch_push_table(const Fields<T>& A, const Fields<T>& B, const T* table, const Parts<T>& P,
                             const PushArgs& a, int* d_step, double* partials, int* err, hipStream_t st,
                             const KTimer& tm, int off)
{
    if (a.np <= 0) return hipSuccess;
    if (!table) return hipErrorInvalidValue;
    const int nb = (a.np + 255) / 256;
    klaunch(tm, push_table_kernel<T>, dim3(8 * ((nb + 7) / 8)), dim3(256), st, A, B, table, P, a, d_step, off,
            partials, err);
    return hipGetLastError();
}
template hipError_t launch_push_table<double>(const Fields<double>&, const Fields<double>&, const double*,
                                              const Parts<double>&, const PushArgs&, int*, double*, int*, hipStream_t,
                                              const KTimer&, int);
template hipError_t launch_push_table<float>(const Fields<float>&, const Fields<float>&, const float*,
                                             const Parts<float>&, const PushArgs&, int*, double*, int*, hipStream_t,
                                             const KTimer&, int);

template <typename T, bool LOGQ>
static void launch_push_t(const Fields<T>& A, const Fields<T>& B, const T* gpl, const Parts<T>& P, const PushArgs& a,
                          int* d_step, int off, double* partials, int* err, hipStream_t st, const KTimer& tm)
{
    const int nb = push_blocks(a.np, a.tpp);
    const dim3 g(8 * ((nb + 7) / 8)), b(push_block_threads(a.tpp));
    switch (a.tpp) {
    case 2: klaunch(tm, push_kernel<T, 2, LOGQ>, g, b, st, A, B, gpl, P, a, d_step, off, partials, err); break;
    case 4: klaunch(tm, push_kernel<T, 4, LOGQ>, g, b, st, A, B, gpl, P, a, d_step, off, partials, err); break;
    case 8: klaunch(tm, push_kernel<T, 8, LOGQ>, g, b, st, A, B, gpl, P, a, d_step, off, partials, err); break;
    default: klaunch(tm, push_kernel<T, 1, LOGQ>, g, b, st, A, B, gpl, P, a, d_step, off, partials, err);
    }
}

template <typename T>
hipError_t launch_push(const Fields<T>& A, const Fields<T>& B, const T* gpl, const Parts<T>& P, const PushArgs& a,
                       int* d_step, double* partials, int* err, hipStream_t st, const KTimer& tm, int off)
{
    if (a.np <= 0) return hipSuccess;
    if (!gpl) return hipErrorInvalidValue;
    if (a.color_log)
        launch_push_t<T, true>(A, B, gpl, P, a, d_step, off, partials, err, st, tm);
    else
        launch_push_t<T, false>(A, B, gpl, P, a, d_step, off, partials, err, st, tm);
    return hipGetLastError();
}

// The particles that left their tile since the last reordering: blocks of
// eight waves (one group of 64 particles, one B_eta part or field per wave,
// above) over the stragglers of kStragTiles consecutive tiles, in list
// order.  Advances the step counter like the push.
template <typename T>
__global__ __launch_bounds__(512) void straggler_kernel(Fields<T> Af, Fields<T> Bf, Parts<T> P, PushArgs a,
                                                        TileParts tp, int ntiles, int* d_step, double* partials,
                                                        int ngroups, int* err)
{
    constexpr int TB = kStragTiles;
    const int nb = (ntiles + TB - 1) / TB, blk = (int)blockIdx.x;
    if (blk >= nb) return;
    const int n = push_step(d_step, blk);
    if (n < a.sc.n_form || n >= a.sc.n_max) return;  // uniform
    __shared__ T shF[kPushRows<8>][64];
    __shared__ int pre[TB + 1];
    const int t0 = blk * TB;
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int j = 0; j < TB; j++) {
            pre[j] = acc;
            acc += t0 + j < ntiles ? tp.strag_count[t0 + j] : 0;
        }
        pre[TB] = acc;
    }
    __syncthreads();
    const int K = pre[TB], lane = (int)threadIdx.x & 63;
    if (tp.strag_total && threadIdx.x == 0 && K > 0) atomicAdd(tp.strag_total, (unsigned long long)K);
    double obs[4] = {0, 0, 0, 0};
    for (int c0 = 0; c0 < K; c0 += 64) {
        const int i = c0 + lane;
        bool live = i < K;
        int p = 0;
        if (live) {
            int j = 0;
            while (j + 1 < TB && pre[j + 1] <= i) j++;
            const int k = tp.tile_start[t0 + j] + (i - pre[j]);
            p = k >= 0 && k < a.np ? tp.strag[k] : -1;
            live = p >= 0 && p < a.np;
        }
        push_particle<T, 8, false, false, true>(Af, Bf, nullptr, P, a, n, err, p, live, obs, shF);
        __syncthreads();  // the next chunk rewrites the helpers' LDS slots
    }
    if (is_record_step(a.sc, n) && threadIdx.x < 64) {
        double* dst = partials + ((size_t)record_slot_of(a.sc, n) * ngroups + ntiles + blk) * 4;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const double v = wave_sum(obs[c]);
            if (lane == 0) dst[c] = v;
        }
    }
}

template <typename T>
hipError_t launch_stragglers(const Fields<T>& A, const Fields<T>& B, const Parts<T>& P, const PushArgs& a,
                             const TileParts& tp, int ntiles, int* d_step, double* partials, int ngroups, int* err,
                             hipStream_t st, const KTimer& tm)
{
    const int nb = (ntiles + kStragTiles - 1) / kStragTiles;
    klaunch(tm, straggler_kernel<T>, dim3(nb), dim3(512), st, A, B, P, a, tp, ntiles, d_step, partials, ngroups, err);
    return hipGetLastError();
}
template hipError_t launch_stragglers<double>(const Fields<double>&, const Fields<double>&, const Parts<double>&,
                                              const PushArgs&, const TileParts&, int, int*, double*, int, int*,
                                              hipStream_t, const KTimer&);
template hipError_t launch_stragglers<float>(const Fields<float>&, const Fields<float>&, const Parts<float>&,
                                             const PushArgs&, const TileParts&, int, int*, double*, int, int*,
                                             hipStream_t, const KTimer&);

// step end of an event without particles (no push): advance the step counter
__global__ void step_advance_kernel(int* d_step)
{
    if (threadIdx.x == 0) d_step[0] = d_step[1] + 1;
}
hipError_t launch_step_advance(int* d_step, hipStream_t st)
{
    hipLaunchKernelGGL(step_advance_kernel, dim3(1), dim3(64), 0, st, d_step);
    return hipGetLastError();
}

// out[c] = sum (or max, bit c of mask) over rows of partials[row][c]; one block,
// rows dealt to threads in a fixed pattern, then a fixed-order block reduction
template <int NC>
__global__ __launch_bounds__(256) void reduce_rows_kernel(const double* __restrict__ partials, int nrows,
                                                          unsigned mask, double* out)
{
    double v[NC];
#pragma unroll
    for (int c = 0; c < NC; c++) v[c] = 0;
    for (int r = threadIdx.x; r < nrows; r += blockDim.x)
#pragma unroll
        for (int c = 0; c < NC; c++) {
            const double x = partials[(size_t)r * NC + c];
            v[c] = ((mask >> c) & 1) ? fmax(v[c], x) : v[c] + x;
        }
    block_reduce_store<NC>(v, mask, out);
}

// samples: block b sums the rows of sample slot first + b (4 columns each)
__global__ __launch_bounds__(256) void reduce_samples_kernel(const double* __restrict__ partials, int nrows, int first,
                                                             double* out)
{
    const int slot = first + (int)blockIdx.x;
    double v[4] = {0, 0, 0, 0};
    for (int r = threadIdx.x; r < nrows; r += blockDim.x)
#pragma unroll
        for (int c = 0; c < 4; c++) v[c] += partials[((size_t)slot * nrows + r) * 4 + c];
    block_reduce_store<4>(v, 0u, out + (size_t)slot * 4);
}
hipError_t launch_reduce_samples(const double* partials, int nrows, int first_slot, int count, double* out,
                                 hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(reduce_samples_kernel, dim3(count), dim3(256), 0, st, partials, nrows, first_slot, out);
    return hipGetLastError();
}

hipError_t launch_reduce_rows(const double* partials, int nrows, int ncols, double* out, hipStream_t st)
{
    if (ncols == 4) {
        hipLaunchKernelGGL(reduce_rows_kernel<4>, dim3(1), dim3(256), 0, st, partials, nrows, 0u, out);
    } else if (ncols == 8) {
        // diagnostics layout: columns 1 and 6 are maxima
        hipLaunchKernelGGL(reduce_rows_kernel<8>, dim3(1), dim3(256), 0, st, partials, nrows, (1u << 1) | (1u << 6),
                           out);
    } else if (ncols == 2) {
        hipLaunchKernelGGL(reduce_rows_kernel<2>, dim3(1), dim3(256), 0, st, partials, nrows, 3u, out);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// The drift watchdog's comparison of the diagnostics dout[10] (the columns
// of cpic_diagnostics) with the baseline taken when the state was installed
// (take_base: store dout as the baseline).  flags: bit 0 a non-finite
// column, 1 unitarity max|UU^+ - 1| > thr[0], 2 Gauss drift
// |max|G| - max|G|_0| > thr[1] max(1, max|G|_0), 3 Casimir drift: max|q2 -
// q2(R)| or max|q3 - q3(R)| moved from its baseline by more than thr[2]
// max(1, q2(R)).  The first breach is kept: watch[0] flags, watch[1] step,
// vals the unitarity and the three drifts.
__global__ void watchdog_kernel(const double* dout, double* base, int take_base, int with_casimir, double thr_u,
                                double thr_g, double thr_c, double q2ref, int n, int* watch, double* vals)
{
    if (threadIdx.x != 0) return;
    if (take_base) {
        for (int k = 0; k < 10; k++) base[k] = dout[k];
        return;
    }
    const double dg = fabs(dout[1] - base[1]);
    const double d2 = with_casimir ? fabs(dout[8] - base[8]) : 0.0, d3 = with_casimir ? fabs(dout[9] - base[9]) : 0.0;
    int f = 0;
    for (int k = 0; k < (with_casimir ? 10 : 8); k++)
        if (!isfinite(dout[k])) f |= 1;
    if (dout[6] > thr_u) f |= 2;
    if (dg > thr_g * fmax(1.0, base[1])) f |= 4;
    if (d2 > thr_c * fmax(1.0, q2ref) || d3 > thr_c * fmax(1.0, q2ref)) f |= 8;
    if (f && watch[0] == 0) {
        watch[0] = f;
        watch[1] = n;
        vals[0] = dout[6];
        vals[1] = dg;
        vals[2] = d2;
        vals[3] = d3;
    }
}
hipError_t launch_watchdog(const double* dout, double* base, bool take_base, bool with_casimir, const double thr[3],
                           double q2ref, int n, int* watch, double* vals, hipStream_t st)
{
    hipLaunchKernelGGL(watchdog_kernel, dim3(1), dim3(64), 0, st, dout, base, take_base ? 1 : 0, with_casimir ? 1 : 0,
                       thr[0], thr[1], thr[2], q2ref, n, watch, vals);
    return hipGetLastError();
}

// per block: max |q2 - q2_0|, max |q3 - q3_0| over the particles
template <typename T>
__global__ __launch_bounds__(256) void part_diag_kernel(Parts<T> P, int np, double q2r, double q3r, double* partials)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    double v[2] = {0, 0};
    if (p < np) {
        a8<double> Q;
        for (int q = 0; q < 8; q++) Q.v[q] = P.r[(size_t)(PQ0 + q) * np + p];
        const m3<double> H = herm(Q);
        const m3<double> H2 = mul(H, H);
        double tr3 = 0;
        for (int i = 0; i < 3; i++)
            for (int k = 0; k < 3; k++) tr3 += H.e[3 * i + k].re * H2.e[3 * k + i].re - H.e[3 * i + k].im * H2.e[3 * k + i].im;
        v[0] = fabs(dot(Q, Q) - q2r);
        v[1] = fabs(4.0 * tr3 - q3r);
    }
    block_reduce_store<2>(v, 3u, partials + (size_t)blockIdx.x * 2);
}
template <typename T>
hipError_t launch_part_diag(const Parts<T>& P, int np, double q2, double q3, double* partials, hipStream_t st)
{
    hipLaunchKernelGGL(part_diag_kernel<T>, dim3(push_blocks(np, 1)), dim3(256), 0, st, P, np, q2, q3, partials);
    return hipGetLastError();
}

template hipError_t launch_push<double>(const Fields<double>&, const Fields<double>&, const double*,
                                        const Parts<double>&, const PushArgs&, int*, double*, int*, hipStream_t,
                                        const KTimer&, int);
template hipError_t launch_push<float>(const Fields<float>&, const Fields<float>&, const float*, const Parts<float>&,
                                       const PushArgs&, int*, double*, int*, hipStream_t, const KTimer&, int);
template hipError_t launch_part_diag<double>(const Parts<double>&, int, double, double, double*, hipStream_t);
template hipError_t launch_part_diag<float>(const Parts<float>&, int, double, double, double*, hipStream_t);

}  // namespace cpic
