// pushbody.h -- the push of one block of particles (Sec. III.B), as the push
// kernels (push.hip) and the pipelined step (step.hip) run it.
#pragma once
#include "reduce.h"
#include "wong.h"

namespace cpic {

// Sub-job placement.  The TPP waves that share a group of 64 particles split
// the eight sub-jobs of the colour fields (cellfields.h); the owner wave
// (role 0) meanwhile rotates Q and, after one barrier, contracts the helpers'
// vectors with Q.  Byte k of the table places sub-job k as (wave << 4 | LDS
// slot of that wave); wave 0 is the owner, which evaluates its sub-jobs
// itself.  Sub-jobs share a slot only if they are parts of the same field
// (B_eta).  Each helper takes one memory round trip per sub-job:
//   TPP 1: the owner evaluates everything;
//   TPP 2: wave 1 E_y (slot 0) and B_eta (slot 1), the owner the rest;
//   TPP 4: the helpers split by the link they transport with:
//          1: E_x, B_y and B_eta part 5 (U_x(c-x)); 2: E_y, B_x and part 6
//          (U_y(c-y)); 3: part 7 (U_y(c-x-y) and U_x(c-x)) and E_eta;
//   TPP 8: one sub-job per helper (E_eta beside part 6 in wave 6), in
//          blocks of 512 threads.
// The links are read as two rows (the third rebuilt).
template <int TPP> __device__ __forceinline__ constexpr int subjob_place(int k)
{
    constexpr uint64_t tab = TPP == 8   ? 0x7060503040612010ull
                             : TPP == 4 ? 0x3022121121312010ull
                             : TPP == 2 ? 0x1111110000001000ull
                                        : 0ull;
    return (int)((tab >> (8 * k)) & 0xffu);
}
template <int TPP> constexpr int kSlots = TPP == 4 ? 3 : 2;  // LDS slots per helper wave

// A helper of a four-wave group (the placement of subjob_place<4>), with the
// loads shared between its sub-jobs.  Role 1 (i = x) and 2 (i = y) gather in
// their first phase what other waves of the group also read (U_i(c-i), U_i(c),
// phi at c +- i, the plaquettes), and form D_i and their part of B_eta; in the
// second phase, with U_i(c-i) kept, E_i at c and c-i at both half steps,
// which no other wave reads.  Lines that several waves read are so fetched
// while they are all in flight, before the L2 turns them over.  Role 3 forms
// part 7 and E_eta in one round trip.  The results go to the wave's LDS slots
// (rows r0 + 8 slot).
template <typename T>
__device__ __forceinline__ void helper4(int role, const View<T>& A, const View<T>& B, const View<T>& Gv, const Cell& c,
                                        int n, T t, bool eonly, T (*shF)[64], int r0, int lane, bool live)
{
    const bool on_e = n > 0, on_bt = n > 0 && !eonly, on_be = !eonly;
    auto put = [&](int slot, const a8<T>& F) {
#pragma unroll
        for (int q = 0; q < 8; q++) shF[r0 + 8 * slot + q][lane] = live ? F.v[q] : T(0);
    };
    if (role == 3) {
        a8<T> part = azero<T>();
        if (on_be) part = subjob<T>(7, A, B, Gv, c, n, t);
        put(0, part);
        put(1, cell_Eeta<T>(A, B, c, n));
        return;
    }
    const int i = role - 1;
    const uint32_t sb = i == 0 ? c.s_xm : c.s_ym, ce = kCompE + 8 * (uint32_t)i;
    const m3<T> L = vU(A, sb, i);
    a8<T> bf = azero<T>(), part = azero<T>();
    if (on_bt) {
        // B_y = +(1/2t) D_x (role 1), B_x = -(1/2t) D_y (role 2)
        const a8<T> f = transport(vU(A, c.s, i), vA(A, i == 0 ? c.s_xp : c.s_yp, kCompPhi));
        const a8<T> b = transport_adj(L, vA(A, sb, kCompPhi));
        const T sc = (i == 0 ? T(1) : T(-1)) / (T(2) * t);
#pragma unroll
        for (int q = 0; q < 8; q++) bf.v[q] = sc * (f.v[q] - b.v[q]);
    }
    if (on_be) {
        part = transport_adj(L, vA(Gv, sb, 0));
        if (i == 0) {
            const a8<T> g0 = vA(Gv, c.s, 0);
#pragma unroll
            for (int q = 0; q < 8; q++) part.v[q] += g0.v[q];
        }
#pragma unroll
        for (int q = 0; q < 8; q++) part.v[q] *= T(-0.25);
    }
    put(1, bf);
    put(2, part);
    CPIC_PHASE();
    a8<T> e = azero<T>();
    if (on_e) {
        const a8<T> h0 = vA(A, c.s, ce), h1 = vA(B, c.s, ce), b0 = vA(A, sb, ce), b1 = vA(B, sb, ce);
        a8<T> back;
#pragma unroll
        for (int q = 0; q < 8; q++) back.v[q] = b0.v[q] + b1.v[q];
        const a8<T> tb = transport_adj(L, back);
        const T w = T(1) / (T(4) * t);
#pragma unroll
        for (int q = 0; q < 8; q++) e.v[q] = w * ((h0.v[q] + h1.v[q]) + tb.v[q]);
    }
    put(0, e);
}
__host__ __device__ constexpr int push_block_threads(int tpp) { return tpp == 8 ? 512 : 256; }

// TPP wavefronts per group of 64 particles: a block holds 256 / TPP particles
// (64 for TPP 8).  Wave w works on particle group w / TPP in role w % TPP, so
// every wave follows one uniform path.  The role-0 wave owns the particle
// state: it rotates Q while the helper waves evaluate their field vectors
// into LDS; after one barrier it contracts all of them with Q and takes the
// Euler step.
template <int TPP> constexpr int kPushPPB = push_block_threads(TPP) / TPP;  // particles per block
// rows ([64]) of LDS for the helpers' field vectors; with four waves and the
// logarithm update also one gauge field
template <int TPP> constexpr int kFieldRows = kPushPPB<TPP> / 64 * (TPP - 1) * kSlots<TPP> * 8;
template <int TPP, bool LOGQ = false>
constexpr int kPushRows = TPP > 1 ? kFieldRows<TPP> + (TPP == 4 && LOGQ ? 8 : 0) : 1;

// Observables: on recording steps the owner wave of each group of 64 writes
// the group's four double-precision sums to partials[slot][group][4]; they
// are added over the groups, in group order, when the samples are read.
//
// LOGQ selects the alternative colour update of Sec. III.B instead of the
// rotation with the links: dQ/dt = i[Q, A_x v_x + A_y v_y + phi v_eta], with
// the gauge fields from the matrix logarithm of the links (A_x on the x link
// whose midpoint is nearest to the particle, (floor(x), NGP row); A_y on
// (NGP column, floor(y)); phi at the grid point; all at t_n), stepped by
// explicit Euler with the state at n like the rest of the particle.  The
// charges are then not renormalised (their Casimir drift is part of the
// method).
//
// TABLE reads the six field vectors at the cell from the per-site force
// table of this step (force_table_kernel) instead of evaluating them: the
// choice for dense ensembles, where several particles share a cell.  GL forms
// the B_eta sub-jobs from the links (no plaquette field; the straggler push
// of the fused step, fused.hip).
//
// push_particle: particle p (live: p is a particle) on the owner lane of its
// group, its broadening terms added to obs on recording steps; every wave of
// the block calls it (one barrier inside with more than one wave per group).
template <typename T, int TPP, bool LOGQ, bool TABLE = false, bool GL = false>
__device__ __forceinline__ void push_particle(const Fields<T>& Af, const Fields<T>& Bf, const T* gpl,
                                              const Parts<T>& P, const PushArgs& a, int n, int* err, int p, bool live,
                                              double (&obs)[4], T (*shF)[64], const T* table = nullptr)
{
    static_assert(!(GL && (TPP == 4 || TABLE)), "B_eta from the links: generic sub-job placements only");
    constexpr int S = kSlots<TPP>;
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const int role = wave % TPP, grp = wave / TPP;
    // helper-wave field vectors: row ((grp * (TPP-1) + role-1) * S + slot) * 8 + a of shF
    const int N = a.N, np = a.np;
    const uint32_t V = (uint32_t)N * N;
    const View<T> A = make_view<T>(Af.U, kRealsPerSite, V), B = make_view<T>(Bf.U, kRealsPerSite, V);
    const View<T> Gv = make_view<T>(gpl, kPlaqReals, V);
    const View<T> R = make_view<T>(P.r, kPartReals, (uint32_t)np);
    const View<int> C = make_view<int>(P.cell, 2, (uint32_t)np);
    const T t = T(n * a.sc.dt);
    const bool record = is_record_step(a.sc, n);
    const bool renorm = is_reunit_step(a.sc, n);
    const bool eonly = a.is_static != 0;
    const uint32_t po = (uint32_t)(live ? p : 0) * sizeof(T), pi = (uint32_t)(live ? p : 0) * sizeof(int);
    Particle<T> s;
    particle_cell(R, C, po, pi, N, a.is_static != 0, s);
    const Cell cell = make_cell<T>(s.nx, s.ny, N);
    T f[6] = {0, 0, 0, 0, 0, 0};
    // The logarithm update's two generators are the longest chain and need
    // nothing but the position: with four waves the owner takes one while the
    // helpers evaluate the fields, and the helper with the least to do the other.
    // Per step at 0.35 particles per site, FP64: 96^2 20.8 -> 13.4 us, 324^2 52.2 ->
    // 46.5, 512^2 117.8 -> 106.4; FP32: 96^2 34.0 -> 11.4, 512^2 58.9 -> 53.8 (with the
    // generator's earlier stop, su3.h).
    constexpr bool SPLIT_LOG = LOGQ && TPP == 4;
    a8<T> gen[2];
    if (role == 0) {
        particle_load_rotate<T, LOGQ, TPP == 8>(A, R, C, po, pi, cell, a, n, live, renorm, err, s);
        CPIC_PHASE();
        if constexpr (SPLIT_LOG) {
            if (live) gen[0] = particle_generator<T>(A, N, s, 0);
            CPIC_PHASE();
        }
        if (TABLE && live) {
            // all six table vectors gathered at once (one memory round trip)
            const View<T> TV = make_view<T>(table, 48, V);
            a8<T> tv[kJobs];
#pragma unroll
            for (int j = 0; j < kJobs; j++) tv[j] = vA(TV, cell.s, 8 * (uint32_t)j);
#pragma unroll
            for (int j = 0; j < kJobs; j++) f[j] += job_active(j, n, eonly) ? dot(s.Q, tv[j]) : T(0);
        } else if constexpr (!TABLE && TPP <= 2) {
            // the owner's own sub-jobs (one or two waves per group)
            if (live) {
#pragma unroll 1
                for (int k = 0; k < kSubJobs; k++) {
                    if ((subjob_place<TPP>(k) >> 4) != 0 || !subjob_active<GL>(k, n, eonly)) continue;
                    CPIC_PHASE();
                    const T dq = dot(s.Q, subjob<T, GL>(k, A, B, Gv, cell, n, t));
                    const int j = subjob_field(k);
#pragma unroll
                    for (int jj = 0; jj < kJobs; jj++) f[jj] += jj == j ? dq : T(0);
                }
            }
        }
    } else if constexpr (TPP == 4) {
        helper4<T>(role, A, B, Gv, cell, n, t, eonly, shF, (grp * (TPP - 1) + role - 1) * S * 8, lane, live);
        if constexpr (SPLIT_LOG)
            if (role == 3) {
                CPIC_PHASE();
                gen[1] = particle_generator<T>(A, N, s, 1);
#pragma unroll
                for (int q = 0; q < 8; q++) shF[kFieldRows<TPP> + q][lane] = gen[1].v[q];
            }
    } else if (TPP > 1) {
        // a helper wave: its sub-jobs, accumulated into its LDS slots (the
        // loop is unrolled, so each sub-job's code is specialised; with eight
        // waves a helper's one or two sub-jobs share one round trip)
        const int row0 = (grp * (TPP - 1) + role - 1) * S * 8;
#pragma unroll
        for (int r = 0; r < S * 8; r++) shF[row0 + r][lane] = T(0);
#pragma unroll
        for (int k = 0; k < kSubJobs; k++) {
            const int pl = subjob_place<TPP>(k);
            if ((pl >> 4) != role || !subjob_active<GL>(k, n, eonly)) continue;
            if (TPP < 8) CPIC_PHASE();
            const a8<T> F = subjob<T, GL>(k, A, B, Gv, cell, n, t);
            const int r = row0 + (pl & 15) * 8;
#pragma unroll
            for (int q = 0; q < 8; q++) shF[r + q][lane] += live ? F.v[q] : T(0);
        }
    }
    if (TPP > 1) {
        __syncthreads();
        if (role == 0 && live) {
            // Q . (vector of each helper slot), each slot counted once
#pragma unroll
            for (int k = 0; k < kSubJobs; k++) {
                const int pl = subjob_place<TPP>(k);
                bool first = (pl >> 4) != 0 && !(GL && k > 5);
#pragma unroll
                for (int i = 0; i < k; i++)
                    if (subjob_place<TPP>(i) == pl) first = false;
                if (!first) continue;
                const int r = ((grp * (TPP - 1) + (pl >> 4) - 1) * S + (pl & 15)) * 8;
                T dq = s.Q.v[0] * shF[r][lane];
#pragma unroll
                for (int q = 1; q < 8; q++) dq = fmaT(s.Q.v[q], shF[r + q][lane], dq);
                const int j = subjob_field(k);
#pragma unroll
                for (int jj = 0; jj < kJobs; jj++) f[jj] += jj == j ? dq : T(0);
            }
        }
    }
    if constexpr (SPLIT_LOG)
        if (role == 0)
#pragma unroll
            for (int q = 0; q < 8; q++) gen[1].v[q] = shF[kFieldRows<TPP> + q][lane];
    if (role == 0 && live)
        particle_update<T, LOGQ>(A, R, C, po, pi, cell, a, n, renorm, record, f, s, obs, SPLIT_LOG ? gen : nullptr);
}

// one particle per owner lane, particle blk * PPB + grp * 64 + lane; the
// owner wave of each group of 64 writes the group's sums on recording steps
template <typename T, int TPP, bool LOGQ, bool TABLE = false>
__device__ __forceinline__ void push_body(const Fields<T>& Af, const Fields<T>& Bf, const T* gpl, const Parts<T>& P,
                                          const PushArgs& a, int n, double* partials, int* err, int blk,
                                          T (*shF)[64], const T* table = nullptr)
{
    if (n < a.sc.n_form || n >= a.sc.n_max) return;  // uniform over the event
    constexpr int NG = kPushPPB<TPP> / 64;  // particle groups per block
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const int role = wave % TPP, grp = wave / TPP;
    const int p = blk * kPushPPB<TPP> + grp * 64 + lane;
    double obs[4] = {0, 0, 0, 0};
    push_particle<T, TPP, LOGQ, TABLE>(Af, Bf, gpl, P, a, n, err, p, p < a.np, obs, shF, table);
    if (is_record_step(a.sc, n) && role == 0) {
        const int ngroups = (a.np + 63) / 64, group = blk * NG + grp;
        double* dst = partials + ((size_t)record_slot_of(a.sc, n) * ngroups + group) * 4;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const double v = wave_sum(obs[c]);
            if (lane == 0 && group < ngroups) dst[c] = v;
        }
    }
}

}  // namespace cpic
