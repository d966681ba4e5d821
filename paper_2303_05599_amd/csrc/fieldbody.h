// fieldbody.h -- the field update of one tile of sites (Sec. II.A leapfrog), as
// the field kernels (field.hip) and the pipelined step (step.hip) run it: one
// thread per site, or four wavefronts per 64 sites on small lattices.
#pragma once
#include "bufio.h"
#include "internal.h"
#include "su3.h"
#include "tiles.h"

namespace cpic {

// The particle push and the force table take B_eta from the plaquette field
// G = Proj U_12 of every site (cellfields.h): with a plaquette buffer gpl
// ([8][V]), the field update stores G from the first step that reads it on
// (sc.n_plaq; at n = 0 the forces vanish with t = 1/t = 0, so the kick is
// still skipped while the plaquettes are formed).
template <typename T> __device__ __forceinline__ bool plaq_on(const T* gpl, const Schedule& sc, int n)
{
    return gpl != nullptr && n >= sc.n_plaq;
}

// ---------------------------------------------------------------- compressed-link LDS tiles
// (LdsLinks2, tiles.h)
template <typename T, int BX, int BY> constexpr size_t kCtileLds = sizeof(T) * 24 * (BX + 2) * (BY + 2);
template <typename T, int BX, int BY, int CP = 0>
__device__ __forceinline__ void field_ctile_body(const Fields<T>& in, const Fields<T>& out, T* gpl, int N, int tile,
                                                 const Schedule& sc, const StepSource& step, void* smem)
{
    constexpr int HX = BX + 2, HS = HX * (BY + 2);
    T* const lds = static_cast<T*>(smem);  // [24][HS]
    const int ntx = (N + BX - 1) / BX;
    const int x0 = (tile % ntx) * BX, y0 = (tile / ntx) * BY;
    const int tid = (int)threadIdx.x;
    const uint32_t V = (uint32_t)N * N;
    const View<T> vi = make_view<T>(in.U, kRealsPerSite, V), vo = make_view<T>(out.U, kRealsPerSite, V);
    stage_links2<T, BX, BY>(lds, vi, x0, y0, N, tid);
    __syncthreads();
    const int tx = tid % BX, ty = tid / BX;
    const int x = x0 + tx, y = y0 + ty;
    if (x >= N || y >= N) return;
    const int n = step.read(tile == 0 && tid == 0);
    const double td = n * sc.dt, thd = (n + 0.5) * sc.dt;
    const T t = T(td), inv_t = n > 0 ? T(1.0 / td) : T(0), dt = T(sc.dt);
    const T eps_drift = T(sc.dt / thd), phi_drift = T(sc.dt * thd);
    const bool kick = n > 0, reunit = is_reunit_step(sc, n);
    const uint32_t s = (uint32_t)((ty + 1) * HX + tx + 1);  // tile site
    const uint32_t xp = s + 1, xm = s - 1, yp = s + HX, ym = s - HX, xpym = s + 1 - HX, xmyp = s - 1 + HX;
    const Nbr g = neighbours<T>(x, y, N);                   // global sites (scalars, E, pi, outputs)
    const LdsLinks2<T, HS> L{lds};
    a8<T> PHI = vA(vi, g.s, kCompPhi);
    a8<T> F1 = azero<T>(), F2 = azero<T>(), Fpi = azero<T>();
    const bool gon = plaq_on(gpl, sc, n);
    if (kick || gon) {
        {   // U_12(x) = U_1(x) U_2(x+1) U_1(x+2)^+ U_2(x)^+
            m3<T> M = mul(L.U(s, 0), L.U(xp, 1));
            M = mul_adj(M, L.U(yp, 0));
            M = mul_adj(M, L.U(s, 1));
            F1 = proj(M);
            if (gon) vA_st(make_view<T>(gpl, kPlaqReals, V), g.s, 0, F1);
#pragma unroll
            for (int a = 0; a < 8; a++) F2.v[a] = -F1.v[a];
        }
        CPIC_PHASE();
        {   // U_{1,-2}(x) = U_1(x) U_2(x+1-2)^+ U_1(x-2)^+ U_2(x-2)
            m3<T> M = mul_adj(L.U(s, 0), L.U(xpym, 1));
            M = mul_adj(M, L.U(ym, 0));
            M = mul(M, L.U(ym, 1));
            const a8<T> p = proj(M);
#pragma unroll
            for (int a = 0; a < 8; a++) F1.v[a] += p.v[a];
        }
        CPIC_PHASE();
        {   // U_{2,-1}(x) = U_2(x) U_1(x-1+2)^+ U_2(x-1)^+ U_1(x-1)
            m3<T> M = mul_adj(L.U(s, 1), L.U(xmyp, 0));
            M = mul_adj(M, L.U(xm, 1));
            M = mul(M, L.U(xm, 0));
            const a8<T> p = proj(M);
#pragma unroll
            for (int a = 0; a < 8; a++) F2.v[a] += p.v[a];
        }
        CPIC_PHASE();
        a8<T> lap;
        {   // phi->_1, phi<-_1
            const a8<T> f1 = transport(L.U(s, 0), vA(vi, g.xp, kCompPhi));
            const a8<T> c1 = icomm(f1, PHI);
            const a8<T> b1 = transport_adj(L.U(xm, 0), vA(vi, g.xm, kCompPhi));
#pragma unroll
            for (int a = 0; a < 8; a++) {
                F1.v[a] = -t * F1.v[a] + inv_t * c1.v[a];
                lap.v[a] = f1.v[a] + b1.v[a] - T(4) * PHI.v[a];
            }
        }
        CPIC_PHASE();
        {   // phi->_2, phi<-_2
            const a8<T> f2 = transport(L.U(s, 1), vA(vi, g.yp, kCompPhi));
            const a8<T> c2 = icomm(f2, PHI);
            const a8<T> b2 = transport_adj(L.U(ym, 1), vA(vi, g.ym, kCompPhi));
#pragma unroll
            for (int a = 0; a < 8; a++) {
                F2.v[a] = -t * F2.v[a] + inv_t * c2.v[a];
                Fpi.v[a] = inv_t * (lap.v[a] + f2.v[a] + b2.v[a]);
            }
        }
    }
    CPIC_PHASE();
    a8<T> E1 = vA(vi, g.s, kCompE), E2 = vA(vi, g.s, kCompE + 8), PI = vA(vi, g.s, kCompPi);
#pragma unroll
    for (int a = 0; a < 8; a++) {
        E1.v[a] += dt * F1.v[a];
        E2.v[a] += dt * F2.v[a];
        PI.v[a] += dt * Fpi.v[a];
    }
    CPIC_PHASE();
    // drift: U_i <- exp(i (dt/t_half) E_i) U_i ; phi <- phi + dt t_half pi
    // CP: cache policy of the new links and phi, which only the next step's
    // field update reads, chosen by the host from the step's working set
    // (set_store_policy in capi.hip); the new E and pi, which this step's push
    // reads right after, keep the default policy.
    m3<T> U1 = mul(expi(E1, eps_drift), L.U(s, 0));
    if (reunit) U1 = reunitarize(U1);
    vU_st<T, CP>(vo, g.s, 0, U1);
    CPIC_PHASE();
    m3<T> U2 = mul(expi(E2, eps_drift), L.U(s, 1));
    if (reunit) U2 = reunitarize(U2);
    vU_st<T, CP>(vo, g.s, 1, U2);
#pragma unroll
    for (int a = 0; a < 8; a++) PHI.v[a] += phi_drift * PI.v[a];
    vA_st<T, CP>(vo, g.s, kCompPhi, PHI);
    vA_st(vo, g.s, kCompE, E1);
    vA_st(vo, g.s, kCompE + 8, E2);
    vA_st(vo, g.s, kCompPi, PI);
}

// ---------------------------------------------------------------- four wavefronts per 64 sites
// For lattices too small to fill the chip with a thread per site: four
// wavefronts share the same 64 sites.  The whole workgroup stages the links of
// the tile and its ring in LDS, with the third rows already rebuilt (once per
// link instead of once per use), while each wavefront loads the scalars and
// momenta of its own part, so the kernel makes one round trip to memory.  Then
//   role 0  U_12 (and G),
//   role 1  U_{1,-2} and phi<-_2,
//   role 2  U_{2,-1} and phi<-_1,
//   role 3  phi->_1, phi->_2 and their commutators with phi,
// and after one barrier role 1 kicks E_x and drifts U_x, role 2 the same along
// y, role 3 kicks pi and drifts phi.  Every sum is taken in the order of
// field_ctile_body, so the two kernels give the same bits.
// Bound: the latency of one chain (stage, one part of the forces, exchange,
// one exponential) on the smallest lattices, memory from about 250^2 on.
// Measured per launch against the thread-per-site tiles (64 x 8 / the best of
// 64 x 4, 32 x 8 and 32 x 4), FP64: 32^2 6.4 us (18.3 / 11.2), 96^2 7.2 (19.1 / 11.9),
// 216^2 13.0 (21.4 / 15.8), 384^2 32.9 (44.1 / 33.3); FP32: 32^2 5.3 us (12.4 / 10.0),
// 96^2 6.0 (13.2 / 10.1), 216^2 10.6 (15.3 / 12.5), 384^2 20.9 (25.1 / 22.2).  Before the
// shorter exponential of su3.h, 512^2: FP64 69.2 us (60.9 / 59.4), FP32 33.8 (29.5).
// Tiles of 16 x 4 sites: 32 x 2 is equal, 8 x 8 up to 10 % slower (half lines), 32 x 4
// slower below 300^2 (two wavefronts of a tile on each SIMD).
template <typename T, int HS> struct LdsLinks3 {
    const cx<T>* l;  // [18][HS]: the nine entries of U_x, then of U_y
    __device__ __forceinline__ m3<T> U(uint32_t h, int i) const
    {
        m3<T> m;
#pragma unroll
        for (int c = 0; c < 9; c++) m.e[c] = l[(9 * i + c) * HS + h];
        return m;
    }
};

template <typename T, int BX, int BY>
constexpr size_t kRolesLds = sizeof(T) * (36 * (BX + 2) * (BY + 2) + 40 * BX * BY);
template <typename T, int BX, int BY, int CP>
__device__ __forceinline__ void field_roles_body(const Fields<T>& in, const Fields<T>& out, T* gpl, int N, int tile,
                                                 const Schedule& sc, const StepSource& step, void* smem)
{
    constexpr int HX = BX + 2, HS = HX * (BY + 2), NS = BX * BY, NT = 4 * NS;
    static_assert(NS % 64 == 0, "whole wavefronts per role");
    cx<T>* const links = static_cast<cx<T>*>(smem);  // [18][HS]
    // [5][8][NS]: U_12, phi<-_2, phi<-_1 and the two commutators
    T(*const ex)[8][NS] = reinterpret_cast<T(*)[8][NS]>(links + 18 * HS);
    const int ntx = (N + BX - 1) / BX;
    const int x0 = (tile % ntx) * BX, y0 = (tile / ntx) * BY;
    const int tid = (int)threadIdx.x;
    const uint32_t V = (uint32_t)N * N;
    const View<T> vi = make_view<T>(in.U, kRealsPerSite, V), vo = make_view<T>(out.U, kRealsPerSite, V);
    const int role = __builtin_amdgcn_readfirstlane(tid / NS), q = tid % NS;
    const int tx = q % BX, ty = q / BX, x = x0 + tx, y = y0 + ty;
    const bool live = x < N && y < N;
    const Nbr g = neighbours<T>(live ? x : 0, live ? y : 0, N);
    // the part's own scalars and momenta, in flight with the links
    a8<T> A0 = azero<T>(), A1 = azero<T>(), A2 = azero<T>(), A3 = azero<T>();
    if (role == 1) {
        A0 = vA(vi, g.ym, kCompPhi);
        A1 = vA(vi, g.s, kCompE);
    } else if (role == 2) {
        A0 = vA(vi, g.xm, kCompPhi);
        A1 = vA(vi, g.s, kCompE + 8);
    } else if (role == 3) {
        A0 = vA(vi, g.xp, kCompPhi);
        A1 = vA(vi, g.s, kCompPi);
        A2 = vA(vi, g.yp, kCompPhi);
        A3 = vA(vi, g.s, kCompPhi);
    }
    const int n = step.read(tile == 0 && tid == 0);
#pragma unroll
    for (int k0 = 0; k0 < 2 * HS; k0 += NT) {
        const int k = k0 + tid;
        if (k < 2 * HS) {
            const int i = k / HS, h = k - i * HS, hy = h / HX, hx = h - hy * HX;
            const int gx = (x0 + hx - 1 + N) % N, gy = (y0 + hy - 1 + N) % N;
            const uint32_t go = (uint32_t)(gy * N + gx) * (uint32_t)sizeof(T) + (uint32_t)(18 * i) * vi.cs;
            const m3<T> m = vU(vi, go, 0);
#pragma unroll
            for (int c = 0; c < 9; c++) links[(9 * i + c) * HS + h] = m.e[c];
        }
    }
    __syncthreads();
    const double td = n * sc.dt, thd = (n + 0.5) * sc.dt;
    const T t = T(td), inv_t = n > 0 ? T(1.0 / td) : T(0), dt = T(sc.dt);
    const T eps_drift = T(sc.dt / thd), phi_drift = T(sc.dt * thd);
    const bool reunit = is_reunit_step(sc, n), gon = plaq_on(gpl, sc, n), forces = n > 0 || gon;
    const uint32_t s = (uint32_t)((ty + 1) * HX + tx + 1);
    const uint32_t xp = s + 1, xm = s - 1, yp = s + HX, ym = s - HX, xpym = s + 1 - HX, xmyp = s - 1 + HX;
    const LdsLinks3<T, HS> L{links};
    a8<T> P = azero<T>(), f1 = azero<T>(), f2 = azero<T>();
    if (forces) {
        auto put = [&](int k, const a8<T>& v) {
#pragma unroll
            for (int a = 0; a < 8; a++) ex[k][a][q] = v.v[a];
        };
        if (role == 0) {
            m3<T> M = mul(L.U(s, 0), L.U(xp, 1));
            M = mul_adj(M, L.U(yp, 0));
            P = proj(mul_adj(M, L.U(s, 1)));
            put(0, P);
            if (gon && live) vA_st(make_view<T>(gpl, kPlaqReals, V), g.s, 0, P);
        } else if (role == 1) {
            m3<T> M = mul_adj(L.U(s, 0), L.U(xpym, 1));
            M = mul_adj(M, L.U(ym, 0));
            P = proj(mul(M, L.U(ym, 1)));
            put(1, transport_adj(L.U(ym, 1), A0));
        } else if (role == 2) {
            m3<T> M = mul_adj(L.U(s, 1), L.U(xmyp, 0));
            M = mul_adj(M, L.U(xm, 1));
            P = proj(mul(M, L.U(xm, 0)));
            put(2, transport_adj(L.U(xm, 0), A0));
        } else {
            f1 = transport(L.U(s, 0), A0);
            put(3, icomm(f1, A3));
            f2 = transport(L.U(s, 1), A2);
            put(4, icomm(f2, A3));
        }
    }
    __syncthreads();
    if (role == 0 || !live) return;
    if (role == 3) {
        if (forces) {
            a8<T> lap;
#pragma unroll
            for (int a = 0; a < 8; a++) lap.v[a] = f1.v[a] + ex[2][a][q] - T(4) * A3.v[a];
#pragma unroll
            for (int a = 0; a < 8; a++) {
                const T F = inv_t * (lap.v[a] + f2.v[a] + ex[1][a][q]);
                A1.v[a] += dt * F;
            }
        }
#pragma unroll
        for (int a = 0; a < 8; a++) A3.v[a] += phi_drift * A1.v[a];
        vA_st<T, CP>(vo, g.s, kCompPhi, A3);
        vA_st(vo, g.s, kCompPi, A1);
        return;
    }
    const int i = role - 1;
    if (forces) {
#pragma unroll
        for (int a = 0; a < 8; a++) {
            T F = i == 0 ? ex[0][a][q] : -ex[0][a][q];
            F += P.v[a];
            F = -t * F + inv_t * ex[3 + i][a][q];
            A1.v[a] += dt * F;
        }
    }
    m3<T> U = mul(expi(A1, eps_drift), L.U(s, i));
    if (reunit) U = reunitarize(U);
    vU_st<T, CP>(vo, g.s + (uint32_t)(18 * i) * vo.cs, 0, U);
    vA_st(vo, g.s, kCompE + 8 * (uint32_t)i, A1);
}

}  // namespace cpic
