// step.hip -- the pipelined step: the particle push of step n and the field
// update of step n + 1 in one launch.
//
// The field update needs nothing from the particles, so inside a stretch of
// steps (one HIP graph) only the first field update and the last push run by
// themselves.  Every launch between holds the workgroups of both: a lattice
// that leaves most of the chip idle in either kernel (both wait for memory and
// for serial chains of products there) runs them beside each other, the last
// wave of the push is filled with tiles, and a step is one launch instead of
// two.  It takes a third field buffer set (the update of step n + 1 may not
// overwrite the state of step n, which the push reads) and a second plaquette
// field.  The step counter does not move inside a stretch: the launches take
// their offset from its first step as an argument.
//
// Each XCD starts with its share of the push, then takes its share of the tiles.
// Spread evenly among each other instead they were slower wherever the chip is
// full (both codes in one CU's instruction cache): 216^2 32.1 against 24.0 us
// a step, 324^2 60.6 against 46.0; tiles first 26.5 and 49.2 (FP64, 0.35
// particles per site, before the shorter exponential of su3.h).
// Per step, two launches -> one, at 0.4 particles per site:
//   FP64: 32^2 15.6 -> 10.4 us, 96^2 18.1 -> 12.8, 216^2 30.2 -> 25.0, 324^2 51.9 ->
//         45.4, 384^2 63.9 -> 62.6
//   FP32: 32^2 14.4 -> 9.5, 96^2 15.8 -> 11.0, 216^2 23.3 -> 17.1, 324^2 35.7 -> 28.3,
//         384^2 42.5 -> 35.1, 432^2 49.7 -> 43.7, 512^2 60.6 -> 54.1
//   with the colour log: FP64 96^2 19.2 -> 13.5, 324^2 53.8 -> 45.7; FP32 512^2 62.1
//         -> 55.1
// Between two lines (pipeline_pays) the steps stay separate: where two buffer sets
// fit into the 256 MB Infinity Cache and three do not, the third one costs more
// memory traffic than the overlap saves (FP64 432^2, 251 MB in three sets: 76.0 ->
// 76.6, 512^2 108.7 -> 112.9; FP32 648^2 96.9 -> 106.4).  Where two do not fit either,
// the push and the field update wait for memory in turns and share the state of
// step n + 1: FP64 648^2 201 -> 191, 768^2 284 -> 275, 1024^2 466 -> 458 (with 0.1
// particles per site 401 -> 382); FP32 768^2 137 -> 140 (134 -> 127), 1024^2 269 -> 260
// (235 -> 219).  SU(2) has its own kernel (su2.hip) under the same rule.
// With the table push (and the light-like paths) the force table of step n runs before
// the launch, on lattices where all that a step touches fits the cache (capi.hip): at
// 1.6 particles per site FP64 96^2 33.3 -> 26.9, 216^2 46.0 -> 42.1, 324^2 80.8 -> 76.1;
// FP32 96^2 27.5 -> 21.7, 216^2 35.1 -> 30.0, 324^2 49.4 -> 44.9.
// The arithmetic is that of the separate kernels, bit for bit (fieldbody.h,
// pushbody.h).
#include <type_traits>

#include "fieldbody.h"
#include "pushbody.h"

namespace cpic {

// Three workgroups per CU with the colour log (FP64: 168 registers with 6 spilled,
// against 201): 384^2 at 0.35 particles per site 61.1 -> 57.2 us, 324^2 45.0 -> 43.4,
// below 216^2 equal; with the rotation 12 are spilled and it lost up to 7 % (162^2
// 16.6 -> 17.8, 384^2 57.3 -> 60.0).
// PUSH: 0 the gather push, 1 with the logarithm update, 2 the table push
template <typename T, bool ROLES, int CP, int PUSH>
__global__ __launch_bounds__(256, PUSH == 1 && ROLES ? 3 : 2) void step_kernel(Fields<T> S0, Fields<T> S1, Fields<T> S2, const T* g0, T* g1,
                                                      Parts<T> P, PushArgs a, const T* table, int off,
                                                      int* d_step, double* partials, int* err)
{
    constexpr int BX = ROLES ? 16 : 64, BY = 4;
    constexpr int TPP = PUSH == 2 ? 1 : 4, PPB = kPushPPB<TPP>;
    constexpr size_t field_lds = ROLES ? kRolesLds<T, 16, 4> : kCtileLds<T, 64, 4>;
    constexpr size_t push_lds = sizeof(T) * 64 * kPushRows<TPP, PUSH == 1>;
    __shared__ __align__(16) char smem[field_lds > push_lds ? field_lds : push_lds];
    const int N = a.N, tiles = ((N + BX - 1) / BX) * ((N + BY - 1) / BY), blocks = (a.np + PPB - 1) / PPB;
    // entry i of XCD x: its push blocks, then its tiles
    const int pt = (tiles + 7) / 8, pb = (blocks + 7) / 8, x = (int)blockIdx.x & 7, i = (int)blockIdx.x >> 3;
    if (i < pb) {
        const int blk = x * pb + i;
        if (blk >= blocks) return;
        const int n = __builtin_amdgcn_readfirstlane(d_step[1] + off);
        push_body<T, TPP, PUSH == 1, PUSH == 2>(S0, S1, g0, P, a, n, partials, err, blk,
                                                reinterpret_cast<T(*)[64]>(smem), table);
    } else {
        const int tile = x * pt + (i - pb);
        if (tile >= tiles) return;
        const StepSource step{d_step + 1, off + 1, nullptr};
        if constexpr (ROLES) field_roles_body<T, BX, BY, CP>(S1, S2, g1, N, tile, a.sc, step, smem);
        else field_ctile_body<T, BX, BY, CP>(S1, S2, g1, N, tile, a.sc, step, smem);
    }
}

template <typename T>
hipError_t launch_step(const Fields<T>& S0, const Fields<T>& S1, const Fields<T>& S2, const T* g0, T* g1,
                       const LaunchCfg& cfg, const Parts<T>& P, const PushArgs& a, const T* table, int off, int* d_step,
                       double* partials, int* err, hipStream_t st)
{
    if (a.np <= 0 || (!table && a.tpp != 4) || (table && a.color_log) || !g0 || !g1 || !S2.U || cfg.split != 3)
        return hipErrorInvalidValue;
    auto go = [&](auto roles, auto cp) {
        constexpr bool R = decltype(roles)::value;
        constexpr int CP = decltype(cp)::value;
        const int N = a.N, bx = R ? 16 : 64, ppb = table ? kPushPPB<1> : kPushPPB<4>;
        const int tiles = ((N + bx - 1) / bx) * ((N + 3) / 4), blocks = (a.np + ppb - 1) / ppb;
        const dim3 g(8 * ((tiles + 7) / 8 + (blocks + 7) / 8)), b(256);
        if (table)
            hipLaunchKernelGGL((step_kernel<T, R, CP, 2>), g, b, 0, st, S0, S1, S2, g0, g1, P, a, table, off, d_step, partials, err);
        else if (a.color_log)
            hipLaunchKernelGGL((step_kernel<T, R, CP, 1>), g, b, 0, st, S0, S1, S2, g0, g1, P, a, table, off, d_step, partials, err);
        else
            hipLaunchKernelGGL((step_kernel<T, R, CP, 0>), g, b, 0, st, S0, S1, S2, g0, g1, P, a, table, off, d_step, partials, err);
    };
    using NT = std::integral_constant<int, kStoreNT>;
    using Plain = std::integral_constant<int, 0>;
    if (cfg.roles) {
        if (cfg.nt_store) go(std::true_type{}, NT{}); else go(std::true_type{}, Plain{});
    } else {
        if (cfg.nt_store) go(std::false_type{}, NT{}); else go(std::false_type{}, Plain{});
    }
    return hipGetLastError();
}
template hipError_t launch_step<double>(const Fields<double>&, const Fields<double>&, const Fields<double>&,
                                        const double*, double*, const LaunchCfg&, const Parts<double>&, const PushArgs&,
                                        const double*, int, int*, double*, int*, hipStream_t);
template hipError_t launch_step<float>(const Fields<float>&, const Fields<float>&, const Fields<float>&, const float*,
                                       float*, const LaunchCfg&, const Parts<float>&, const PushArgs&, const float*,
                                       int, int*, double*, int*, hipStream_t);

}  // namespace cpic
