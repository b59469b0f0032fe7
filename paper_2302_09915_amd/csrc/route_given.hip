// Instances of the scatter that counts and ranks a given routing itself (count_given): tamoe_dispatch and
// tamoe_dispatch_padded of few pairs in one launch.
#include "route_scatter.h"

namespace tamoe {

template <int TH, int KK, int U, bool ROWU>
static void launch_u(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    const dim3 grid((unsigned)(1 + a.copy_blocks + a.N * a.fill_parts)), block(TH);
    const auto launch = [&](auto st_c) {
        constexpr int ST = decltype(st_c)::value;
        if constexpr (ROWU && U >= 4)   // more than 4 MiB of x; less is loaded to stay also beside 84 MiB of padding
            if (!how.keep) {
                launch_kernel(route_table_kernel<TH, KK, U, ROWU, ST, kLoadStream, 0>, grid, block, st, a.x, a.topk_idx, nullptr, nullptr, a.slot, a.send, a);
                return;
            }
        launch_kernel(route_table_kernel<TH, KK, U, ROWU, ST, kLoadKeep, 0>, grid, block, st, a.x, a.topk_idx, nullptr, nullptr, a.slot, a.send, a);
    };
    if constexpr (!ROWU)   // rows by wavefront of these sizes go through L2
        if (how.store == kStoreBack) return launch(std::integral_constant<int, kStoreBack>{});
    launch(std::integral_constant<int, kStoreThrough>{});
}

template <int KK>
static void launch_k(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    constexpr int TH = kTableThreads;
    if (!how.by_wave) {
        if (a.threads != TH) launch_u<TH / 2, KK, 1, false>(a, how, st);
        else if (a.units == 1) launch_u<TH, KK, 1, false>(a, how, st);
        else launch_u<TH, KK, 2, false>(a, how, st);
    } else {
        if (a.threads != TH) launch_u<TH / 2, KK, 1, true>(a, how, st);
        else if (a.units == 1) launch_u<TH, KK, 1, true>(a, how, st);
        else if (a.units == 2) launch_u<TH, KK, 2, true>(a, how, st);
        else if (a.units == 4) launch_u<TH, KK, 4, true>(a, how, st);
        else launch_u<TH, KK, 8, true>(a, how, st);
    }
}

void launch_route_given(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    if (a.k == 1) launch_k<1>(a, how, st);
    else if (a.k == 2) launch_k<2>(a, how, st);
    else if (a.k == 3) launch_k<3>(a, how, st);
    else if (a.k == 4) launch_k<4>(a, how, st);
    else launch_k<0>(a, how, st);
}

}  // namespace tamoe
