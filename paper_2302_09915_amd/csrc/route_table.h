// Launches of the scatter that sums a table of pair counts (route_table_kernel), for the translation units that have its instances.
#pragma once

#include "route_scatter.h"

namespace tamoe {

// Only the policies that scatter_store can answer at these sizes are there: a unit is 1 KiB of x at most, and U units per wavefront
// go with fewer than 4096 * U of them (65536 for U = 8; 2048 with the smaller workgroups).
template <int TH, int KK, int U, bool ROWU>
static void launch_route_table_u(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    const dim3 grid((unsigned)(1 + a.copy_blocks + a.N * a.fill_parts)), block(TH);
    constexpr int kX = (U == 8 ? 64 : 4 * U) / (TH == kTableThreads ? 1 : 2);   // MiB of x
    constexpr int kMiB = kX * (KK > 0 ? KK : TAMOE_MAX_K);                       // of rows
    constexpr bool kKeepsAll = U == 1;   // but for much padding, where 4 MiB of x do not matter
    static_assert(!kKeepsAll || kX + kMiB <= kKeepGiven, "nothing of its size streams");
    const StorePolicy policy = how.store;
    // the smallest tables in a kernel that is shorter by seven requests and their sums
    const int64_t pieces = (int64_t)a.n_blocks * (a.stride / 8);
    const bool one = U == 1 && pieces <= TH;
    const bool large = pieces > kTableBatch * TH;   // fewer than 32768 units then (table_units)
    constexpr bool kLarge = TH == kTableThreads && ROWU && KK != 1 && !(KK == 2 && U == 1);
    constexpr bool kLargeStreams = KK == 0 || (KK > 2 && U == 8);   // otherwise at most 96 MiB behind a gate, and none elsewhere
    const bool keep = kKeepsAll || how.keep || (large && !kLargeStreams);
    const auto launch_ld = [&](auto st_c, auto ld_c) {
        constexpr int ST = decltype(st_c)::value, LD = decltype(ld_c)::value;
        const auto go = [&](auto b) {
            launch_kernel(route_table_kernel<TH, KK, U, ROWU, ST, LD, decltype(b)::value>, grid, block, st, a.x, a.topk_idx, a.local_pos,
                          a.counts, a.slot, a.send, a);
        };
        if constexpr (U == 1)
            if (one) return go(std::integral_constant<int, 1>{});
        if constexpr (kLarge && (kLargeStreams || LD == kLoadKeep) && (KK != 4 || ST == kStoreThrough || ST == kStoreStream))
            if (large) return go(std::integral_constant<int, 2 * kTableBatch>{});
        go(std::integral_constant<int, kTableBatch>{});
    };
    const auto launch = [&](auto st_c) {
        constexpr int ST = decltype(st_c)::value;
        constexpr bool kBeyond = ST == kStoreOut || (ST == kStoreBack && ROWU && KK == 4);   // more than scatter_load keeps
        if constexpr (kBeyond || !kKeepsAll)
            if (kBeyond || !keep) return launch_ld(st_c, std::integral_constant<int, kLoadStream>{});
        if constexpr (!kBeyond) launch_ld(st_c, std::integral_constant<int, kLoadKeep>{});
    };
    if constexpr (kMiB > 16)   // half lines
        if (policy == kStoreStream) return launch(std::integral_constant<int, kStoreStream>{});
    const bool beyond = KK != 4 || !large;   // 240 MiB with four choices are more units than go with a large table
    if constexpr (!ROWU || (KK == 0 && kMiB > 24) || (KK == 4 && kMiB > 240))
        if (policy == kStoreBack && beyond) return launch(std::integral_constant<int, kStoreBack>{});
    if constexpr (ROWU && kMiB > 240)
        if (policy == kStoreOut && beyond) return launch(std::integral_constant<int, kStoreOut>{});
    launch(std::integral_constant<int, kStoreThrough>{});
}
template <int KK>
static void launch_table_of(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    constexpr int TH = kTableThreads;
    if (!how.by_wave) {
        if (a.threads != TH) launch_route_table_u<TH / 2, KK, 1, false>(a, how, st);
        else if (a.units == 1) launch_route_table_u<TH, KK, 1, false>(a, how, st);
        else launch_route_table_u<TH, KK, 2, false>(a, how, st);
    } else {
        if (a.threads != TH) launch_route_table_u<TH / 2, KK, 1, true>(a, how, st);
        else if (a.units == 1) launch_route_table_u<TH, KK, 1, true>(a, how, st);
        else if (a.units == 2) launch_route_table_u<TH, KK, 2, true>(a, how, st);
        else if (a.units == 4) launch_route_table_u<TH, KK, 4, true>(a, how, st);
        else launch_route_table_u<TH, KK, 8, true>(a, how, st);
    }
}

}  // namespace tamoe
