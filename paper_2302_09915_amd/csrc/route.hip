// tamoe_gate_dispatch: the forward path up to the send buffer in two or three launches (paper Section 3.1:
// gate, softmax, top-k, l_aux and local capacity; Section 4.1: one merged delivery per device;
// Section 4.3: l_topo, variable chunk sizes).  Same results as tamoe_gate + tamoe_aux_loss +
// tamoe_dispatch.  tamoe_dispatch and tamoe_dispatch_padded take the same stages behind a kernel that ranks
// a routing that is given (run_dispatch).
//
//   1. the gate kernel (gate_tile.h), or route_rank_kernel for a given routing (of few pairs: the scatter itself,
//      count_given), leaves per token tile b the number of pairs per (expert e, choice j) and for every pair its position among the pairs of
//      (b, e, j);
//   2. route_expert_kernel, one workgroup per expert: mean probability, count, the exclusive prefix of
//      the expert's pair counts in priority order (choice-major, then token order), kept rows.  Not
//      where the table of counts is small (table_units): every workgroup of the next kernel sums it by
//      itself, and this launch is left out;
//   3. route_copy_kernel or route_table_kernel: the scatter.  A pair's slot is offset[e] + prefix[e][j][b] + position, kept
//      iff prefix + position < cap[e]; offset[e] is the sum of the kept rows of the experts before e,
//      which every wavefront takes from the N kept counts by a scan of its own (two loads and a dozen
//      lane shifts: cheaper than one more pass over the experts in front of the scatter); every
//      thread derives the slots of its token on the way to moving its 16-byte chunk, and the thread
//      with the row's first chunk writes them to slot[].  The first workgroup writes what
//      describes the layer as a whole: expert offsets, rows per destination device, the loss; in the
//      fixed-size layout the last ones clear every expert's unused rows.
//      How rows are loaded and stored depends on what the caches can do for them (scatter_load, scatter_store).
// The scatter's kernels are in route_scatter.h, their instances for small tables in route_table.hip and
// route_table_k.hip, those for few pairs in route_given.hip.
#include <algorithm>

#include "route_scatter.h"

namespace tamoe {

// ---- a routing that is given ------------------------------------------------------------------------
// What the gate kernel leaves behind, from topk_idx: one workgroup of eight wavefronts per TOK tokens, of which each
// ranks 64 at a time for one choice.  An index outside [0, N) is no pair.

template <int NB, int TOK>
__global__ __launch_bounds__(512) void route_rank_kernel(const int32_t* __restrict__ idx, int64_t S, int N, int k,
                                                         const GateStats gs) {
    constexpr int WAVES = 8;
    __shared__ int32_t pairs[(TOK / 64) * TAMOE_MAX_K * NB * 32];
    __shared__ signed char sel[TOK * TAMOE_MAX_K];
    __shared__ unsigned char rank[TOK * TAMOE_MAX_K];
    const int64_t tile0 = (int64_t)linear_block() * TOK;
    if (tile0 >= S) return;   // past the last tile (grid_of)
    const int n = (int)(S - tile0 < TOK ? S - tile0 : TOK) * k;
    for (int i = threadIdx.x; i < TOK * k; i += WAVES * 64) {
        const int32_t e = i < n ? idx[tile0 * k + i] : -1;
        sel[i] = (signed char)(e >= 0 && e < N ? e : -1);
    }
    finish_block<NB, WAVES, TOK, false>(nullptr, sel, rank, pairs, threadIdx.x & 63,
                                        __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tile0, S, N, k, gs);
}

// ---- large tables -------------------------------------------------------------------------------------
// One workgroup per expert e: the exclusive prefix of the expert's pair counts in priority order (in
// place), its total, kept rows and mean probability.  A single workgroup for all experts would be a
// chain of memory round trips through one compute unit's few outstanding misses (measured: 27 us for
// 640 KiB on the large configuration); spread over N compute units each has two kilobytes to fetch.
// Nothing here needs another expert: what does (offsets, rows per device, the loss) is left to the
// kernel that follows, which has to wait for this one anyway.
constexpr int kExpertThreads = 256;

// m_part, m, c_expert and cap may be NULL (a routing that is given, no capacities).
// Nothing but latency: everything the expert needs is requested at the start and waited for once, and up to 1024
// counts take one barrier.  With a wait for the sums, one for the counts and one for the capacity: 4096 x 512,
// 16 experts 3.4 -> 3.1 us, 65536 x 64, 64 experts 3.4 -> 2.5.
__global__ __launch_bounds__(kExpertThreads) void route_expert_kernel(
    const float* __restrict__ m_part, int32_t* __restrict__ tile_pairs, int n_blocks, int entries, int pitch,
    int64_t S, const int32_t* __restrict__ cap, int pad_C, float* __restrict__ m, int32_t* __restrict__ c_expert,
    int32_t* __restrict__ kept_expert) {
    constexpr int kWaves = kExpertThreads / 64;
    __shared__ int32_t wave_cnt[2][kWaves];   // of even and odd pieces
    __shared__ float wave_sum[kWaves];

    const int e = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;

    // pair counts of this expert, 1024 entries (16 bytes per thread) at a time
    int32_t* row = tile_pairs + (size_t)e * pitch;
    auto fetch = [&](int q0) {
        const int q = q0 + 4 * tid;
        return *reinterpret_cast<const int4*>(row + (q < entries ? q : 0));
    };
    int4 v = fetch(0);
    const int32_t cap_e = WordBuffer(cap, cap != nullptr ? (int)gridDim.x : 0).load<int32_t>(e);

    // probability sums of this expert: thread-wise over ascending pieces, then lanes, then wavefronts
    // (rows of n_blocks floats are not 16-byte aligned in general)
    const WordBuffer mrow(m_part + (size_t)e * n_blocks, m != nullptr ? n_blocks : 0);
    float acc = 0.f;
    for (int q0 = 0; q0 < n_blocks; q0 += 4 * kExpertThreads) {
        const int q = q0 + 4 * tid;
        const float x0 = mrow.load<float>(q), x1 = mrow.load<float>(q + 1);
        const float x2 = mrow.load<float>(q + 2), x3 = mrow.load<float>(q + 3);
        acc += (x0 + x1) + (x2 + x3);
    }
    acc = wave_total(acc);
    if (lane == 0) wave_sum[wave] = acc;   // read behind the barrier of the first piece

    int32_t carry = 0;
    for (int q0 = 0, odd = 0; q0 < entries; q0 += 4 * kExpertThreads, odd ^= 1) {
        const int q = q0 + 4 * tid;
        // entries past the end of the row are padding of unknown content
        const int32_t a = q < entries ? v.x : 0, b = q + 1 < entries ? v.y : 0;
        const int32_t c = q + 2 < entries ? v.z : 0, d = q + 3 < entries ? v.w : 0;
        if (q0 + 4 * kExpertThreads < entries) v = fetch(q0 + 4 * kExpertThreads);
        const int32_t s4 = a + b + c + d;
        const int32_t incl = wave_inclusive_scan(s4);
        if (lane == 63) wave_cnt[odd][wave] = incl;
        __syncthreads();
        int32_t before = 0, piece = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            before += w < wave ? wave_cnt[odd][w] : 0;
            piece += wave_cnt[odd][w];
        }
        const int32_t first = carry + before + incl - s4;
        if (q < entries) *reinterpret_cast<int4*>(row + q) = make_int4(first, first + a, first + a + b, first + a + b + c);
        carry += piece;
    }

    if (tid == 0) {
        const float sum = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
        const int32_t lim = pair_limit(cap_e, cap != nullptr, pad_C);
        if (m != nullptr) m[e] = sum / (float)S;
        if (c_expert != nullptr) c_expert[e] = carry;
        kept_expert[e] = carry < lim ? carry : lim;
    }
}

// Workgroups that move rows.
static int64_t copy_workgroups(int64_t S, int cpr, int k) {
    const int U = copy_units(k);
    return scatter_by_wave(S, cpr, k) ? ceil_div(S * (int64_t)row_waves(cpr), kCopyThreads / 64 * U)
                             : ceil_div(S * (int64_t)cpr, kCopyThreads * U);
}

// Rows that the scatter writes at most.
static int64_t rows_sent(const RouteArgs& a) {
    const int64_t pairs = a.S * a.k, room = (int64_t)a.N * a.pad_C;
    return a.pad_C > 0 && room < pairs ? room : pairs;
}

// How rows are moved and x is loaded: by what it and the rows take, the unused ones of the fixed-size layout too, and by what the
// combine of as many rows will do.  The packed dispatch follows a gate on the same x.
static RowPolicies row_policies(const RouteArgs& a, bool ranks = false) {
    const bool by_wave = scatter_by_wave(a.S, a.cpr, a.k);
    const int64_t rows = rows_sent(a), buffer = a.pad_C > 0 ? (int64_t)a.N * a.pad_C : rows;
    const RowLines lines = row_lines(a.send, a.cpr);
    const bool combine_keeps = combine_load(a.S, buffer, a.cpr, a.k, lines) == kLoadKeep;
    return RowPolicies{by_wave, scatter_load(a.S, buffer, a.cpr, a.pad_C == 0, ranks, combine_keeps) == kLoadKeep,
                       scatter_store(lines, rows, a.cpr, a.k, by_wave, a.m_part != nullptr, a.pad_C > 0)};
}

// Fills in the launch geometry.
static void plan_copy(RouteArgs& a, bool given = false) {
    const bool by_wave = scatter_by_wave(a.S, a.cpr, a.k);
    a.wpr = row_waves(a.cpr);
    a.shift = pow2_shift(by_wave ? a.wpr : a.cpr);
    a.copy_blocks = a.units == 0 ? (int)copy_workgroups(a.S, a.cpr, a.k)
                                 : (int)ceil_div(move_units(a.S, a.cpr, a.k), a.threads / 64 * a.units);
    a.fill_streams = fill_streams((int64_t)a.N * a.pad_C, rows_sent(a), a.cpr);
    // about 4096 workgroups clear rows (512 of the larger ones that sum the table), at most one per 16 bytes per thread
    // where each of them counts the routing, as many as are resident beside the others, two to a compute unit
    const int wgs = a.units == 0 ? 4096 : !given ? 512 : std::max(128, 512 - a.N - a.copy_blocks);
    a.fill_parts = a.pad_C == 0 ? 0 : (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(wgs, a.N),
                                                                     ceil_div((int64_t)a.pad_C * a.cpr, a.threads)));
}

template <int KK>
static void launch_route_copy(const RouteArgs& a, const RowPolicies& how, hipStream_t st) {
    constexpr int U = copy_units(KK);
    const dim3 grid = grid_of(1 + (int64_t)a.copy_blocks + (int64_t)a.N * a.fill_parts, kCopyThreads), block(kCopyThreads);
    const int32_t* caps = a.cap != nullptr ? a.cap : a.table;   // N entries at least
    const bool rowu = how.by_wave, keep = how.keep;
    const StorePolicy policy = how.store;
#define TAMOE_ROUTE_COPY(RU, ST, LD)                                                          \
    launch_kernel(route_copy_kernel<KK, U, RU, ST, LD>, grid, block, st, a.x, a.topk_idx, a.local_pos, a.table, caps, a.slot, a.send, a)
#define TAMOE_ROUTE_COPY_LD(ST, LD)                                                          \
    do {                                                                                     \
        if (rowu) TAMOE_ROUTE_COPY(true, ST, LD); else TAMOE_ROUTE_COPY(false, ST, LD);      \
    } while (0)
#define TAMOE_ROUTE_COPY_ST(ST)                                                              \
    do {                                                                                     \
        if (keep) TAMOE_ROUTE_COPY_LD(ST, kLoadKeep); else TAMOE_ROUTE_COPY_LD(ST, kLoadStream); \
    } while (0)
    if (policy == kStoreOut) TAMOE_ROUTE_COPY_LD(kStoreOut, kLoadStream);   // more than scatter_load keeps
    else if (policy == kStoreStream) TAMOE_ROUTE_COPY_ST(kStoreStream);
    else if (policy == kStoreThrough) TAMOE_ROUTE_COPY_ST(kStoreThrough);
    else TAMOE_ROUTE_COPY_ST(kStoreBack);
#undef TAMOE_ROUTE_COPY_ST
#undef TAMOE_ROUTE_COPY_LD
#undef TAMOE_ROUTE_COPY
}

// Stages 2 and 3, for table and positions as `run` describes them.
static int run_copy(const char* fn, const GateRun& run, RouteArgs a, const char* label, hipStream_t st) {
    int rc;
    a.local_pos = run.stats.local_pos;
    a.table = run.stats.tile_pairs;
    a.counts = run.stats.counts;
    a.stride = run.stats.stride;
    a.n_blocks = run.stats.n_blocks;
    a.pitch = run.stats.pitch;
    a.tile_shift = pow2_shift(run.tile_tokens);
    const bool table = a.counts != nullptr;
    a.units = table ? table_units(a.S, a.cpr, a.N, a.k, run.tile_tokens, a.m_part != nullptr) : 0;
    a.threads = table ? table_threads(a.S, a.cpr, a.k, (int64_t)a.n_blocks * (a.stride / 8)) : kCopyThreads;
    plan_copy(a);
    if (!table) {
        TraceScope tr("route_expert_kernel", st);
        launch_kernel(route_expert_kernel, dim3(a.N), dim3(kExpertThreads), st, a.m_part, run.stats.tile_pairs, a.n_blocks,
                                                                        a.k * a.n_blocks, a.pitch, a.S, a.cap, a.pad_C,
                                                                        a.m, a.c_expert, a.kept_expert);
        if ((rc = check_launch(fn, "route_expert_kernel")) != TAMOE_OK) return rc;
    }
    {
        TraceScope tr(label, st);
        const RowPolicies how = row_policies(a);
        if (table && a.k <= 2) launch_route_table_few(a, how, st);
        else if (table) launch_route_table_many(a, how, st);
        else if (a.k == 1) launch_route_copy<1>(a, how, st);
        else if (a.k == 2) launch_route_copy<2>(a, how, st);
        else if (a.k == 3) launch_route_copy<3>(a, how, st);
        else if (a.k == 4) launch_route_copy<4>(a, how, st);
        else launch_route_copy<0>(a, how, st);
    }
    return check_launch(fn, table ? "route_table_kernel" : "route_copy_kernel");
}

int run_dispatch(const char* fn, const void* x, const int32_t* topk_idx, const int32_t* cap, int64_t S, int cpr, int N,
                 int P, int k, int pad_C, void* send, int32_t* slot, int32_t* kept_expert,
                 int32_t* expert_offset, int32_t* send_count_dev, void* ws, const Workspace& lay, hipStream_t st) {
    int rc;
    // a few more workgroups are added
    if (S > 0 && std::max(ceil_div(S * (int64_t)cpr, kCopyThreads), copy_workgroups(S, cpr, k)) >= 0x7fff0000)
        return fail(TAMOE_UNSUPPORTED, "%s: x is too large for one launch", fn);
    RouteArgs a{};
    a.x = static_cast<const vec16*>(x);
    a.topk_idx = topk_idx;
    a.cap = cap;
    a.slot = slot;
    a.send = static_cast<vec16*>(send);
    a.S = S;
    a.N = N;
    a.P = P;
    a.k = k;
    a.cpr = cpr;
    a.pad_C = pad_C;
    a.kept_expert = kept_expert;
    a.expert_offset = expert_offset;
    a.send_count_dev = send_count_dev;
    if ((a.units = given_units(S, cpr, N, k, &a.threads)) > 0) {
        const RowPolicies how = row_policies(a, true);
        if (how.store == kStoreThrough || (how.store == kStoreBack && !how.by_wave)) {   // what there are instances for
            plan_copy(a, true);
            a.k_magic = k > 1 ? (uint32_t)((((uint64_t)1 << 32) + k - 1) / k) : 0;
            {
                TraceScope tr("dispatch_copy_kernel", st);
                launch_route_given(a, how, st);
            }
            return check_launch(fn, "route_table_kernel");
        }
    }
    const bool table = table_units(S, cpr, N, k, rank_tokens(S, N, k), false) > 0;
    const int tok = rank_tokens(S, N, k);
    const int64_t blocks = ceil_div(S, tok);
    GateRun run{};
    run.stats = stats_in(ws, lay, N, k, blocks, table);
    run.tile_tokens = tok;
    if (blocks > 0) {
        TraceScope tr("route_rank_kernel", st);
        const dim3 grid = grid_of(blocks, 512), block(512);
#define TAMOE_RANK(NB)                                                                                  \
    do {                                                                                                \
        if (tok == 128) launch_kernel(route_rank_kernel<NB, 128>, grid, block, st, topk_idx, S, N, k, run.stats); \
        else if (tok == 256) launch_kernel(route_rank_kernel<NB, 256>, grid, block, st, topk_idx, S, N, k, run.stats); \
        else launch_kernel(route_rank_kernel<NB, 512>, grid, block, st, topk_idx, S, N, k, run.stats);           \
    } while (0)
        if (N <= 32) TAMOE_RANK(1);
        else if (N <= 64) TAMOE_RANK(2);
        else TAMOE_RANK(4);
#undef TAMOE_RANK
        if ((rc = check_launch(fn, "route_rank_kernel")) != TAMOE_OK) return rc;
    }
    return run_copy(fn, run, a, "dispatch_copy_kernel", st);
}

}  // namespace tamoe

using namespace tamoe;

extern "C" int tamoe_gate_dispatch(const void* x, const void* w, int dtype, int64_t S, int d, int N, int P, int k,
                                   const float* penalty, const int32_t* cap, float* logits, int32_t* topk_idx,
                                   float* topk_w, float* m, int32_t* c_expert, int32_t* c_device, float* loss,
                                   void* send, int32_t* slot, int32_t* kept_expert, int32_t* expert_offset,
                                   int32_t* send_count_dev, void* ws, size_t ws_bytes, void* stream) {
    const char* fn = "tamoe_gate_dispatch";
    clear_error();
    int rc, cpr = 0;   // 16-byte chunks per row
    if ((rc = check_shape(fn, S, N, P, k)) != TAMOE_OK) return rc;
    if ((rc = check_rows(fn, dtype, d, &cpr)) != TAMOE_OK) return rc;
    if (S > 0) {
        if ((rc = check_ptr(fn, "x", x, 16)) != TAMOE_OK) return rc;
        if ((rc = check_ptr(fn, "w", w, 16)) != TAMOE_OK) return rc;
        if ((rc = check_ptr(fn, "send", send, 16)) != TAMOE_OK) return rc;
        if ((rc = check_ptr(fn, "slot", slot, 4)) != TAMOE_OK) return rc;
    }
    if ((rc = check_ptr(fn, "cap", cap, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "kept_expert", kept_expert, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "expert_offset", expert_offset, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "send_count_dev", send_count_dev, 4)) != TAMOE_OK) return rc;
    if (penalty != nullptr && (rc = check_ptr(fn, "penalty", penalty, 4)) != TAMOE_OK) return rc;
    if (loss != nullptr && (rc = check_ptr(fn, "loss", loss, 4)) != TAMOE_OK) return rc;
    const Workspace lay = workspace_layout(S, N, k);
    if ((rc = check_select_outputs(fn, S, topk_idx, topk_w, m, c_expert, c_device, ws, ws_bytes, lay)) != TAMOE_OK)
        return rc;
    // one more workgroup is added
    if (S > 0 && std::max(ceil_div(S * (int64_t)cpr, kCopyThreads), copy_workgroups(S, cpr, k)) >= 0x7fffffff)
        return fail(TAMOE_UNSUPPORTED, "%s: x is too large for one launch", fn);
    hipStream_t st = static_cast<hipStream_t>(stream);

    GateRun run{};
    const bool table = table_units(S, cpr, N, k, gate_tile_tokens(S, N), true) > 0;
    if ((rc = run_gate_stage(fn, x, w, dtype, S, d, N, k, logits, topk_idx, topk_w, table, ws, lay, st, &run)) != TAMOE_OK)
        return rc;

    RouteArgs a{};
    a.x = static_cast<const vec16*>(x);
    a.topk_idx = topk_idx;
    a.cap = cap;
    a.m_part = run.stats.m_part;
    a.slot = slot;
    a.send = static_cast<vec16*>(send);
    a.S = S;
    a.N = N;
    a.P = P;
    a.k = k;
    a.cpr = cpr;
    a.penalty = penalty;
    // scale in double on the host, one rounding to fp32 (as tamoe_aux_loss); S = 0 has no loss
    a.loss_scale = S > 0 ? (float)((penalty != nullptr ? (double)N * (double)P : 1.0) / (double)S) : 0.f;
    a.m = m;
    a.c_expert = c_expert;
    a.c_device = c_device;
    a.loss = loss;
    a.kept_expert = kept_expert;
    a.expert_offset = expert_offset;
    a.send_count_dev = send_count_dev;
    return run_copy(fn, run, a, "route_copy_kernel", st);
}
