// tamoe_combine: y[t] = sum over the kept choices j of topk_w[t][j] * recv[slot[t][j]]
// (paper Section 3.1: the layer output aggregates the computed results).
//
// One 16-byte chunk of y per thread (two for k = 1), no LDS: a thread gathers the same chunk of the (up to k)
// source rows (flat rows with more than four choices: four at a time, in a loop), accumulates in fp32 in
// ascending j with one fused multiply-add per term, rounds once to the storage type and writes
// the chunk of y.  Bound by HBM: d*b bytes read per kept pair, d*b written per token; the HBM
// latency is covered by the number of independent wavefronts, as in a plain copy.
#include "chunk.h"
#include "internal.h"

namespace tamoe {

constexpr int kThreads = 256;

// KK > 0: k is the compile-time constant KK; KK == 0: any k up to TAMOE_MAX_K.
// UNITW: every weight is 1 (the transpose of the scatter: dx[t] = sum of the rows its slots name).
// Rows by whole wavefronts (combine_by_wave), U segments of 64 chunks each: all slots, weights and rows of
// a token are requested without a branch between them.
template <int DT, int KK, int U, bool UNITW, int ST, int LD>
__global__ __launch_bounds__(kThreads) void combine_kernel(const vec16* __restrict__ recv, int64_t K_rows,
                                                           const int32_t* __restrict__ slot,
                                                           const float* __restrict__ topk_w, int64_t S, int k_arg,
                                                           int cpr, int wpr, int shift, vec16* __restrict__ y) {
    constexpr int KM = KK > 0 ? KK : TAMOE_MAX_K;
    const int k = KK > 0 ? KK : k_arg;
    const uint32_t wave = linear_block() * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int tok[U], col[U];
    int32_t sl[U][KM];
    float wgt[U][KM];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int seg;
        split_wave(wave * U + u, wpr, shift, tok[u], seg);
        if (tok[u] >= S) {   // past the end: its rows are not there
            tok[u] = (int)S - 1;
            seg = wpr;
        }
        col[u] = seg * 64 + lane;
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            const int64_t p = (int64_t)tok[u] * k + (KK > 0 || j < k ? j : k - 1);
            sl[u][j] = __builtin_amdgcn_readfirstlane(slot[p]);
            wgt[u][j] = UNITW ? 1.0f : topk_w[p];
        }
    }
    vec16 v[U][KM];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            const bool use = (KK > 0 || j < k) && (uint32_t)sl[u][j] < (uint64_t)K_rows;   // a dropped pair is -1
            v[u][j] = RowBuffer(recv + (size_t)(use ? sl[u][j] : 0) * cpr, cpr, use).template load<LD>(col[u]);
            wgt[u][j] = use ? wgt[u][j] : 0.f;   // adds 0 * 0: the same bits as leaving it out
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KM; ++j) Chunk<DT>::fma(acc, wgt[u][j], v[u][j]);
        RowBuffer(y + (size_t)tok[u] * cpr, cpr, true).template store<ST>(col[u], Chunk<DT>::pack(acc));
    }
}

// By wavefront or flat?  Flat with a poor last wavefront and about as many choices as wavefronts: 65536 rows of 1040
// bytes, two choices 40.5 us by wavefront, 38.2 flat (transpose 42.3, 37.8), 8000 of them 6.4 and 5.6, 65536 of 2064 bytes
// 73.1 and 71.2, four choices 124.4 and 118.7.  With more lanes in the last wavefront or other numbers of choices it is
// the other way round: 8000 rows of 1120 bytes, three choices 6.7 and 7.9; 65536 of 2304 bytes 76.7 and 80.3, of 1040
// bytes, four choices 59.6 and 62.3, of 2064 bytes, one choice 48.6 and 49.8.
static bool combine_by_wave(int64_t S, int cpr, int k) {
    const int wpr = row_waves(cpr);
    return rows_by_wave(cpr) && !(poor_last_wave(S, cpr, 4) && k >= wpr - 1 && k <= wpr + 1);
}

// Other rows: chunks flat over the lanes.  More than four choices (KK == 0) are taken four at a time: loads
// under a condition per lane hold registers across each other, and eight of them left room for one
// wavefront per SIMD in fp32.
template <int DT, int KK, int U, bool UNITW, int ST, int LD>
__global__ __launch_bounds__(kThreads) void combine_flat_kernel(const vec16* __restrict__ recv, int64_t K_rows,
                                                                const int32_t* __restrict__ slot,
                                                                const float* __restrict__ topk_w, int64_t total_chunks,
                                                                int k_arg, int cpr, int shift, vec16* __restrict__ y) {
    constexpr int KG = KK > 0 ? KK : 4;
    const int k = KK > 0 ? KK : k_arg;
    const int64_t base = (int64_t)linear_block() * (kThreads * U) + threadIdx.x;
    int tok[U], col[U];
    float acc[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = base + (int64_t)u * kThreads;
        split_chunk(c < total_chunks ? c : total_chunks - 1, total_chunks, cpr, shift, tok[u], col[u]);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[u][i] = 0.f;
    }
#pragma unroll 1
    for (int j0 = 0; j0 < k; j0 += KG) {
        int32_t sl[U][KG];
        float wgt[U][KG];
        vec16 v[U][KG];
        // all slots and weights before the first row
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KG; ++j) {
                const bool there = KK > 0 || j0 + j < k;
                const int64_t p = (int64_t)tok[u] * k + (there ? j0 + j : k - 1);
                sl[u][j] = there ? slot[p] : -1;
                wgt[u][j] = UNITW ? 1.0f : topk_w[p];
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KG; ++j) {
                const bool use = sl[u][j] >= 0 && (int64_t)sl[u][j] < K_rows;
                wgt[u][j] = use ? wgt[u][j] : 0.f;
                v[u][j] = vec16{0u, 0u, 0u, 0u};
                if (use) v[u][j] = load_chunk<LD>(recv + (size_t)sl[u][j] * cpr + col[u]);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KG; ++j) Chunk<DT>::fma(acc[u], wgt[u][j], v[u][j]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = base + (int64_t)u * kThreads;
        if (c < total_chunks) store_chunk<ST>(y + c, Chunk<DT>::pack(acc[u]));
    }
}

template <int DT, int KK, int U, bool UNITW, int ST, int LD>
static void launch_combine_s(const void* recv, int64_t K_rows, const int32_t* slot, const float* topk_w, int64_t S,
                             int k, int cpr, void* y, hipStream_t st) {
    const vec16* r = static_cast<const vec16*>(recv);
    vec16* out = static_cast<vec16*>(y);
    if (combine_by_wave(S, cpr, k)) {
        const int wpr = row_waves(cpr);
        const dim3 grid = grid_of(ceil_div(S * (int64_t)wpr, kThreads / 64 * U), kThreads), block(kThreads);
        launch_kernel(combine_kernel<DT, KK, U, UNITW, ST, LD>, grid, block, st, r, K_rows, slot, topk_w, S, k, cpr, wpr, pow2_shift(wpr), out);
    } else {
        const int64_t total = S * (int64_t)cpr;
        const dim3 grid = grid_of(ceil_div(total, kThreads * U), kThreads), block(kThreads);
        launch_kernel(combine_flat_kernel<DT, KK, U, UNITW, ST, LD>, grid, block, st, r, K_rows, slot, topk_w, total, k, cpr, pow2_shift(cpr), out);
    }
}

template <int DT, int KK, int U, bool UNITW>
static void launch_combine_k(const void* recv, int64_t K_rows, const int32_t* slot, const float* topk_w, int64_t S,
                             int k, int cpr, void* y, hipStream_t st) {
    const bool by_wave = combine_by_wave(S, cpr, k);
    const bool out = combine_store(row_lines(y, cpr), S, cpr, k, by_wave) == kStoreOut;
    if constexpr (UNITW) {
        // what dispatch_bwd_load keeps has two choices at most and shares lines, which combine_store streams (behind a recv that begins
        // within a line y may have whole ones: then recv streams too)
        if constexpr (KK == 1 || KK == 2) {
            if (dispatch_bwd_load(row_lines(recv, cpr), S, cpr, k, by_wave) == kLoadKeep && !out)
                return launch_combine_s<DT, KK, U, true, kStoreStream, kLoadKeep>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
        }
    } else if (combine_load(S, K_rows, cpr, k, row_lines(recv, cpr)) == kLoadKeep) {
        if (out) return launch_combine_s<DT, KK, U, false, kStoreOut, kLoadKeep>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
        return launch_combine_s<DT, KK, U, false, kStoreStream, kLoadKeep>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    }
    if (out) launch_combine_s<DT, KK, U, UNITW, kStoreOut, kLoadStream>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else launch_combine_s<DT, KK, U, UNITW, kStoreStream, kLoadStream>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
}

template <int DT, bool UNITW>
static void launch_combine(const void* recv, int64_t K_rows, const int32_t* slot, const float* topk_w, int64_t S,
                           int k, int cpr, void* y, hipStream_t st) {
    TraceScope tr(UNITW ? "dispatch_bwd_kernel" : "combine_kernel", st);
    if (k == 1)
        launch_combine_k<DT, 1, 2, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else if (k == 2)
        launch_combine_k<DT, 2, 1, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else if (k == 3)
        launch_combine_k<DT, 3, 1, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else if (k == 4)
        launch_combine_k<DT, 4, 1, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else
        launch_combine_k<DT, 0, 1, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
}

template <bool UNITW>
static void launch_combine_typed(int dtype, const void* recv, int64_t K_rows, const int32_t* slot, const float* topk_w,
                                 int64_t S, int k, int cpr, void* y, hipStream_t st) {
    if (dtype == TAMOE_F32)
        launch_combine<TAMOE_F32, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else if (dtype == TAMOE_F16)
        launch_combine<TAMOE_F16, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else
        launch_combine<TAMOE_BF16, UNITW>(recv, K_rows, slot, topk_w, S, k, cpr, y, st);
}

}  // namespace tamoe

using namespace tamoe;

static int combine_entry(const char* fn, const void* recv, int64_t K_rows, const int32_t* slot, const float* topk_w,
                         bool weighted, int dtype, int64_t S, int d, int k, void* y, void* stream) {
    clear_error();
    int rc;
    if (S < 0 || K_rows < 0) return fail(TAMOE_INVALID_ARG, "%s: S and K_rows must not be negative", fn);
    if (k <= 0) return fail(TAMOE_INVALID_ARG, "%s: k = %d must be positive", fn, k);
    if (k > TAMOE_MAX_K) return fail(TAMOE_UNSUPPORTED, "%s: k = %d exceeds the limit of %d", fn, k, TAMOE_MAX_K);
    if (S * (int64_t)k >= (int64_t)1 << 31) return fail(TAMOE_UNSUPPORTED, "%s: S*k does not fit int32", fn);
    int cpr = 0;   // 16-byte chunks per row
    if ((rc = check_rows(fn, dtype, d, &cpr)) != TAMOE_OK) return rc;
    if (S == 0) return TAMOE_OK;
    if (K_rows > 0 && (rc = check_ptr(fn, weighted ? "recv" : "d_send", recv, 16)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "slot", slot, 4)) != TAMOE_OK) return rc;
    if (weighted && (rc = check_ptr(fn, "topk_w", topk_w, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, weighted ? "y" : "d_x", y, 16)) != TAMOE_OK) return rc;
    if (ceil_div(S * (int64_t)cpr, kThreads * 1) > 0x7fffffff ||
        (rows_by_wave(cpr) && ceil_div(S * (int64_t)row_waves(cpr), kThreads / 64) > 0x7fffffff))
        return fail(TAMOE_UNSUPPORTED, "%s: the output is too large for one launch", fn);
    hipStream_t st = static_cast<hipStream_t>(stream);
    K_rows = slot_bound(K_rows);
    if (weighted)
        launch_combine_typed<false>(dtype, recv, K_rows, slot, topk_w, S, k, cpr, y, st);
    else   // unit weights (tamoe_dispatch_bwd)
        launch_combine_typed<true>(dtype, recv, K_rows, slot, nullptr, S, k, cpr, y, st);
    return check_launch(fn, "combine_kernel");
}

extern "C" int tamoe_combine(const void* recv, int64_t K_rows, const int32_t* slot, const float* topk_w, int dtype,
                             int64_t S, int d, int k, void* y, void* stream) {
    return combine_entry("tamoe_combine", recv, K_rows, slot, topk_w, true, dtype, S, d, k, y, stream);
}

extern "C" int tamoe_dispatch_bwd(const void* d_send, int64_t K_rows, const int32_t* slot, int dtype, int64_t S, int d,
                                  int k, void* d_x, void* stream) {
    return combine_entry("tamoe_dispatch_bwd", d_send, K_rows, slot, nullptr, false, dtype, S, d, k, d_x, stream);
}
