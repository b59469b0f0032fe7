// Backward of the path, for training with the auxiliary loss added to the train loss (paper
// Sections 3.1 and 4.3):
//   tamoe_gate_bwd     gradient to the gate scores through the softmax: from the combine weights
//                      and from l_topo (or l_aux), routing fixed
//   tamoe_combine_bwd  transpose of the combine: d_recv (weighted scatter of dy) and d_topk_w
//                      (one dot product per kept pair)
// (tamoe_dispatch_bwd, the transpose of the scatter, is the combine kernel with unit weights.)
#include <type_traits>

#include "chunk.h"
#include "internal.h"

namespace tamoe {

constexpr int kThreads = 256;

// ---- combine backward ---------------------------------------------------------------------------
// One 16-byte chunk per thread, like the forward row movers: a thread requests its chunk of dy and of the
// k source rows, then stores its k products.  A loop of such steps would wait for the stores of one step
// before the loads of the next are back (stores and loads retire in one order): one wavefront per
// token took 146 us where this takes 90 (bf16, 32768 x 768, k = 4; 34 -> 10 us for 65536 rows of 128 bytes).  d_w is a
// fixed-order sum: a butterfly over the lanes of a row segment, then the row's segments in ascending order.
//
// Rows of 64 chunks and more: a row takes whole wavefronts of one workgroup (ceil(cpr / 64) of them, at
// most kRowWaves, each of which takes every kRowWaves-th segment of a longer row), several rows share a
// workgroup of four wavefronts.  KK > 0: k is the compile-time constant KK; KK == 0: any k.
// ST: how d_recv is stored (combine_bwd_store).
constexpr int kRowWaves = 16;

template <int DT, int KK, int ST, int LD>
__global__ __launch_bounds__(kRowWaves * 64) void combine_bwd_kernel(
    const vec16* __restrict__ dy, const vec16* __restrict__ recv, int64_t K_rows, const int32_t* __restrict__ slot,
    const float* __restrict__ topk_w, int64_t S, int k_arg, int cpr, int row_waves, vec16* __restrict__ d_recv,
    float* __restrict__ d_w) {
    constexpr int KM = KK > 0 ? KK : TAMOE_MAX_K;
    const int k = KK > 0 ? KK : k_arg;
    __shared__ float part[kRowWaves][KM];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rows = (int)(blockDim.x >> 6) / row_waves;                     // rows of this workgroup
    const int in_wg = wave / row_waves, seg0 = wave - in_wg * row_waves;
    const int64_t t64 = (int64_t)linear_block() * rows + in_wg;
    const bool live = t64 < S;                                               // the same for the whole wavefront
    const int t = (int)(live ? t64 : S - 1);
    int32_t s[KM];
    float w[KM], dot[KM];
    bool use[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        const int64_t p = (int64_t)t * k + (KK > 0 || j < k ? j : k - 1);
        s[j] = __builtin_amdgcn_readfirstlane(slot[p]);
        w[j] = topk_w[p];
        dot[j] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        use[j] = live && (KK > 0 || j < k) && (uint32_t)s[j] < (uint64_t)K_rows;   // a dropped pair is -1
        s[j] = use[j] ? s[j] : 0;
    }
    const RowBuffer gy(dy + (size_t)t * cpr, cpr, live);
    for (int seg = seg0; seg * 64 < cpr; seg += row_waves) {
        const int c = seg * 64 + lane;
        const vec16 g = gy.template load<LD>(c);
        vec16 r[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) r[j] = RowBuffer(recv + (size_t)s[j] * cpr, cpr, use[j]).template load<LD>(c);
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            dot[j] = chunk_dot<DT>(g, r[j], dot[j]);
            float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            Chunk<DT>::fma(acc, w[j], g);
            RowBuffer(d_recv + (size_t)s[j] * cpr, cpr, use[j]).template store<ST>(c, Chunk<DT>::pack(acc));
        }
    }
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        float v = dot[j];
        v += __shfl_xor(v, 32);
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 8);
        v += __shfl_xor(v, 4);
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 1);
        if (lane == 0) part[wave][j] = use[j] ? v : 0.f;   // g may hold infinities: zeros for r are not enough
    }
    __syncthreads();
    if (live && seg0 == 0 && lane < k) {
        float v = 0.f;
        for (int i = 0; i < row_waves; ++i) v += part[wave + i][lane];
        d_w[(int64_t)t * k + lane] = v;
    }
}

// Other rows (fewer than 64 chunks): a row takes G consecutive lanes (the power of two that holds it).  More
// than four choices (KK == 0) are taken four at a time, as in combine_flat_kernel.
template <int DT, int KK, int ST, int LD>
__global__ __launch_bounds__(kThreads) void combine_bwd_short_kernel(
    const vec16* __restrict__ dy, const vec16* __restrict__ recv, int64_t K_rows, const int32_t* __restrict__ slot,
    const float* __restrict__ topk_w, int64_t S, int k_arg, int cpr, int g_shift, vec16* __restrict__ d_recv,
    float* __restrict__ d_w) {
    constexpr int KG = KK > 0 ? KK : 4;
    const int k = KK > 0 ? KK : k_arg;
    const int64_t i = (int64_t)linear_block() * kThreads + threadIdx.x;
    const int c = (int)i & ((1 << g_shift) - 1);
    const bool live = (i >> g_shift) < S;
    const int t = (int)(live ? i >> g_shift : S - 1);
    const bool inside = live && c < cpr;
    vec16 g = vec16{0u, 0u, 0u, 0u};
    if (inside) g = load_chunk<LD>(dy + (size_t)t * cpr + c);
#pragma unroll 1
    for (int j0 = 0; j0 < k; j0 += KG) {
        int32_t s[KG];
        float w[KG], dot[KG];
        vec16 r[KG];
#pragma unroll
        for (int j = 0; j < KG; ++j) {
            const bool there = KK > 0 || j0 + j < k;
            const int64_t p = (int64_t)t * k + (there ? j0 + j : k - 1);
            s[j] = there ? slot[p] : -1;
            w[j] = topk_w[p];
        }
#pragma unroll
        for (int j = 0; j < KG; ++j) {
            s[j] = (inside && s[j] >= 0 && (int64_t)s[j] < K_rows) ? s[j] : -1;
            r[j] = vec16{0u, 0u, 0u, 0u};
            if (s[j] >= 0) r[j] = load_chunk<LD>(recv + (size_t)s[j] * cpr + c);
        }
#pragma unroll
        for (int j = 0; j < KG; ++j) {
            dot[j] = chunk_dot<DT>(g, r[j], 0.f);
            float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            Chunk<DT>::fma(acc, w[j], g);
            const vec16 o = Chunk<DT>::pack(acc);
            if (s[j] >= 0) store_chunk<ST>(d_recv + (size_t)s[j] * cpr + c, o);
        }
#pragma unroll
        for (int j = 0; j < KG; ++j) {
            float v = dot[j];
            for (int m = (1 << g_shift) >> 1; m > 0; m >>= 1) v += __shfl_xor(v, m);
            // lane c == 0 has its chunk, so s[j] is -1 for a dropped pair alone (g may hold infinities)
            if (live && c == 0 && (KK > 0 || j0 + j < k)) d_w[(int64_t)t * k + j0 + j] = s[j] >= 0 ? v : 0.f;
        }
    }
}

// ---- gate backward ------------------------------------------------------------------------------
// value of lane (lane ^ MASK), MASK < 32, through the LDS crossbar
template <int MASK>
__device__ __forceinline__ float lane_xor(float v) {
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), (MASK << 10) | 0x1f));
}
template <int LPT>
__device__ __forceinline__ float butterfly_max(float v) {
    if constexpr (LPT > 1) v = fmaxf(v, lane_xor<1>(v));
    if constexpr (LPT > 2) v = fmaxf(v, lane_xor<2>(v));
    if constexpr (LPT > 4) v = fmaxf(v, lane_xor<4>(v));
    if constexpr (LPT > 8) v = fmaxf(v, lane_xor<8>(v));
    if constexpr (LPT > 16) v = fmaxf(v, lane_xor<16>(v));
    return v;
}
template <int LPT>
__device__ __forceinline__ float butterfly_sum(float v) {
    if constexpr (LPT > 1) v += lane_xor<1>(v);
    if constexpr (LPT > 2) v += lane_xor<2>(v);
    if constexpr (LPT > 4) v += lane_xor<4>(v);
    if constexpr (LPT > 8) v += lane_xor<8>(v);
    if constexpr (LPT > 16) v += lane_xor<16>(v);
    return v;
}

// A token's score row is spread over LPT consecutive lanes, four consecutive experts per lane
// (4*LPT >= N), so that a wavefront reads and writes whole rows contiguously; the three
// reductions of a row (max, sum of exponentials, sum of u*G) are butterflies over those lanes.
//   u[e]  = coef[e] + sum_j d_w[t][j] * [idx[t][j] == e],   coef[e] = scale * p[e] * c[e]
//   dl[e] = G[e] * (u[e] - sum_e' u[e'] G[e'])
// VEC: N is a multiple of 4, rows are 16-byte aligned and each lane moves one dwordx4.
// Latency at most sizes: a lane requests its scores, its four penalties and counts and the token's pairs before it waits
// for anything.  (With the coefficients made once per workgroup in LDS behind a barrier, the pairs requested one after the
// other and ordinary stores the three backward calls took, before and now: 16384 x 64, 64 experts, two choices and rows
// of 2 KiB 48.2 us, 47.3, four choices and rows of 128 bytes 15.0, 13.7; 65536, 128 experts, eight 61.8, 55.1.)
// KK > 0: k is the compile-time constant KK; KK == 0: any k.
template <int LPT, bool VEC, int KK>
__global__ __launch_bounds__(kThreads) void gate_bwd_kernel(const float* __restrict__ logits,
                                                            const int32_t* __restrict__ idx,
                                                            const float* __restrict__ d_w,
                                                            const float* __restrict__ penalty,
                                                            const int32_t* __restrict__ c, float scale, int64_t S,
                                                            int N, int k_arg, float* __restrict__ d_logits) {
    constexpr int KM = KK > 0 ? KK : TAMOE_MAX_K;
    const int k = KK > 0 ? KK : k_arg;
    const int tid = threadIdx.x;
    const int64_t token = ((int64_t)linear_block() * kThreads + tid) / LPT;
    const int e0 = (tid % LPT) * 4;
    const bool token_ok = token < S;
    const int64_t tk = token_ok ? token : 0;
    const float* row = logits + (size_t)tk * N;

    float l[4];
    if (VEC) {
        const float4 q = *reinterpret_cast<const float4*>(row + (e0 < N ? e0 : 0));
        l[0] = q.x; l[1] = q.y; l[2] = q.z; l[3] = q.w;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) l[i] = row[e0 + i < N ? e0 + i : 0];
    }
    // zeros beyond N
    const __amdgpu_buffer_rsrc_t cb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(c), 0, N * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t pb =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(penalty), 0, penalty != nullptr ? N * 4 : 0, 0x00020000);
    const int4 cnt = __builtin_bit_cast(int4, __builtin_amdgcn_raw_buffer_load_b128(cb, e0 * 4, 0, 0));
    const float4 pen = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(pb, e0 * 4, 0, 0));
    int sel[KM];
    float dw[KM];
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        const int64_t p = tk * k + (KK > 0 || j < k ? j : k - 1);
        sel[j] = idx[p];
        dw[j] = d_w[p];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) l[i] = (token_ok && e0 + i < N) ? l[i] : -INFINITY;

    float mx = butterfly_max<LPT>(fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])));
    if (!token_ok) mx = 0.f;
    float g[4], part = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        g[i] = __builtin_amdgcn_exp2f((l[i] - mx) * 1.44269504088896340736f);
        part += g[i];
    }
    const float den = butterfly_sum<LPT>(part);
    const float inv = token_ok ? 1.0f / den : 0.f;
    const float pe[4] = {pen.x, pen.y, pen.z, pen.w};
    const int32_t ce[4] = {cnt.x, cnt.y, cnt.z, cnt.w};
    float u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        g[i] *= inv;
        u[i] = scale * (penalty != nullptr ? pe[i] : 1.0f) * (float)ce[i];
    }
#pragma unroll
    for (int j = 0; j < KM; ++j) {
        const bool there = token_ok && (KK > 0 || j < k);
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] += there && sel[j] == e0 + i ? dw[j] : 0.f;
    }
    float ub = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) ub = __builtin_fmaf(u[i], g[i], ub);
    const float ubar = butterfly_sum<LPT>(ub);
    if (token_ok) {
        float* out = d_logits + (size_t)token * N;
        if (VEC) {
            if (e0 < N)
                store_chunk<kStoreThrough>(reinterpret_cast<vec16*>(out + e0),
                                           vec16{__float_as_uint(g[0] * (u[0] - ubar)), __float_as_uint(g[1] * (u[1] - ubar)),
                                                 __float_as_uint(g[2] * (u[2] - ubar)), __float_as_uint(g[3] * (u[3] - ubar))});
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (e0 + i < N) out[e0 + i] = g[i] * (u[i] - ubar);
        }
    }
}

template <int LPT>
static void launch_gate_bwd(const float* logits, const int32_t* idx, const float* d_w, const float* penalty,
                            const int32_t* c, float scale, int64_t S, int N, int k, float* d_logits, hipStream_t st) {
    const dim3 grid = grid_of(ceil_div(S * LPT, kThreads), kThreads), block(kThreads);
    const bool vec = N % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(d_logits) % 16 == 0;
#define TAMOE_GATE_BWD(KK)                                                                                              \
    do {                                                                                                                \
        if (vec)                                                                                                        \
            launch_kernel(gate_bwd_kernel<LPT, true, KK>, grid, block, st, logits, idx, d_w, penalty, c, scale, S, N, k, d_logits);  \
        else                                                                                                            \
            launch_kernel(gate_bwd_kernel<LPT, false, KK>, grid, block, st, logits, idx, d_w, penalty, c, scale, S, N, k, d_logits); \
    } while (0)
    if (k == 1) TAMOE_GATE_BWD(1);
    else if (k == 2) TAMOE_GATE_BWD(2);
    else TAMOE_GATE_BWD(0);
#undef TAMOE_GATE_BWD
}

template <int DT, int KK, int ST, int LD>
static void launch_combine_bwd_s(const vec16* dy, const vec16* recv, int64_t K_rows, const int32_t* slot,
                                 const float* topk_w, int64_t S, int k, int cpr, vec16* d_recv, float* d_w,
                                 hipStream_t st) {
    if (rows_by_wave(cpr)) {
        const int rw = row_waves(cpr) < kRowWaves ? row_waves(cpr) : kRowWaves;
        const int rows = rw < 4 ? 4 / rw : 1;
        const dim3 grid = grid_of(ceil_div(S, rows), rows * rw * 64), block(rows * rw * 64);
        launch_kernel(combine_bwd_kernel<DT, KK, ST, LD>, grid, block, st, dy, recv, K_rows, slot, topk_w, S, k, cpr, rw, d_recv, d_w);
    } else {
        int g_shift = 0;
        while ((1 << g_shift) < cpr) ++g_shift;
        const dim3 grid = grid_of(ceil_div(S << g_shift, kThreads), kThreads), block(kThreads);
        launch_kernel(combine_bwd_short_kernel<DT, KK, ST, LD>, grid, block, st, dy, recv, K_rows, slot, topk_w, S, k, cpr, g_shift, d_recv, d_w);
    }
}

template <int DT, int KK>
static void launch_combine_bwd_k(const vec16* dy, const vec16* recv, int64_t K_rows, const int32_t* slot,
                                 const float* topk_w, int64_t S, int k, int cpr, vec16* d_recv, float* d_w,
                                 hipStream_t st) {
    const StorePolicy policy = combine_bwd_store(row_lines(d_recv, cpr), S, cpr, k);
    const bool keep = combine_bwd_load(row_lines(recv, cpr), S, cpr, k) == kLoadKeep;
    const auto launch = [&](auto st_c) {
        constexpr int ST = decltype(st_c)::value;
        if (keep) launch_combine_bwd_s<DT, KK, ST, kLoadKeep>(dy, recv, K_rows, slot, topk_w, S, k, cpr, d_recv, d_w, st);
        else launch_combine_bwd_s<DT, KK, ST, kLoadStream>(dy, recv, K_rows, slot, topk_w, S, k, cpr, d_recv, d_w, st);
    };
    if constexpr (KK == 1)   // one choice alone
        if (policy == kStoreStream) return launch(std::integral_constant<int, kStoreStream>{});
    if (policy == kStoreBack) launch(std::integral_constant<int, kStoreBack>{});
    else launch(std::integral_constant<int, kStoreThrough>{});
}

template <int DT>
static void launch_combine_bwd(const void* dy, const void* recv, int64_t K_rows, const int32_t* slot,
                               const float* topk_w, int64_t S, int k, int cpr, void* d_recv, float* d_w,
                               hipStream_t st) {
    const vec16* g = static_cast<const vec16*>(dy);
    const vec16* r = static_cast<const vec16*>(recv);
    vec16* o = static_cast<vec16*>(d_recv);
    TraceScope tr("combine_bwd_kernel", st);
    if (k == 1)
        launch_combine_bwd_k<DT, 1>(g, r, K_rows, slot, topk_w, S, k, cpr, o, d_w, st);
    else if (k == 2)
        launch_combine_bwd_k<DT, 2>(g, r, K_rows, slot, topk_w, S, k, cpr, o, d_w, st);
    else if (k == 3)
        launch_combine_bwd_k<DT, 3>(g, r, K_rows, slot, topk_w, S, k, cpr, o, d_w, st);
    else if (k == 4)
        launch_combine_bwd_k<DT, 4>(g, r, K_rows, slot, topk_w, S, k, cpr, o, d_w, st);
    else
        launch_combine_bwd_k<DT, 0>(g, r, K_rows, slot, topk_w, S, k, cpr, o, d_w, st);
}

}  // namespace tamoe

using namespace tamoe;

extern "C" int tamoe_combine_bwd(const void* dy, const void* recv, int64_t K_rows, const int32_t* slot,
                                 const float* topk_w, int dtype, int64_t S, int d, int k, void* d_recv,
                                 float* d_topk_w, void* stream) {
    const char* fn = "tamoe_combine_bwd";
    clear_error();
    int rc;
    if (S < 0 || K_rows < 0) return fail(TAMOE_INVALID_ARG, "%s: S and K_rows must not be negative", fn);
    if (k <= 0) return fail(TAMOE_INVALID_ARG, "%s: k = %d must be positive", fn, k);
    if (k > TAMOE_MAX_K) return fail(TAMOE_UNSUPPORTED, "%s: k = %d exceeds the limit of %d", fn, k, TAMOE_MAX_K);
    if (S * (int64_t)k >= (int64_t)1 << 31) return fail(TAMOE_UNSUPPORTED, "%s: S*k does not fit int32", fn);
    int cpr = 0;   // 16-byte chunks per row
    if ((rc = check_rows(fn, dtype, d, &cpr)) != TAMOE_OK) return rc;
    if (S == 0) return TAMOE_OK;
    if ((rc = check_ptr(fn, "dy", dy, 16)) != TAMOE_OK) return rc;
    if (K_rows > 0 && (rc = check_ptr(fn, "recv", recv, 16)) != TAMOE_OK) return rc;
    if (K_rows > 0 && (rc = check_ptr(fn, "d_recv", d_recv, 16)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "slot", slot, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "topk_w", topk_w, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "d_topk_w", d_topk_w, 4)) != TAMOE_OK) return rc;
    if (S > 0x7fffffff) return fail(TAMOE_UNSUPPORTED, "%s: too many tokens for one launch", fn);
    hipStream_t st = static_cast<hipStream_t>(stream);
    K_rows = slot_bound(K_rows);
    if (dtype == TAMOE_F32)
        launch_combine_bwd<TAMOE_F32>(dy, recv, K_rows, slot, topk_w, S, k, cpr, d_recv, d_topk_w, st);
    else if (dtype == TAMOE_F16)
        launch_combine_bwd<TAMOE_F16>(dy, recv, K_rows, slot, topk_w, S, k, cpr, d_recv, d_topk_w, st);
    else
        launch_combine_bwd<TAMOE_BF16>(dy, recv, K_rows, slot, topk_w, S, k, cpr, d_recv, d_topk_w, st);
    return check_launch(fn, "combine_bwd_kernel");
}

extern "C" int tamoe_gate_bwd(const float* logits, const int32_t* topk_idx, const float* d_topk_w,
                              const float* penalty, const int32_t* c_expert, float loss_scale, int64_t S, int N, int P,
                              int k, float* d_logits, void* stream) {
    const char* fn = "tamoe_gate_bwd";
    clear_error();
    int rc;
    if ((rc = check_shape(fn, S, N, P, k)) != TAMOE_OK) return rc;
    if (S == 0) return TAMOE_OK;
    if ((rc = check_ptr(fn, "logits", logits, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "topk_idx", topk_idx, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "d_topk_w", d_topk_w, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "c_expert", c_expert, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "d_logits", d_logits, 4)) != TAMOE_OK) return rc;
    if (penalty != nullptr && (rc = check_ptr(fn, "penalty", penalty, 4)) != TAMOE_OK) return rc;
    // d l_topo / d G[t][e] = loss_scale * N*P * p[e] * c[e] / S^2 (l_aux: no N*P, unit weights); the
    // part that does not depend on e is folded into one fp32 factor on the host, in double
    const float scale =
        (float)((double)loss_scale * (penalty != nullptr ? (double)N * (double)P : 1.0) / ((double)S * (double)S));
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (ceil_div(S * 32, kThreads) > 0x7fffffff) return fail(TAMOE_UNSUPPORTED, "%s: too many tokens for one launch", fn);
    {
        TraceScope tr("gate_bwd_kernel", st);
        if (N <= 4)
            launch_gate_bwd<1>(logits, topk_idx, d_topk_w, penalty, c_expert, scale, S, N, k, d_logits, st);
        else if (N <= 8)
            launch_gate_bwd<2>(logits, topk_idx, d_topk_w, penalty, c_expert, scale, S, N, k, d_logits, st);
        else if (N <= 16)
            launch_gate_bwd<4>(logits, topk_idx, d_topk_w, penalty, c_expert, scale, S, N, k, d_logits, st);
        else if (N <= 32)
            launch_gate_bwd<8>(logits, topk_idx, d_topk_w, penalty, c_expert, scale, S, N, k, d_logits, st);
        else if (N <= 64)
            launch_gate_bwd<16>(logits, topk_idx, d_topk_w, penalty, c_expert, scale, S, N, k, d_logits, st);
        else
            launch_gate_bwd<32>(logits, topk_idx, d_topk_w, penalty, c_expert, scale, S, N, k, d_logits, st);
    }
    return check_launch(fn, "gate_bwd_kernel");
}
