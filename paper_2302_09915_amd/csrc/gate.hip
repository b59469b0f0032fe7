// tamoe_gate / tamoe_select: gate scores, softmax, top-k and the load statistics
// (paper Section 3.1: gate network G with softmax, top-k experts per token, c_ie, m_i;
// Section 4.1: per-destination-device volume).
//
// gate_bf16_kernel / gate_f16_kernel / gate_f32_kernel (one tile code, three element types), and gate_direct_kernel for
// small tiles (launch_gate_small): the one dense contraction of the path, on the matrix cores.  v_mfma_f32_32x32x16_bf16 (or _f16; fp32 operands
// are split into three bf16 parts each) with A = a 32-expert block of W and B = 32 tokens of x,
// both from LDS tiles filled by coalesced loads of 128-byte K chunks.  The scores of a workgroup's tokens
// end in an LDS tile; softmax and top-k read it with a token over 4 to 16 lanes, so that all
// wavefronts share the selection however the contraction was split between them.
// The kernel is bound by the HBM read of x (intensity ~N flop/byte), not by the MFMA rate.
//
// tamoe_select runs the same selection code on a score matrix in memory (select_kernel).
//
// Determinism: probability sums are reduced in a fixed tree (lanes, wavefronts, workgroups);
// counts are integers.  A second small kernel folds the per-workgroup partials.
#include "gate_tile.h"
#include "scan128.h"

namespace tamoe {

// Selection stage on a score matrix in memory: 8 wavefronts, 64 tokens per workgroup, the lanes of a token read its
// scores straight from memory.  (With 32 tokens per wavefront, staged through LDS into the accumulator layout: 512 x 8
// 7.6 -> 6.3 us, 16384 x 64 two choices 10.3 -> 7.3, eight 33.7 -> 10.4, 65536 x 128 18.5 -> 17.5, 262144 x 127 151 -> 50.)
constexpr int kSelectTokens = 64;

template <int NB>
__global__ __launch_bounds__(512) void select_kernel(const float* __restrict__ logits, int64_t S, int N, int k,
                                                     int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                     const GateStats gs) {
    constexpr int ROWS = NB * 32, WAVES = 8, TOK = kSelectTokens;
    __shared__ float m_w[WAVES * ROWS];
    __shared__ int32_t pairs[TAMOE_MAX_K * ROWS];
    __shared__ signed char sel[TOK * TAMOE_MAX_K];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile0 = (int64_t)linear_block() * TOK;
    if (tile0 >= S) return;   // past the last tile (grid_of)
    auto load_scores = [&](int tl, int q, auto& sc) {   // a token's lanes read consecutive pieces
        using SG = SelectGeom<NB, WAVES, TOK>;
        const int64_t t = tile0 + tl < S ? tile0 + tl : S - 1;
#pragma unroll
        for (int c = 0; c < SG::EPL; ++c) {
            const int e = SG::expert_at(c, q);
            sc[c] = logits[t * N + (e < N ? e : N - 1)];
        }
    };
    select_tokens<NB, WAVES, TOK>(load_scores, lane, wave, tile0, S, N, k, nullptr, topk_idx, topk_w, sel,
                                  m_w + wave * ROWS);
    finish_block<NB, WAVES, TOK>(m_w, sel, nullptr, pairs, lane, wave, tile0, S, N, k, gs);
}

// Fixed-order sums of the per-workgroup partials: one workgroup per expert, then one per device (E experts).
// entries = k * n_blocks.  Latency only: each thread requests four words at a time without a branch, and one barrier
// joins the wavefronts.  (With the sums of a device's experts one after the other in its first expert's workgroup,
// two waits and nine barriers each: 16 experts per device, 16384 tokens 23.8 -> 3.7 us; 32 per device, 65536
// tokens, k = 8 90.7 -> 7.8; 3 per device, 5003 tokens 6.8 -> 3.9.)
__global__ __launch_bounds__(256) void gate_finalize_kernel(const float* __restrict__ m_part,
                                                            const int32_t* __restrict__ tile_pairs, int n_blocks,
                                                            int entries, int pitch, int N, int E, int64_t S,
                                                            float* __restrict__ m, int32_t* __restrict__ c_expert,
                                                            int32_t* __restrict__ c_device) {
    __shared__ float fs[4];
    __shared__ int32_t cs[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    const bool device = b >= N;
    const int e0 = device ? (b - N) * E : b;
    const int rows = device ? E : 1;
    float s = 0.f;
    int32_t c = 0;
    const WordBuffer mrow(m_part + (size_t)e0 * n_blocks, device ? 0 : n_blocks);
    for (int i = tid; i < n_blocks; i += 1024)
        s += (mrow.load<float>(i) + mrow.load<float>(i + 256)) + (mrow.load<float>(i + 512) + mrow.load<float>(i + 768));
    // rows of the table start at multiples of 16 bytes; entries past the end of a row are padding of unknown content
    for (int q0 = 0; q0 < entries; q0 += 1024) {
        const int q = q0 + 4 * tid;
        const int32_t* at = tile_pairs + (size_t)e0 * pitch + (q < entries ? q : 0);
        const bool in0 = q < entries, in1 = q + 1 < entries, in2 = q + 2 < entries, in3 = q + 3 < entries;
#pragma unroll 4
        for (int r = 0; r < rows; ++r) {
            const int4 v = *reinterpret_cast<const int4*>(at + (size_t)r * pitch);
            c += ((in0 ? v.x : 0) + (in1 ? v.y : 0)) + ((in2 ? v.z : 0) + (in3 ? v.w : 0));
        }
    }
    s = wave_total(s);
    c = wave_total(c);
    if ((tid & 63) == 0) {
        fs[tid >> 6] = s;
        cs[tid >> 6] = c;
    }
    __syncthreads();
    if (tid == 0) {
        const int32_t total = (cs[0] + cs[1]) + (cs[2] + cs[3]);
        if (device) {
            c_device[b - N] = total;
        } else {
            m[e0] = S > 0 ? ((fs[0] + fs[1]) + (fs[2] + fs[3])) / (float)S : 0.f;
            c_expert[e0] = total;
        }
    }
}

// ---- host side ------------------------------------------------------------------------------

static void launch_select(int64_t blocks, hipStream_t st, const float* logits, int64_t S, int N, int k,
                          int32_t* topk_idx, float* topk_w, const GateStats& gs) {
    const dim3 grid = grid_of(blocks, 512), block(512);
    TraceScope tr("select_kernel", st);
    if (N <= 32)
        launch_kernel(select_kernel<1>, grid, block, st, logits, S, N, k, topk_idx, topk_w, gs);
    else if (N <= 64)
        launch_kernel(select_kernel<2>, grid, block, st, logits, S, N, k, topk_idx, topk_w, gs);
    else
        launch_kernel(select_kernel<4>, grid, block, st, logits, S, N, k, topk_idx, topk_w, gs);
}

int check_select_outputs(const char* fn, int64_t S, int32_t* topk_idx, float* topk_w, float* m, int32_t* c_expert,
                         int32_t* c_device, void* ws, size_t ws_bytes, const Workspace& lay) {
    int rc;
    if (S > 0) {
        if ((rc = check_ptr(fn, "topk_idx", topk_idx, 4)) != TAMOE_OK) return rc;
        if ((rc = check_ptr(fn, "topk_w", topk_w, 4)) != TAMOE_OK) return rc;
    }
    if ((rc = check_ptr(fn, "m", m, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "c_expert", c_expert, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "c_device", c_device, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "ws", ws, 256)) != TAMOE_OK) return rc;
    if (ws_bytes < lay.total)
        return fail(TAMOE_WORKSPACE_TOO_SMALL, "%s: workspace has %zu bytes, %zu needed", fn, ws_bytes, lay.total);
    return TAMOE_OK;
}

GateStats stats_in(void* ws, const Workspace& lay, int N, int k, int64_t blocks, bool compact) {
    GateStats gs{};
    gs.m_part = reinterpret_cast<float*>(static_cast<char*>(ws) + lay.m_part);
    gs.tile_pairs = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + lay.tile_pairs);
    gs.local_pos = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + lay.local_pos);
    gs.n_blocks = (int)blocks;
    gs.pitch = (int)pair_pitch(k, blocks);
    gs.counts = compact ? reinterpret_cast<uint16_t*>(gs.tile_pairs) : nullptr;
    gs.stride = count_stride(N, k);
    return gs;
}

int run_select_stage(const char* fn, const float* logits, int64_t S, int N, int k, int32_t* topk_idx, float* topk_w,
                     void* ws, const Workspace& lay, hipStream_t st, GateRun* run) {
    const int64_t blocks = ceil_div(S, kSelectTokens);
    if ((int64_t)k * blocks > 0x3fffffff) return fail(TAMOE_UNSUPPORTED, "%s: too many token tiles", fn);
    run->stats = stats_in(ws, lay, N, k, blocks, false);
    run->tile_tokens = kSelectTokens;
    if (blocks > 0) {
        launch_select(blocks, st, logits, S, N, k, topk_idx, topk_w, run->stats);
        return check_launch(fn, "select_kernel");
    }
    return TAMOE_OK;
}

int run_gate_stage(const char* fn, const void* x, const void* w, int dtype, int64_t S, int d, int N, int k,
                   float* logits, int32_t* topk_idx, float* topk_w, bool compact, void* ws, const Workspace& lay,
                   hipStream_t st, GateRun* run) {
    run->stats = stats_in(ws, lay, N, k, 0, compact);
    run->tile_tokens = 32;
    if (S <= 0) return TAMOE_OK;
    const int tokens = gate_tile_tokens(S, N);
    const int64_t blocks = ceil_div(S, tokens);
    if ((int64_t)k * blocks > 0x3fffffff) return fail(TAMOE_UNSUPPORTED, "%s: too many token tiles", fn);
    // the tile code addresses rows in 2-byte units: an fp32 row of d values is a row of 2*d units
    if (dtype == TAMOE_F32 && d > 0x3fffffff) return fail(TAMOE_UNSUPPORTED, "%s: d = %d is too large", fn, d);
    run->stats = stats_in(ws, lay, N, k, blocks, compact);
    run->tile_tokens = tokens;
    GateLaunch g{};
    g.tile_tokens = tokens;
    g.blocks = blocks;
    g.st = st;
    g.x = static_cast<const uint16_t*>(x);
    g.w = static_cast<const uint16_t*>(w);
    g.S = S;
    g.d_units = dtype == TAMOE_F32 ? 2 * d : d;
    g.N = N;
    g.k = k;
    g.logits = logits;
    g.topk_idx = topk_idx;
    g.topk_w = topk_w;
    g.stats = run->stats;
    if (dtype == TAMOE_F32)
        launch_gate_f32(g);
    else if (dtype == TAMOE_F16)
        launch_gate_f16(g);
    else
        launch_gate_bf16(g);
    return check_launch(fn, gate_kernel_name(dtype));
}

static int finalize(const char* fn, const GateRun& run, int N, int P, int k, int64_t S, float* m, int32_t* c_expert,
                    int32_t* c_device, hipStream_t st) {
    {
        TraceScope tr("gate_finalize_kernel", st);
        launch_kernel(gate_finalize_kernel, dim3(N + P), dim3(256), st, run.stats.m_part, run.stats.tile_pairs, run.stats.n_blocks,
                                                            k * run.stats.n_blocks, run.stats.pitch, N, N / P, S, m,
                                                            c_expert, c_device);
    }
    return check_launch(fn, "gate_finalize_kernel");
}

}  // namespace tamoe

using namespace tamoe;

extern "C" int tamoe_select(const float* logits, int64_t S, int N, int P, int k, int32_t* topk_idx, float* topk_w,
                            float* m, int32_t* c_expert, int32_t* c_device, void* ws, size_t ws_bytes, void* stream) {
    const char* fn = "tamoe_select";
    clear_error();
    int rc;
    if ((rc = check_shape(fn, S, N, P, k)) != TAMOE_OK) return rc;
    if (S > 0 && (rc = check_ptr(fn, "logits", logits, 4)) != TAMOE_OK) return rc;
    const Workspace lay = workspace_layout(S, N, k);
    if ((rc = check_select_outputs(fn, S, topk_idx, topk_w, m, c_expert, c_device, ws, ws_bytes, lay)) != TAMOE_OK)
        return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    GateRun run{};
    if ((rc = run_select_stage(fn, logits, S, N, k, topk_idx, topk_w, ws, lay, st, &run)) != TAMOE_OK) return rc;
    return finalize(fn, run, N, P, k, S, m, c_expert, c_device, st);
}

extern "C" int tamoe_gate(const void* x, const void* w, int dtype, int64_t S, int d, int N, int P, int k,
                          float* logits, int32_t* topk_idx, float* topk_w, float* m, int32_t* c_expert,
                          int32_t* c_device, void* ws, size_t ws_bytes, void* stream) {
    const char* fn = "tamoe_gate";
    clear_error();
    int rc;
    if ((rc = check_shape(fn, S, N, P, k)) != TAMOE_OK) return rc;
    if ((rc = check_rows(fn, dtype, d)) != TAMOE_OK) return rc;
    if (S > 0) {
        if ((rc = check_ptr(fn, "x", x, 16)) != TAMOE_OK) return rc;
        if ((rc = check_ptr(fn, "w", w, 16)) != TAMOE_OK) return rc;
    }
    const Workspace lay = workspace_layout(S, N, k);
    if ((rc = check_select_outputs(fn, S, topk_idx, topk_w, m, c_expert, c_device, ws, ws_bytes, lay)) != TAMOE_OK)
        return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    GateRun run{};
    if ((rc = run_gate_stage(fn, x, w, dtype, S, d, N, k, logits, topk_idx, topk_w, false, ws, lay, st, &run)) != TAMOE_OK)
        return rc;
    return finalize(fn, run, N, P, k, S, m, c_expert, c_device, st);
}
