// tamoe_gate_dispatch: the forward path up to the send buffer in two or three launches (paper Section 3.1:
// gate, softmax, top-k, l_aux and local capacity; Section 4.1: one merged delivery per device;
// Section 4.3: l_topo, variable chunk sizes).  Same results as tamoe_gate + tamoe_aux_loss +
// tamoe_dispatch.  tamoe_dispatch and tamoe_dispatch_padded take the same stages behind a kernel that ranks
// a routing that is given (run_dispatch).
//
//   1. the gate kernel (gate_tile.h), or route_rank_kernel for a given routing, leaves per token tile b the
//      number of pairs per (expert e, choice j) and for every pair its position among the pairs of
//      (b, e, j);
//   2. route_expert_kernel, one workgroup per expert: mean probability, count, the exclusive prefix of
//      the expert's pair counts in priority order (choice-major, then token order), kept rows.  Only
//      where the table of counts is large: a small one (kTableReads) is scanned by every
//      workgroup of the next kernel by itself, and this launch is left out;
//   3. route_copy_kernel: the scatter.  A pair's slot is offset[e] + prefix[e][j][b] + position, kept
//      iff prefix + position < cap[e]; offset[e] is the sum of the kept rows of the experts before e,
//      which every wavefront takes from the N kept counts by a scan of its own (two loads and a dozen
//      lane shifts: cheaper than one more pass over the experts in front of the scatter); every
//      thread derives the slots of its token on the way to moving its 16-byte chunk, and the thread
//      with the row's first chunk writes them to slot[].  The first workgroup writes what
//      describes the layer as a whole: expert offsets, rows per destination device, the loss; in the
//      fixed-size layout the last ones clear every expert's unused rows.
//      How rows are stored depends on what the caches can do for them (scatter_store).
#include <algorithm>

#include "gate_tile.h"
#include "internal.h"
#include "scan128.h"

namespace tamoe {

constexpr int kCopyThreads = 256;

// When the workgroups of the scatter scan the table of pair counts themselves: in one generation of
// workgroups (kTableBlocks, all resident) that read kTableReads counts together.  The kernel that this
// replaces takes 3 us and more on its own; the scan adds 0.6 us to 16 workgroups (512 x 64, 128 counts),
// 1.1 us to 512 (1024 x 2 KiB, 4096 counts), 3.3 us to 1024 with 4096 counts (4096 x 1 KiB: no gain), and
// 2.5 us to every generation of a longer launch (16384 x 4 KiB: 10 us).
constexpr int64_t kTableBlocks = 1024;
constexpr int64_t kTableReads = (int64_t)2 << 20;

// ---- a routing that is given ------------------------------------------------------------------------
// What the gate kernel leaves behind, from topk_idx: one workgroup of eight wavefronts per TOK tokens, of which each
// ranks 64 at a time for one choice.  An index outside [0, N) is no pair.
// Few tiles keep the table of counts small; but with 512 tokens whatever k, the wavefronts did k turns one after the
// other in a handful of workgroups.  Two turns each (512 tokens, from three choices 256, from five 128), while an
// expert's counts stay within the 1024 that route_expert_kernel takes in one pass: 600 tokens, k = 8 9.5 -> 4.1 us,
// 16384, k = 8 10.9 -> 6.2, 5003, k = 4 6.6 -> 4.6, 65536, k = 4 6.1 -> 5.1 (512 tokens throughout -> now).
// Never below the gate's tiles, for which the table has room.
static int rank_tokens(int64_t S, int N, int k) {
    int tok = k <= 2 ? 512 : k <= 4 ? 256 : 128;
    while (tok < 512 && (tok < gate_tile_tokens(S, N) || k * ceil_div(S, tok) > 1024)) tok *= 2;
    return tok;
}

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

// ---- the scatter ----------------------------------------------------------------------------------------
// What the kernels behind the ranking are given.
struct RouteArgs {
    const vec16* x;
    const int32_t* topk_idx;
    const int32_t* local_pos;
    const int32_t* table;       // pairs per (expert; choice, tile); their prefix once route_expert_kernel ran
    const int32_t* cap;         // may be NULL when pad_C > 0
    const float* m_part;        // [N][n_blocks] sums of gate probabilities, NULL for a given routing
    int32_t* slot;
    vec16* send;
    int64_t S;
    int N, P, k;
    int cpr, wpr, shift;        // chunks per row, wavefronts per row, log2 of wpr (flat: of cpr) or -1
    int n_blocks, pitch, tile_shift;
    int pad_C;                  // rows per expert of the fixed-size layout, 0: packed
    int copy_blocks, fill_parts;
    bool fill_streams;
    // outputs; m, c_expert, c_device and loss are NULL for a given routing, expert_offset and
    // send_count_dev in the fixed-size layout
    const float* penalty;
    float loss_scale;
    float* m;
    int32_t* c_expert;
    int32_t* c_device;
    float* loss;
    int32_t* kept_expert;
    int32_t* expert_offset;
    int32_t* send_count_dev;
};

// offset[e] = kept rows of the experts before e, for the (at most two) experts a lane is asked about:
// every wavefront scans the N <= 128 kept counts by itself.  Called by all 64 lanes.
struct WaveOffsets {
    int32_t ex0, ex1;   // exclusive prefix at expert lane, lane + 64
};
// The lane's two kept counts: requested at the top of a kernel, scanned (wave_offsets) only where the
// first offset is needed, so that the round trip runs beside the kernel's other loads.
struct KeptPair {
    int32_t k0, k1;
};
__device__ __forceinline__ KeptPair load_kept(const int32_t* __restrict__ kept_expert, int N) {
    static_assert(TAMOE_MAX_EXPERTS <= 128, "two experts per lane");
    const int lane = threadIdx.x & 63;
    return KeptPair{lane < N ? kept_expert[lane] : 0, lane + 64 < N ? kept_expert[lane + 64] : 0};
}
__device__ __forceinline__ WaveOffsets wave_offsets(const KeptPair& kp) {
    const int32_t i0 = wave_inclusive_scan(kp.k0);
    const int32_t i1 = wave_inclusive_scan(kp.k1) + __builtin_amdgcn_readlane(i0, 63);
    return WaveOffsets{i0 - kp.k0, i1 - kp.k1};
}
// e in [0, 128).  UNIFORM: e is the same in every lane (read through the scalar unit, no lane exchange);
// otherwise any value per lane, and all 64 lanes must take part.
template <bool UNIFORM>
__device__ __forceinline__ int32_t offset_of(const WaveOffsets& o, int e) {
    if constexpr (UNIFORM) {
        const int eu = __builtin_amdgcn_readfirstlane(e);
        const int32_t lo = __builtin_amdgcn_readlane(o.ex0, eu & 63), hi = __builtin_amdgcn_readlane(o.ex1, eu & 63);
        return eu < 64 ? lo : hi;
    } else {
        const int32_t lo = __shfl(o.ex0, e & 63), hi = __shfl(o.ex1, e & 63);
        return e < 64 ? lo : hi;
    }
}

// Lanes that share an expert's row of a table: all 256 threads over N experts, at most a wavefront each.
__device__ __forceinline__ int lanes_per_expert(int N) {
    int l = 64;
    while (l > 1 && l * N > kCopyThreads) l >>= 1;
    return l;
}

// The workgroup's own scan of a small table: kept[e] = min(pairs of e, its limit), and before[j][e] = pairs
// of e that precede choice j of token tile blk0.  kept, before (KM rows), total: LDS.  Every thread
// calls; ends with a barrier.
template <int KM>
__device__ __forceinline__ void scan_table(const RouteArgs& a, int blk0, int32_t* kept, int32_t (*before)[TAMOE_MAX_EXPERTS],
                                           int32_t* total) {
    const int lpe = lanes_per_expert(a.N);
    const int e = threadIdx.x / lpe, l = threadIdx.x & (lpe - 1);
    const int entries = a.k * a.n_blocks;
    if (e < a.N) {
        const int32_t lim = pair_limit(a.cap, e, a.pad_C);
        const int32_t* row = a.table + (size_t)e * a.pitch;
        int32_t sum = 0, bef[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) bef[j] = 0;
#pragma unroll 4
        for (int q = 4 * l; q < entries; q += 4 * lpe) {
            const int4 v = *reinterpret_cast<const int4*>(row + q);   // rows are padded to 64 entries
            const int32_t c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int32_t n = q + i < entries ? c[i] : 0;         // the padding holds anything
                sum += n;
#pragma unroll
                for (int j = 0; j < KM; ++j) bef[j] += q + i < j * a.n_blocks + blk0 ? n : 0;
            }
        }
        for (int sft = lpe >> 1; sft > 0; sft >>= 1) {
            sum += __shfl_xor(sum, sft);
#pragma unroll
            for (int j = 0; j < KM; ++j) bef[j] += __shfl_xor(bef[j], sft);
        }
        if (l == 0) {
            kept[e] = sum < lim ? sum : lim;
            if (total != nullptr) total[e] = sum;
            if (before != nullptr) {
#pragma unroll
                for (int j = 0; j < KM; ++j)
                    if (j < a.k) before[j][e] = bef[j];
            }
        }
    }
    __syncthreads();
}

// What describes the layer as a whole, by one workgroup that does nothing else
// (every thread calls): expert offsets (Section 4.3: what the size exchange carries), rows and pairs per
// destination device, the loss; with TABLE also what route_expert_kernel would have written.  N <= 128
// values: the first wavefront holds two experts per lane, scans and sums them with lane operations
// (fixed order), and hands offsets to the threads that write the per-device numbers through LDS.
template <bool TABLE>
__device__ __forceinline__ void route_layer_outputs(const RouteArgs& a) {
    __shared__ int32_t total[TAMOE_MAX_EXPERTS];
    __shared__ int32_t kept[TAMOE_MAX_EXPERTS];
    __shared__ float mean[TAMOE_MAX_EXPERTS];
    __shared__ int32_t off[TAMOE_MAX_EXPERTS + 1];
    const int tid = threadIdx.x;
    const int N = a.N;
    if constexpr (TABLE) {
        if (a.m != nullptr) {
            const int lpe = lanes_per_expert(N);
            const int e = tid / lpe, l = tid & (lpe - 1);
            if (e < N) {
                float s = 0.f;
#pragma unroll 4
                for (int b = l; b < a.n_blocks; b += lpe) s += a.m_part[(size_t)e * a.n_blocks + b];
                for (int sft = lpe >> 1; sft > 0; sft >>= 1) s += __shfl_xor(s, sft);
                if (l == 0) {
                    mean[e] = a.S > 0 ? s / (float)a.S : 0.f;
                    a.m[e] = mean[e];
                }
            }
        }
        scan_table<1>(a, 0, kept, nullptr, total);
        if (tid < N) {
            a.kept_expert[tid] = kept[tid];
            if (a.c_expert != nullptr) a.c_expert[tid] = total[tid];
        }
    } else {
        if (tid < N) {
            kept[tid] = a.kept_expert[tid];
            if (a.c_expert != nullptr) total[tid] = a.c_expert[tid];
            if (a.m != nullptr) mean[tid] = a.m[tid];
        }
        __syncthreads();
    }
    if (tid < 64) {
        const int e0 = tid, e1 = tid + 64;
        const int32_t k0 = e0 < N ? kept[e0] : 0, k1 = e1 < N ? kept[e1] : 0;
        const int32_t i0 = wave_inclusive_scan(k0);
        const int32_t i1 = wave_inclusive_scan(k1) + __builtin_amdgcn_readlane(i0, 63);
        off[e0] = i0 - k0;
        off[e1] = i1 - k1;
        if (e0 == N - 1) off[N] = i0;
        if (e1 == N - 1) off[N] = i1;
        if (a.loss != nullptr) {
            float t0 = 0.f, t1 = 0.f;
            if (e0 < N) t0 = mean[e0] * (float)total[e0] * (a.penalty != nullptr ? a.penalty[e0] : 1.f);
            if (e1 < N) t1 = mean[e1] * (float)total[e1] * (a.penalty != nullptr ? a.penalty[e1] : 1.f);
            float term = t0 + t1;
#pragma unroll
            for (int sft = 32; sft > 0; sft >>= 1) term += __shfl_xor(term, sft);
            if (tid == 0) a.loss[0] = term * a.loss_scale;
        }
    }
    __syncthreads();
    if (a.expert_offset != nullptr && tid <= N) a.expert_offset[tid] = off[tid];
    if (tid < a.P) {
        const int E = N / a.P;
        if (a.send_count_dev != nullptr) a.send_count_dev[tid] = off[(tid + 1) * E] - off[tid * E];
        if (a.c_device != nullptr) {
            int32_t c = 0;
            for (int q = 0; q < E; ++q) c += total[tid * E + q];
            a.c_device[tid] = c;
        }
    }
}

// The scatter with the slot assignment folded in.  Workgroup 0 writes the layer's outputs and moves no rows:
// as part of a copying workgroup that tail would end after every other workgroup of a short launch.
// Then copy_blocks workgroups move rows, and N * fill_parts clear the unused rows of the fixed-size
// layout.  ROWU: rows by whole wavefronts (scatter_by_wave), U segments each; otherwise U chunks per
// thread, flat.  ST: how rows are stored (scatter_store).  TABLE: no route_expert_kernel ran;
// the workgroup scans the table of pair counts itself.
// (What the copying workgroups read comes as arguments of its own: only a pointer that is declared not to
// alias is read through the scalar unit.  cap is never NULL here: without capacities it is the table, whose
// entries are then not looked at, so that no branch stands between the look-ups.)
template <int KK, int U, bool ROWU, int ST, bool TABLE>
__global__ __launch_bounds__(kCopyThreads) void route_copy_kernel(
    const vec16* __restrict__ x, const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ local_pos,
    const int32_t* __restrict__ tile_table, const int32_t* __restrict__ cap, int32_t* __restrict__ slot,
    vec16* __restrict__ send, const RouteArgs a) {
    const uint32_t wg = linear_block();
    if (wg == 0) {
        route_layer_outputs<TABLE>(a);
        return;
    }
    constexpr int KM = KK > 0 ? KK : TAMOE_MAX_K;
    __shared__ int32_t kept_w[TABLE ? TAMOE_MAX_EXPERTS : 1];
    __shared__ int32_t before_w[TABLE ? KM : 1][TABLE ? TAMOE_MAX_EXPERTS : 1];
    const int N = a.N, cpr = a.cpr;
    const int lane = threadIdx.x & 63;

    if (wg > (uint32_t)a.copy_blocks) {   // zero rows e*C + kept[e] .. (e+1)*C - 1, a share of them
        const int f = (int)(wg - 1 - (uint32_t)a.copy_blocks);
        if (f >= N * a.fill_parts) return;   // past the last workgroup (grid_of)
        const int e = f / a.fill_parts, part = f - e * a.fill_parts;
        if constexpr (TABLE) scan_table<1>(a, 0, kept_w, nullptr, nullptr);
        const int32_t used = TABLE ? kept_w[TABLE ? e : 0] : a.kept_expert[e];
        const int64_t n = (int64_t)(a.pad_C - used) * cpr;             // chunks to clear, >= 0
        const int64_t per = (n + a.fill_parts - 1) / a.fill_parts;
        const int64_t i0 = (int64_t)part * per;
        const int64_t i1 = i0 + per < n ? i0 + per : n;
        vec16* base = a.send + ((int64_t)e * a.pad_C + used) * cpr;
        const vec16 zero = {0u, 0u, 0u, 0u};
        if (a.fill_streams) {
            for (int64_t i = i0 + threadIdx.x; i < i1; i += kCopyThreads) store_chunk<kStoreStream>(base + i, zero);
        } else {
            for (int64_t i = i0 + threadIdx.x; i < i1; i += kCopyThreads) store_chunk<ST>(base + i, zero);
        }
        return;
    }

    const int k = KK > 0 ? KK : a.k;
    const uint32_t blk = wg - 1;
    const int64_t total = a.S * cpr;
    int tok[U], col[U], seg[U];
    bool inside[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (ROWU) {
            const uint32_t wv = (blk * (kCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * U + u;
            split_wave(wv, a.wpr, a.shift, tok[u], seg[u]);
            inside[u] = tok[u] < a.S;      // the same for the whole wavefront
            tok[u] = inside[u] ? tok[u] : (int)a.S - 1;
            col[u] = seg[u] * 64 + lane;
        } else {
            const int64_t c = (int64_t)blk * (kCopyThreads * U) + (int64_t)u * kCopyThreads + threadIdx.x;
            inside[u] = c < total;
            split_chunk(inside[u] ? c : total - 1, total, cpr, a.shift, tok[u], col[u]);
            seg[u] = col[u];               // 0: the row's first chunk
        }
    }
    // experts and positions of all choices, requested together
    int32_t e[U][KM], pos[U][KM];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            const int64_t p = (int64_t)tok[u] * k + (KK > 0 || j < k ? j : k - 1);
            e[u][j] = topk_idx[p];
            pos[u][j] = local_pos[p];
            if constexpr (ROWU) {
                e[u][j] = __builtin_amdgcn_readfirstlane(e[u][j]);
                pos[u][j] = __builtin_amdgcn_readfirstlane(pos[u][j]);
            }
        }
    // A small launch requests the row itself at once, whether or not a choice of its token is kept: behind
    // the two look-ups it would be a third memory round trip (5.9 -> 5.5 us for 1024 x 2 KiB).  A large one
    // is bound by bytes and leaves out the rows of dropped tokens (65536 x 8 KiB: 258 us, at once 262; half
    // the tokens of 16384 x 4 KiB dropped: 15.9 us, at once 17.2).
    vec16 v[U];
    if constexpr (TABLE) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (ROWU)
                v[u] = RowBuffer(x + (size_t)tok[u] * cpr, cpr, inside[u]).load(col[u]);
            else
                v[u] = __builtin_nontemporal_load(x + (size_t)tok[u] * cpr + col[u]);
        }
    }
    KeptPair kp = {0, 0};
    int blk0 = 0;
    if constexpr (TABLE) {
        // token tile of the workgroup's first token: the same value in every thread
        int t0;
        if constexpr (ROWU) {
            int s0;
            split_wave(blk * (kCopyThreads / 64) * U, a.wpr, a.shift, t0, s0);
        } else {
            int c0;
            split_chunk((int64_t)blk * (kCopyThreads * U), total, cpr, a.shift, t0, c0);
        }
        blk0 = t0 >> a.tile_shift;
        scan_table<KM>(a, blk0, kept_w, before_w, nullptr);
        kp = load_kept(kept_w, N);
    } else {
        kp = load_kept(a.kept_expert, N);
    }
    // table entries and limits of all choices, requested together (expert 0 stands in for a missing one)
    bool use[U][KM], live[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int tile = tok[u] >> a.tile_shift;
        int32_t first[KM], cap_e[KM];
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            use[u][j] = inside[u] && (KK > 0 || j < k) && (uint32_t)e[u][j] < (uint32_t)N;
            e[u][j] = use[u][j] ? e[u][j] : 0;
            cap_e[j] = cap[e[u][j]];
            if constexpr (TABLE) {
                first[j] = before_w[j][e[u][j]];
                for (int b = blk0; b < tile; ++b)   // tiles that begin inside this workgroup's tokens
                    first[j] += tile_table[(size_t)e[u][j] * a.pitch + (size_t)(KK > 0 || j < k ? j : 0) * a.n_blocks + b];
            } else {
                first[j] = tile_table[(size_t)e[u][j] * a.pitch + (size_t)(KK > 0 || j < k ? j : 0) * a.n_blocks + tile];
            }
            if constexpr (ROWU) first[j] = __builtin_amdgcn_readfirstlane(first[j]);
        }
        live[u] = false;
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            pos[u][j] += first[j];
            const bool kept = pos[u][j] < pair_limit(cap_e[j], a.cap != nullptr, a.pad_C);
            use[u][j] = use[u][j] & kept;   // no short cut: it would put a branch around the look-ups
            live[u] |= use[u][j];
        }
    }
    if constexpr (!TABLE) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (ROWU) {
                v[u] = RowBuffer(x + (size_t)tok[u] * cpr, cpr, live[u]).load(col[u]);
            } else {
                v[u] = vec16{0u, 0u, 0u, 0u};
                if (live[u]) v[u] = __builtin_nontemporal_load(x + (size_t)tok[u] * cpr + col[u]);
            }
        }
    }
    // every lane is here: the scan and, without ROWU, the lane exchange of offset_of need them all
    const WaveOffsets wo = wave_offsets(kp);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int j = 0; j < KM; ++j) {
            const int32_t off = a.pad_C > 0 ? e[u][j] * a.pad_C : offset_of<ROWU>(wo, e[u][j]);
            const int32_t sl = use[u][j] ? off + pos[u][j] : -1;
            if (inside[u] && (KK > 0 || j < k) && seg[u] == 0 && (!ROWU || lane == 0)) slot[(int64_t)tok[u] * k + j] = sl;
            if constexpr (ROWU) {
                RowBuffer(send + (size_t)(use[u][j] ? sl : 0) * cpr, cpr, use[u][j]).template store<ST>(col[u], v[u]);
            } else if (use[u][j]) {
                store_chunk<ST>(send + (size_t)sl * cpr + col[u], v[u]);
            }
        }
    }
}

constexpr int copy_units(int k) { return k == 1 ? 2 : 1; }   // chunks per thread

// By wavefront or flat?  Flat with a poor last wavefront: 65536 rows of 2064 bytes, two choices 107.8 us by wavefront,
// 100.7 flat, 1040 bytes 53.4 and 51.5, one choice 31.9 and 28.6, whole calls on 8000 x 1040
// with two 14.9 and 13.4, on 8000 x 1184 with one 11.3 and 10.4; from 12 lanes on, or 4 behind two full wavefronts, the
// other way round (2288 bytes 47.6 and 49.2, 3184 bytes 78.7 and 85.3, calls on 30000 x 2176 43.5 and 45.5).  And flat with more than four choices, for
// which a wavefront keeps eight of everything, if a tenth of its lanes would idle and rows are no whole lines: 16500 x
// 2064, eight choices 105.6 and 96.7, 11520 x 6368 166.9 and 161.7; but 9000 x 4000, six choices (2 % idle) 2.9 us less
// by wavefront, and 1536 bytes (whole lines, 25 % idle) 5 us less behind the gate, 5 more on its own.
static bool scatter_by_wave(int64_t S, int cpr, int k) {
    if (!rows_by_wave(cpr)) return false;
    if (poor_last_wave(S, cpr, row_waves(cpr) == 2 ? 12 : 4)) return false;
    const int lanes = row_waves(cpr) * 64;
    return k <= 4 || cpr % 8 == 0 || (lanes - cpr) * 10 <= lanes || S * row_waves(cpr) < 8192;
}

// How `rows` rows of send are written.  What decides is whether the last-level cache (256 MB) keeps them for whoever reads
// them next, and who merges the lines that a row shares with its neighbours.  Us of gate_dispatch and combine, N = 32,
// with ordinary / streaming / through stores:
//  - rows of whole lines go straight through L2 as long as they fit the last-level cache (30720 x 2 KiB, two choices 44.5 /
//    46.4 / 43.7; 14720 x 8 KiB, two 133.9 / 140.7 / 134.0; 17280 x 8 KiB, two 181 / 174 / 181; 34560 x 8 KiB, one 238 /
//    252 / 235).  Small buffers that nothing but the combine of an identity layer reads are
//    partly in L2 then (6144 x 1 KiB, two 18.2 / 20.0 / 18.9; dispatch alone 20.9 and 19.6 with through stores), short rows
//    of many choices gain on their own too (8192 x 512 bytes, eight 27.8 and 28.6);
//  - rows that are no whole lines, by wavefront: through (9830 x 4000, two 45.8 / 46.1 / 44.9; 47185 x 2000, two 134.5 /
//    137.6 / 132.2), with many choices from L2, which merges their lines (11320 x 6368, eight 273 / 287 / 286);
//    rows of half lines stream (39321 x 1600, two 93 / 88 / 92, 9611 x 3008, four 70 / 67 / 69);
//  - flat ones from L2 (57974 x 1040, four 111 / 136 / 121; 115651 x 272, two 61 / 65 / 65), one choice streaming beyond
//    96 MiB;
//  - the fixed-size layout streams beyond 96 MiB: its padding takes the place of rows (14117 x 7328, two, 237 MiB 131
//    streaming, 149 through; 56000 x 1 KiB, three, 205 MiB 99 and 101).
static int scatter_store(int64_t rows, int cpr, int k, bool by_wave, bool behind_gate, bool padded) {
    const int64_t mib = rows * cpr * 16 >> 20;
    if (padded && mib > 96) return kStoreStream;
    if (cpr % 8 == 0) {
        const int from = behind_gate && by_wave ? 8 : 0;
        const int to = behind_gate ? (k <= 2 ? 16 : 24) : !by_wave && k > 4 ? 32 : 0;
        if (mib >= from && mib < to) return kStoreBack;
        return mib <= (k == 1 ? 360 : 240) ? kStoreThrough : kStoreStream;
    }
    if (!by_wave) return mib <= (k == 1 ? 96 : k == 2 ? 240 : 640) ? kStoreBack : kStoreStream;
    if (mib <= 24) return kStoreThrough;
    if (k <= 4 && cpr % 4 == 0) return kStoreStream;
    if (k <= 4 && mib <= 240) return kStoreThrough;
    return k > 2 && mib <= 640 ? kStoreBack : kStoreStream;
}

// Workgroups that move rows.
static int64_t copy_workgroups(int64_t S, int cpr, int k) {
    const int U = copy_units(k);
    return scatter_by_wave(S, cpr, k) ? ceil_div(S * (int64_t)row_waves(cpr), kCopyThreads / 64 * U)
                             : ceil_div(S * (int64_t)cpr, kCopyThreads * U);
}

// Fills in the launch geometry.
static void plan_copy(RouteArgs& a) {
    a.wpr = row_waves(a.cpr);
    a.shift = pow2_shift(scatter_by_wave(a.S, a.cpr, a.k) ? a.wpr : a.cpr);
    a.copy_blocks = (int)copy_workgroups(a.S, a.cpr, a.k);
    // zeros of a large buffer would take the place of its rows in the last-level cache: 53902 x 1536 bytes, half of them
    // padding 86 us, streamed 78; 8192 x 8 KiB 66 and 61; but 6144 x 2 KiB (48 MiB) 28.7 and 29.2
    a.fill_streams = (int64_t)a.N * a.pad_C * a.cpr * 16 > (int64_t)64 << 20;
    // about 4096 workgroups clear rows, at most one per 4 KiB of an expert's rows
    a.fill_parts = a.pad_C == 0 ? 0 : (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(4096, a.N),
                                                                     ceil_div((int64_t)a.pad_C * a.cpr, kCopyThreads)));
}

template <int KK>
static void launch_route_copy(const RouteArgs& a, bool table, hipStream_t st) {
    constexpr int U = copy_units(KK);
    const dim3 grid = grid_of(1 + (int64_t)a.copy_blocks + (int64_t)a.N * a.fill_parts, kCopyThreads), block(kCopyThreads);
    const int64_t rows = a.pad_C > 0 ? (int64_t)a.N * a.pad_C : a.S * a.k;
    const int32_t* caps = a.cap != nullptr ? a.cap : a.table;   // N entries at least
#define TAMOE_ROUTE_COPY(RU, ST)                                                         \
    do {                                                                                 \
        if (table)                                                                       \
            route_copy_kernel<KK, U, RU, ST, true><<<grid, block, 0, st>>>(              \
                a.x, a.topk_idx, a.local_pos, a.table, caps, a.slot, a.send, a);        \
        else                                                                             \
            route_copy_kernel<KK, U, RU, ST, false><<<grid, block, 0, st>>>(             \
                a.x, a.topk_idx, a.local_pos, a.table, caps, a.slot, a.send, a);        \
    } while (0)
    const bool rowu = scatter_by_wave(a.S, a.cpr, a.k);
    const int policy = scatter_store(rows, a.cpr, a.k, rowu, a.m_part != nullptr, a.pad_C > 0);
#define TAMOE_ROUTE_COPY_ST(ST)                                                          \
    do {                                                                                 \
        if (rowu) TAMOE_ROUTE_COPY(true, ST); else TAMOE_ROUTE_COPY(false, ST);          \
    } while (0)
    if (policy == kStoreStream) TAMOE_ROUTE_COPY_ST(kStoreStream);
    else if (policy == kStoreThrough) TAMOE_ROUTE_COPY_ST(kStoreThrough);
    else TAMOE_ROUTE_COPY_ST(kStoreBack);
#undef TAMOE_ROUTE_COPY_ST
#undef TAMOE_ROUTE_COPY
}

// Stages 2 and 3, for table and positions as `run` describes them.
static int run_copy(const char* fn, const GateRun& run, RouteArgs a, const char* label, hipStream_t st) {
    int rc;
    a.local_pos = run.stats.local_pos;
    a.table = run.stats.tile_pairs;
    a.n_blocks = run.stats.n_blocks;
    a.pitch = run.stats.pitch;
    a.tile_shift = pow2_shift(run.tile_tokens);
    plan_copy(a);
    const int64_t blocks = (int64_t)a.copy_blocks + (int64_t)a.N * a.fill_parts;
    const bool table = a.S == 0 || (blocks <= kTableBlocks && blocks * a.N * a.k * a.n_blocks <= kTableReads);
    if (!table) {
        TraceScope tr("route_expert_kernel", st);
        route_expert_kernel<<<dim3(a.N), dim3(kExpertThreads), 0, st>>>(a.m_part, run.stats.tile_pairs, a.n_blocks,
                                                                        a.k * a.n_blocks, a.pitch, a.S, a.cap, a.pad_C,
                                                                        a.m, a.c_expert, a.kept_expert);
        if ((rc = check_launch(fn, "route_expert_kernel")) != TAMOE_OK) return rc;
    }
    {
        TraceScope tr(label, st);
        if (a.k == 1)
            launch_route_copy<1>(a, table, st);
        else if (a.k == 2)
            launch_route_copy<2>(a, table, st);
        else if (a.k == 3)
            launch_route_copy<3>(a, table, st);
        else if (a.k == 4)
            launch_route_copy<4>(a, table, st);
        else
            launch_route_copy<0>(a, table, st);
    }
    return check_launch(fn, "route_copy_kernel");
}

int run_dispatch(const char* fn, const void* x, const int32_t* topk_idx, const int32_t* cap, int64_t S, int cpr, int N,
                 int P, int k, int pad_C, void* send, int32_t* slot, int32_t* kept_expert,
                 int32_t* expert_offset, int32_t* send_count_dev, void* ws, const Workspace& lay, hipStream_t st) {
    int rc;
    // a few more workgroups are added
    if (S > 0 && std::max(ceil_div(S * (int64_t)cpr, kCopyThreads), copy_workgroups(S, cpr, k)) >= 0x7fff0000)
        return fail(TAMOE_UNSUPPORTED, "%s: x is too large for one launch", fn);
    const int tok = rank_tokens(S, N, k);
    const int64_t blocks = ceil_div(S, tok);
    GateRun run{};
    run.stats = stats_in(ws, lay, k, blocks);
    run.tile_tokens = tok;
    if (blocks > 0) {
        TraceScope tr("route_rank_kernel", st);
        const dim3 grid = grid_of(blocks, 512), block(512);
#define TAMOE_RANK(NB)                                                                                  \
    do {                                                                                                \
        if (tok == 128) route_rank_kernel<NB, 128><<<grid, block, 0, st>>>(topk_idx, S, N, k, run.stats); \
        else if (tok == 256) route_rank_kernel<NB, 256><<<grid, block, 0, st>>>(topk_idx, S, N, k, run.stats); \
        else route_rank_kernel<NB, 512><<<grid, block, 0, st>>>(topk_idx, S, N, k, run.stats);           \
    } while (0)
        if (N <= 32) TAMOE_RANK(1);
        else if (N <= 64) TAMOE_RANK(2);
        else TAMOE_RANK(4);
#undef TAMOE_RANK
        if ((rc = check_launch(fn, "route_rank_kernel")) != TAMOE_OK) return rc;
    }
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
    if ((rc = run_gate_stage(fn, x, w, dtype, S, d, N, k, logits, topk_idx, topk_w, ws, lay, st, &run)) != TAMOE_OK)
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
