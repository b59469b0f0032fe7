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
//      How rows are stored depends on what the caches can do for them (scatter_store).
#include <algorithm>
#include <type_traits>

#include "gate_tile.h"
#include "internal.h"
#include "scan128.h"

namespace tamoe {

constexpr int kCopyThreads = 256;

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
    const int32_t* table;       // prefix of the pairs per (expert; choice, tile), left by route_expert_kernel
    const uint16_t* counts;     // or the pairs themselves: rows of `stride` per tile, (e, j) at j*N + e
    const int32_t* cap;         // may be NULL when pad_C > 0
    const float* m_part;        // [N][n_blocks] sums of gate probabilities, NULL for a given routing
    int32_t* slot;
    vec16* send;
    int64_t S;
    int N, P, k;
    int cpr, wpr, shift;        // chunks per row, wavefronts per row, log2 of wpr (flat: of cpr) or -1
    int n_blocks, pitch, tile_shift;
    int stride, units;          // small tables: count_stride, chunks of 64 lanes per wavefront of the scatter
    int threads;                // of the scatter
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

// ---- small tables -------------------------------------------------------------------------------------
// Every workgroup of the scatter sums the pair counts itself: a row per token tile, read 16 bytes per lane, added
// up two to a register, first over a lane's rows, then over the lanes and wavefronts with the same
// columns.  Latency: one memory round trip (1.5 us after the 0.7 that a workgroup needs to its first request), beside which
// the rows are on their way too, then 0.9 us.  What was measured to count is the length of the code, which a wavefront
// runs once, from cold instruction caches: with bytes for counts (half the requests, three times the additions)
// small_forward took 17.8 us, with the steps of sum_columns under a condition each 15.9, now 14.8.
constexpr int kTableThreads = 512;   // or half as many (table_threads)
constexpr int kTableBatch = 8;   // rows per lane, requested together (one in the smallest tables)
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

template <int TH>
struct TableLds {
    uint32_t part[TH / 64][64][8];                           // by wavefront and column: all tiles, tiles before blk0
    int32_t before[TAMOE_MAX_K * TAMOE_MAX_EXPERTS];         // pairs of e that precede choice j of tile blk0, at j*N + e
    int32_t total[TAMOE_MAX_K * TAMOE_MAX_EXPERTS];          // pairs of (e, j), where a thread has one choice
    int32_t pairs[TAMOE_MAX_EXPERTS], kept[TAMOE_MAX_EXPERTS];
};

// Sums over the lanes of a wavefront that are a multiple of C (a power of two) apart, of each of M values 4 bytes wide.
template <class T, int M>
__device__ __forceinline__ void sum_columns(T (&v)[M], int C) {
    const auto u = [](T t) { return __builtin_bit_cast(uint32_t, t); };
    const auto h = [](uint32_t t) { return __builtin_bit_cast(T, t); };
    if (C <= 32) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const auto s = __builtin_amdgcn_permlane32_swap(u(v[i]), u(v[i]), false, false);
            v[i] = h(s[0]) + h(s[1]);
        }
    }
    if (C <= 16) {
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const auto s = __builtin_amdgcn_permlane16_swap(u(v[i]), u(v[i]), false, false);
            v[i] = h(s[0]) + h(s[1]);
        }
    }
    if (C <= 8) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += h((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(v[i]), 0x128, 0xf, 0xf, true));   // row_ror:8
    }
    if (C <= 4) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += h((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(v[i]), 0x124, 0xf, 0xf, true));   // row_ror:4
    }
    if (C <= 2) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += h((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(v[i]), 0x122, 0xf, 0xf, true));   // row_ror:2
    }
    if (C <= 1) {
#pragma unroll
        for (int i = 0; i < M; ++i) v[i] += h((uint32_t)__builtin_amdgcn_update_dpp(0, (int)u(v[i]), 0x121, 0xf, 0xf, true));   // row_ror:1
    }
}

// Fills in t; also calls while_waiting(), between the requests for the counts and their use.  Every thread calls; ends
// with a barrier.
template <int TH, int KK, int B, class Body>
__device__ __forceinline__ void scan_counts(const RouteArgs& a, int blk0, TableLds<TH>& t, Body while_waiting) {
    constexpr int kWaves = TH / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int C = a.stride >> 3, shift = 31 - __builtin_clz(C);
    const int col = tid & (C - 1), r0 = tid >> shift, R = TH >> shift;
    const __amdgpu_buffer_rsrc_t rows =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.counts), 0, a.n_blocks * a.stride * 2, 0x00020000);
    const int32_t cap_e = WordBuffer(a.cap, a.cap != nullptr ? a.N : 0).load<int32_t>(tid);
    vec16 v[B];
#pragma unroll
    for (int i = 0; i < B; ++i)   // rows past the end are zeros
        v[i] = __builtin_bit_cast(vec16, __builtin_amdgcn_raw_buffer_load_b128(rows, (r0 + i * R) * a.stride * 2 + col * 16, 0, 0));
    __builtin_amdgcn_sched_barrier(0);
    while_waiting();
    __builtin_amdgcn_sched_barrier(0);
    u16x2 sums[8] = {};   // all tiles, tiles before blk0
#pragma unroll
    for (int i = 0; i < B; ++i) {
        const uint32_t mask = r0 + i * R < blk0 ? 0xffffffffu : 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t w = v[i][q];
            sums[q] += __builtin_bit_cast(u16x2, w);
            sums[q + 4] += __builtin_bit_cast(u16x2, w & mask);
        }
    }
    sum_columns(sums, C);
    if (lane < C) {
        uint4* dst = reinterpret_cast<uint4*>(t.part[wave][lane]);
        auto bits = [](u16x2 x) { return __builtin_bit_cast(uint32_t, x); };
        dst[0] = make_uint4(bits(sums[0]), bits(sums[1]), bits(sums[2]), bits(sums[3]));
        dst[1] = make_uint4(bits(sums[4]), bits(sums[5]), bits(sums[6]), bits(sums[7]));
    }
    __syncthreads();
    const int half = C > 64 ? 1 : 0;   // 128 columns: the even wavefronts have the first 64 of them
    auto column = [&](int i, int32_t& all, int32_t& bef) {
        const int c = i >> 3, q = (i & 7) >> 1, sh = (i & 1) * 16;
        uint32_t n[kWaves], b[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t* at = t.part[(w << half & (kWaves - 1)) | c >> 6][c & 63];
            n[w] = w < kWaves >> half ? at[q] : 0u;
            b[w] = w < kWaves >> half ? at[q + 4] : 0u;
        }
        all = bef = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            all += n[w] >> sh & 0xffffu;
            bef += b[w] >> sh & 0xffffu;
        }
    };
    if constexpr (KK == 0) {   // a thread per choice too: one after the other they take 2 us (404 x 768 bytes, six)
        for (int i = tid; i < a.k * a.N; i += TH) column(i, t.total[i], t.before[i]);
        __syncthreads();
    }
    if (tid < a.N) {
        int32_t run = 0;
        if constexpr (KK > 0) {
#pragma unroll
            for (int j = 0; j < KK; ++j) {
                int32_t all, bef;
                column(j * a.N + tid, all, bef);
                t.before[j * a.N + tid] = run + bef;
                run += all;
            }
        } else {
            int32_t all[TAMOE_MAX_K], bef[TAMOE_MAX_K];
#pragma unroll
            for (int j = 0; j < TAMOE_MAX_K; ++j) {
                const int i = (j < a.k ? j : 0) * a.N + tid;
                all[j] = t.total[i];
                bef[j] = t.before[i];
            }
#pragma unroll
            for (int j = 0; j < TAMOE_MAX_K; ++j) {
                if (j >= a.k) break;
                t.before[j * a.N + tid] = run + bef[j];
                run += all[j];
            }
        }
        const int32_t lim = pair_limit(cap_e, a.cap != nullptr, a.pad_C);
        t.pairs[tid] = run;
        t.kept[tid] = run < lim ? run : lim;
    }
    __syncthreads();
}

// What describes the layer as a whole, by one workgroup that does nothing else
// (every thread calls): expert offsets (Section 4.3: what the size exchange carries), rows and pairs per
// destination device, the loss; with TABLE also what route_expert_kernel would have written.  N <= 128
// values: the first wavefront holds two experts per lane, scans and sums them with lane operations
// (fixed order), and looks up the per-device numbers in LDS.
template <int TH, bool TABLE, int KK, int B>
__device__ __forceinline__ void route_layer_outputs(const RouteArgs& a, TableLds<TH>* t) {
    constexpr int kWaves = TH / 64;
    __shared__ float4 sums[TABLE ? kWaves : 1][TAMOE_MAX_EXPERTS / 4];
    __shared__ int32_t off[TAMOE_MAX_EXPERTS + 1], pairs_off[TAMOE_MAX_EXPERTS + 1];
    const int tid = threadIdx.x;
    const int N = a.N;
    const int e0 = tid & 63, e1 = e0 + 64;
    // requested before anything is waited for
    const WordBuffer pen(a.penalty, a.penalty != nullptr ? N : 0);
    const float p0 = pen.load<float>(e0), p1 = pen.load<float>(e1);
    int32_t k0, k1, c0, c1;   // kept rows and pairs of the lane's experts, 0 beyond N
    float m0 = 0.f, m1 = 0.f;
    if constexpr (TABLE) {
        // sums of gate probabilities, four experts of a tile per lane
        const int P4 = sum_stride(N) / 4, R = TH / P4;
        const int r0 = tid / P4, q = tid & (P4 - 1);
        scan_counts<TH, KK, B>(a, 0, *t, [&] {
            if (a.m == nullptr) return;
            const __amdgpu_buffer_rsrc_t rows =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.m_part), 0, a.n_blocks * P4 * 16, 0x00020000);
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
            for (int r = 0; r < a.n_blocks; r += 8 * R) {
                float4 v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i)   // tiles past the end are zeros
                    v[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rows, ((r + r0 + i * R) * P4 + q) * 16, 0, 0));
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    acc[0] += v[i].x;
                    acc[1] += v[i].y;
                    acc[2] += v[i].z;
                    acc[3] += v[i].w;
                }
            }
            sum_columns(acc, P4);
            if ((tid & 63) < P4) sums[tid >> 6][q] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        });
        if (tid >= 64) return;
        k0 = e0 < N ? t->kept[e0] : 0;
        k1 = e1 < N ? t->kept[e1] : 0;
        c0 = e0 < N ? t->pairs[e0] : 0;
        c1 = e1 < N ? t->pairs[e1] : 0;
        if (a.m != nullptr) {
            const float* part = reinterpret_cast<const float*>(sums);
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                m0 += e0 < N ? part[w * TAMOE_MAX_EXPERTS + e0] : 0.f;
                m1 += e1 < N ? part[w * TAMOE_MAX_EXPERTS + e1] : 0.f;
            }
            m0 = a.S > 0 ? m0 / (float)a.S : 0.f;
            m1 = a.S > 0 ? m1 / (float)a.S : 0.f;
            if (e0 < N) a.m[e0] = m0;
            if (e1 < N) a.m[e1] = m1;
        }
        if (e0 < N) a.kept_expert[e0] = k0;
        if (e1 < N) a.kept_expert[e1] = k1;
        if (a.c_expert != nullptr) {
            if (e0 < N) a.c_expert[e0] = c0;
            if (e1 < N) a.c_expert[e1] = c1;
        }
    } else {
        if (tid >= 64) return;
        const WordBuffer kept(a.kept_expert, N), pairs(a.c_expert, a.c_expert != nullptr ? N : 0), mean(a.m, a.m != nullptr ? N : 0);
        k0 = kept.load<int32_t>(e0);
        k1 = kept.load<int32_t>(e1);
        c0 = pairs.load<int32_t>(e0);
        c1 = pairs.load<int32_t>(e1);
        m0 = mean.load<float>(e0);
        m1 = mean.load<float>(e1);
    }
    // one wavefront from here on, no barriers
    auto prefix = [&](int32_t v0, int32_t v1, int32_t* out) {   // out[N] is the total
        const int32_t i0 = wave_inclusive_scan(v0);
        const int32_t i1 = wave_inclusive_scan(v1) + __builtin_amdgcn_readlane(i0, 63);
        out[e0] = i0 - v0;
        out[e1] = i1 - v1;
        if (e1 == TAMOE_MAX_EXPERTS - 1) out[TAMOE_MAX_EXPERTS] = i1;
    };
    prefix(k0, k1, off);
    prefix(c0, c1, pairs_off);
    if (a.loss != nullptr) {
        const float t0 = m0 * (float)c0 * (a.penalty != nullptr ? p0 : 1.f);
        const float t1 = m1 * (float)c1 * (a.penalty != nullptr ? p1 : 1.f);
        const float term = wave_total((e0 < N ? t0 : 0.f) + (e1 < N ? t1 : 0.f));
        if (tid == 0) a.loss[0] = term * a.loss_scale;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int E = N / a.P;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = tid + 64 * h;
        if (a.expert_offset != nullptr && i < N) a.expert_offset[i] = off[i];
        if (i < a.P) {
            if (a.send_count_dev != nullptr) a.send_count_dev[i] = off[(i + 1) * E] - off[i * E];
            if (a.c_device != nullptr) a.c_device[i] = pairs_off[(i + 1) * E] - pairs_off[i * E];
        }
    }
    if (a.expert_offset != nullptr && tid == 0) a.expert_offset[N] = off[N];
}

// Clears rows e*C + kept[e] .. (e+1)*C - 1 of the fixed-size layout, share f of all (N * fill_parts shares).
template <int ST>
__device__ __forceinline__ void clear_unused(const RouteArgs& a, int f, const int32_t* kept, int threads) {
    const int e = f / a.fill_parts, part = f - e * a.fill_parts;
    const int32_t used = kept[e];
    const int64_t n = (int64_t)(a.pad_C - used) * a.cpr;               // chunks to clear, >= 0
    const int64_t per = (n + a.fill_parts - 1) / a.fill_parts;
    const int64_t i0 = (int64_t)part * per;
    const int64_t i1 = i0 + per < n ? i0 + per : n;
    vec16* base = a.send + ((int64_t)e * a.pad_C + used) * a.cpr;
    const vec16 zero = {0u, 0u, 0u, 0u};
    if (a.fill_streams) {
        for (int64_t i = i0 + threadIdx.x; i < i1; i += threads) store_chunk<kStoreStream>(base + i, zero);
    } else {
        for (int64_t i = i0 + threadIdx.x; i < i1; i += threads) store_chunk<ST>(base + i, zero);
    }
}

// The scatter with the slot assignment folded in, behind route_expert_kernel.  Workgroup 0 writes the layer's outputs
// and moves no rows: as part of a copying workgroup that tail would end after every other workgroup of a short
// launch.  Then copy_blocks workgroups move rows, and N * fill_parts clear the unused rows of the fixed-size
// layout.  ROWU: rows by whole wavefronts (scatter_by_wave), U segments each; otherwise U chunks per
// thread, flat.  ST: how rows are stored (scatter_store).
// (What the copying workgroups read comes as arguments of its own: only a pointer that is declared not to
// alias is read through the scalar unit.  cap is never NULL here: without capacities it is the table, whose
// entries are then not looked at, so that no branch stands between the look-ups.)
template <int KK, int U, bool ROWU, int ST, int LD>
__global__ __launch_bounds__(kCopyThreads) void route_copy_kernel(
    const vec16* __restrict__ x, const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ local_pos,
    const int32_t* __restrict__ tile_table, const int32_t* __restrict__ cap, int32_t* __restrict__ slot,
    vec16* __restrict__ send, const RouteArgs a) {
    const uint32_t wg = linear_block();
    if (wg == 0) {
        route_layer_outputs<kCopyThreads, false, KK, 1>(a, nullptr);
        return;
    }
    constexpr int KM = KK > 0 ? KK : TAMOE_MAX_K;
    const int N = a.N, cpr = a.cpr;
    const int lane = threadIdx.x & 63;

    if (wg > (uint32_t)a.copy_blocks) {
        const int f = (int)(wg - 1 - (uint32_t)a.copy_blocks);
        if (f < N * a.fill_parts) clear_unused<ST>(a, f, a.kept_expert, kCopyThreads);   // else past the last workgroup (grid_of)
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
    const KeptPair kp = load_kept(a.kept_expert, N);
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
            first[j] = tile_table[(size_t)e[u][j] * a.pitch + (size_t)(KK > 0 || j < k ? j : 0) * a.n_blocks + tile];
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
    // Rows of dropped tokens are left out: a launch of this size is bound by bytes (65536 x 8 KiB: 258 us, requested at
    // once 262; half the tokens of 16384 x 4 KiB dropped: 15.9 us, at once 17.2).
    vec16 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (ROWU) {
            v[u] = RowBuffer(x + (size_t)tok[u] * cpr, cpr, live[u]).template load<LD>(col[u]);
        } else {
            v[u] = vec16{0u, 0u, 0u, 0u};
            if (live[u]) v[u] = load_chunk<LD>(x + (size_t)tok[u] * cpr + col[u]);
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

// The same for a small table of pair counts (table_units), which every workgroup sums up by itself: one launch less, 2.5 to
// 4.7 us (gate_dispatch and combine, us before and now: 4096 x 1 KiB, 16 experts 16.7, 14.8; 16384 x 2 KiB, 64 experts 46.0,
// 42.8; fp32 4096 x 4 KiB 34.8, 31.7).  A wavefront has U units (64 chunks of one row, ROWU, or 64 chunks
// anywhere), whose rows it requests, kept or not, behind the counts and before it waits for them.  At most 128
// registers: two workgroups share a compute unit.
// ROWU: a lane has one of the wavefront's pairs (unit, choice) and works out its slot; the stores read the slots from
// the lanes.
template <int TH, int KK, int U, bool ROWU, int ST, int LD, int B>
__global__ __launch_bounds__(TH, 4) void route_table_kernel(
    const vec16* __restrict__ x, const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ local_pos,
    const uint16_t* __restrict__ counts, int32_t* __restrict__ slot, vec16* __restrict__ send, const RouteArgs a) {
    constexpr int KM = KK > 0 ? KK : TAMOE_MAX_K;
    __shared__ TableLds<TH> t;
    const int wg = (int)blockIdx.x;   // one generation
    if (wg == 0) {
        route_layer_outputs<TH, true, KK, B>(a, &t);
        return;
    }
    const int N = a.N, cpr = a.cpr, k = KK > 0 ? KK : a.k;
    if (wg > a.copy_blocks) {
        scan_counts<TH, KK, B>(a, 0, t, [] {});
        clear_unused<ST>(a, wg - 1 - a.copy_blocks, t.kept, TH);
        return;
    }
    const int lane = threadIdx.x & 63;
    const uint32_t first_unit = (uint32_t)(wg - 1) * (TH / 64) * U;
    const uint32_t unit0 = first_unit + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * U;
    const int64_t total = a.S * cpr;
    // token tile of the workgroup's first token
    int t0, c0;
    if constexpr (ROWU) split_wave(first_unit, a.wpr, a.shift, t0, c0);
    else split_chunk((int64_t)first_unit * 64, total, cpr, a.shift, t0, c0);
    const int blk0 = t0 >> a.tile_shift;
    // Slot of choice j of token tok, from its expert and position; -1: none, or dropped.  All lanes call.
    auto slot_of = [&](const WaveOffsets& wo, int32_t e, int32_t pos, int tok, int j, bool there) {
        const bool ok = there && (uint32_t)e < (uint32_t)N;
        e = ok ? e : 0;
        const int at = j * N + e, tile = tok >> a.tile_shift;
        pos += t.before[at];
        for (int b = blk0; b < tile; ++b) pos += counts[(size_t)b * a.stride + at];   // tiles that begin inside this workgroup
        const int32_t off = a.pad_C > 0 ? e * a.pad_C : offset_of<false>(wo, e);
        return ok && pos < t.kept[e] ? off + pos : -1;
    };
    vec16 v[U];
    if constexpr (ROWU) {
        static_assert(U * KM <= 64, "a lane per pair of the wavefront");
        const int pu = lane / KM, pj = lane % KM;
        int ptok, pseg;
        split_wave(unit0 + (pu < U ? pu : 0), a.wpr, a.shift, ptok, pseg);
        const bool there = pu < U && pj < k && ptok < a.S;
        const int64_t p = there ? (int64_t)ptok * k + pj : 0;
        const int32_t e = topk_idx[p], pos = local_pos[p];
        int tok[U], seg[U];
        split_wave(unit0, a.wpr, a.shift, tok[0], seg[0]);
#pragma unroll
        for (int u = 1; u < U; ++u) {
            const bool next = seg[u - 1] + 1 == a.wpr;
            tok[u] = tok[u - 1] + next;
            seg[u] = next ? 0 : seg[u - 1] + 1;
        }
        scan_counts<TH, KK, B>(a, blk0, t, [&] {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = tok[u] < a.S;
                v[u] = RowBuffer(x + (size_t)(in ? tok[u] : 0) * cpr, cpr, in).template load<LD>(seg[u] * 64 + lane);
            }
        });
        const WaveOffsets wo = wave_offsets(load_kept(t.kept, N));
        const int32_t sl = slot_of(wo, e, pos, there ? ptok : t0, pj < k ? pj : 0, there);
        if (there && pseg == 0) slot[p] = sl;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                const int32_t to = __builtin_amdgcn_readlane(sl, u * KM + j);   // -1 where there is no such choice
                RowBuffer(send + (size_t)(to >= 0 ? to : 0) * cpr, cpr, to >= 0).template store<ST>(seg[u] * 64 + lane, v[u]);
            }
    } else {
        int tok[U], col[U];
        bool inside[U];
        int32_t e[U][KM], pos[U][KM];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = (int64_t)(unit0 + u) * 64 + lane;
            inside[u] = c < total;
            split_chunk(inside[u] ? c : total - 1, total, cpr, a.shift, tok[u], col[u]);
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                const int64_t p = (int64_t)tok[u] * k + (KK > 0 || j < k ? j : k - 1);
                e[u][j] = topk_idx[p];
                pos[u][j] = local_pos[p];
            }
        }
        scan_counts<TH, KK, B>(a, blk0, t, [&] {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = load_chunk<LD>(x + (size_t)tok[u] * cpr + col[u]);
        });
        const WaveOffsets wo = wave_offsets(load_kept(t.kept, N));
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < KM; ++j) {
                const bool there = inside[u] && (KK > 0 || j < k);
                const int32_t sl = slot_of(wo, e[u][j], pos[u][j], tok[u], KK > 0 || j < k ? j : 0, there);
                if (there && col[u] == 0) slot[(int64_t)tok[u] * k + j] = sl;
                if (sl >= 0) store_chunk<ST>(send + (size_t)sl * cpr + col[u], v[u]);
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

// Units of 64 chunks: of one row each, or anywhere (flat).
static int64_t move_units(int64_t S, int cpr, int k) {
    return scatter_by_wave(S, cpr, k) ? S * row_waves(cpr) : ceil_div(S * (int64_t)cpr, 64);
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

// How x is loaded: by what it and the rows take, the unused ones of the fixed-size layout too.
static bool keeps_x(const RouteArgs& a) {
    return scatter_load(a.S, a.pad_C > 0 ? (int64_t)a.N * a.pad_C : rows_sent(a), a.cpr, a.m_part != nullptr) == kLoadKeep;
}

// Fills in the launch geometry.
static void plan_copy(RouteArgs& a) {
    const bool by_wave = scatter_by_wave(a.S, a.cpr, a.k);
    a.wpr = row_waves(a.cpr);
    a.shift = pow2_shift(by_wave ? a.wpr : a.cpr);
    a.copy_blocks = a.units == 0 ? (int)copy_workgroups(a.S, a.cpr, a.k)
                                 : (int)ceil_div(move_units(a.S, a.cpr, a.k), a.threads / 64 * a.units);
    a.fill_streams = fill_streams((int64_t)a.N * a.pad_C, rows_sent(a), a.cpr);
    // about 4096 workgroups clear rows (512 of the larger ones that sum the table), at most one per 16 bytes per thread
    const int wgs = a.units == 0 ? 4096 : 512;
    a.fill_parts = a.pad_C == 0 ? 0 : (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(wgs, a.N),
                                                                     ceil_div((int64_t)a.pad_C * a.cpr, a.threads)));
}

template <int KK>
static void launch_route_copy(const RouteArgs& a, hipStream_t st) {
    constexpr int U = copy_units(KK);
    const dim3 grid = grid_of(1 + (int64_t)a.copy_blocks + (int64_t)a.N * a.fill_parts, kCopyThreads), block(kCopyThreads);
    const int32_t* caps = a.cap != nullptr ? a.cap : a.table;   // N entries at least
    const bool rowu = scatter_by_wave(a.S, a.cpr, a.k), behind_gate = a.m_part != nullptr;
    const StorePolicy policy = scatter_store(row_lines(a.send, a.cpr), rows_sent(a), a.cpr, a.k, rowu, behind_gate, a.pad_C > 0);
    const bool keep = keeps_x(a);
#define TAMOE_ROUTE_COPY(RU, ST, LD)                                                          \
    route_copy_kernel<KK, U, RU, ST, LD><<<grid, block, 0, st>>>(a.x, a.topk_idx, a.local_pos, a.table, caps, a.slot, a.send, a)
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

// Units (64 chunks) per wavefront with which the scatter sums the table itself (route_table_kernel); 0: with
// route_expert_kernel and route_copy_kernel.
// The table has to be one batch of scan_counts: a second one is a second memory round trip (5003 x 2000 bytes, 157 tiles
// of 192 counts: 65.9 us for a training pass, 65.7 with the launch).  Units: as many as leave a workgroup per compute
// unit, since each one sums the table (small_forward, 4096 units: with two 14.8, with one 17.5; gpt_moe_forward, 32768: with
// eight 43.0, with four 45.3; 6681 x 3456 bytes, eight choices, 26724: with eight 71.9, with two 75.0, with the launch 75.2); beyond 65536 of
// them (64 MiB of x) the launch that is saved counts for little (31106 x 2304, three, 93318: 102.4 with it, 99.9 without), and for a
// routing that is given, behind which x does not come from the last-level cache, beyond 32768 (skewed_separate, 65536: 53.7 with the
// launch, 54.7 without; fused, 16384 x 4 KiB, one choice 59.7 and 56.7).  Flat rows have the work of a slot in every lane, and
// at most two units (60623 x 256, one choice, 15156: 23.6 with the launch, 24.6 with two, 28.7 with one).
static int table_units(int64_t S, int cpr, int N, int k, int tile_tokens, bool behind_gate) {
    // 16 bits hold the sums of a wavefront's share of the tiles, whatever the routing: with R = 512 / C rows of C pieces requested at a
    // time it has ceil(tiles / R) times max(1, 64 / C) tiles, (S + tile) / 8 + 64 * tile / C tokens at most, which are 57 832 for
    // S = 200 000, C = 1 and tiles of 512, and a token counts once per expert and choice
    if (S > 200000 || ceil_div(S, tile_tokens) * (count_stride(N, k) / 8) > kTableBatch * kTableThreads) return 0;
    const bool by_wave = scatter_by_wave(S, cpr, k);
    const int64_t units = move_units(S, cpr, k);
    if (units > (!by_wave ? 8192 : behind_gate ? 65536 : 32768)) return 0;
    int U = 1;
    while (U < (by_wave ? 8 : 2) && units >= kTableThreads / 64 * U * 2 * 256) U *= 2;
    return U;
}

// Threads of a workgroup that sums the table: half as many where workgroups of 512 would be fewer than the compute units, as
// long as the table is one batch of theirs (forward calls, us with 512 and 256: 435 x 400 bytes, four choices 15.0, 14.4; 704 x 128,
// four 13.5, 12.7; 1024 x 1 KiB, 72 experts 14.9, 14.5; fixed-size layout, 704 x 352, eight 17.1, 15.7; 128 threads are no better: 1958 x
// 1792 13.8, 256 13.1).
static int table_threads(int64_t S, int cpr, int k, int64_t pieces) {
    constexpr int kHalf = kTableThreads / 2;
    // a fourth of the tiles per wavefront: fits 16 bits, as in table_units
    return move_units(S, cpr, k) < kTableThreads / 64 * 256 && S <= 100000 && pieces <= kTableBatch * kHalf ? kHalf : kTableThreads;
}

// Only the policies that scatter_store can answer at these sizes are there: a unit is 1 KiB of x at most, and U units per wavefront
// go with fewer than 4096 * U of them (65536 for U = 8; 2048 with the smaller workgroups).
template <int TH, int KK, int U, bool ROWU>
static void launch_route_table_u(const RouteArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)(1 + a.copy_blocks + a.N * a.fill_parts)), block(TH);
    const StorePolicy policy = scatter_store(row_lines(a.send, a.cpr), rows_sent(a), a.cpr, a.k, ROWU, a.m_part != nullptr, a.pad_C > 0);
    constexpr int kX = (U == 8 ? 64 : 4 * U) / (TH == kTableThreads ? 1 : 2);   // MiB of x
    constexpr int kMiB = kX * (KK > 0 ? KK : TAMOE_MAX_K);                       // of rows
    constexpr bool kKeepsAll = U == 1;   // but for much padding, where 4 MiB of x do not matter
    static_assert(!kKeepsAll || kX + kMiB <= kKeepGiven, "nothing of its size streams");
    const bool keep = kKeepsAll || keeps_x(a);
    // the smallest tables in a kernel that is shorter by seven requests and their sums
    const bool one = U == 1 && (int64_t)a.n_blocks * (a.stride / 8) <= TH;
    const auto launch_ld = [&](auto st_c, auto ld_c) {
        constexpr int ST = decltype(st_c)::value, LD = decltype(ld_c)::value;
        if (one)
            route_table_kernel<TH, KK, U, ROWU, ST, LD, U == 1 ? 1 : kTableBatch>
                <<<grid, block, 0, st>>>(a.x, a.topk_idx, a.local_pos, a.counts, a.slot, a.send, a);
        else
            route_table_kernel<TH, KK, U, ROWU, ST, LD, kTableBatch>
                <<<grid, block, 0, st>>>(a.x, a.topk_idx, a.local_pos, a.counts, a.slot, a.send, a);
    };
    const auto launch = [&](auto st_c) {
        constexpr bool kOut = decltype(st_c)::value == kStoreOut;   // more than scatter_load keeps
        if constexpr (kOut || !kKeepsAll)
            if (kOut || !keep) return launch_ld(st_c, std::integral_constant<int, kLoadStream>{});
        if constexpr (!kOut) launch_ld(st_c, std::integral_constant<int, kLoadKeep>{});
    };
    if constexpr (kMiB > 16)   // half lines
        if (policy == kStoreStream) return launch(std::integral_constant<int, kStoreStream>{});
    if constexpr (!ROWU || (KK == 0 && kMiB > 24) || (KK == 4 && kMiB > 240))
        if (policy == kStoreBack) return launch(std::integral_constant<int, kStoreBack>{});
    if constexpr (ROWU && kMiB > 128)
        if (policy == kStoreOut) return launch(std::integral_constant<int, kStoreOut>{});
    launch(std::integral_constant<int, kStoreThrough>{});
}
template <int KK>
static void launch_route_table(const RouteArgs& a, hipStream_t st) {
    constexpr int TH = kTableThreads;
    if (!scatter_by_wave(a.S, a.cpr, a.k)) {
        if (a.threads != TH) launch_route_table_u<TH / 2, KK, 1, false>(a, st);
        else if (a.units == 1) launch_route_table_u<TH, KK, 1, false>(a, st);
        else launch_route_table_u<TH, KK, 2, false>(a, st);
    } else {
        if (a.threads != TH) launch_route_table_u<TH / 2, KK, 1, true>(a, st);
        else if (a.units == 1) launch_route_table_u<TH, KK, 1, true>(a, st);
        else if (a.units == 2) launch_route_table_u<TH, KK, 2, true>(a, st);
        else if (a.units == 4) launch_route_table_u<TH, KK, 4, true>(a, st);
        else launch_route_table_u<TH, KK, 8, true>(a, st);
    }
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
        route_expert_kernel<<<dim3(a.N), dim3(kExpertThreads), 0, st>>>(a.m_part, run.stats.tile_pairs, a.n_blocks,
                                                                        a.k * a.n_blocks, a.pitch, a.S, a.cap, a.pad_C,
                                                                        a.m, a.c_expert, a.kept_expert);
        if ((rc = check_launch(fn, "route_expert_kernel")) != TAMOE_OK) return rc;
    }
    {
        TraceScope tr(label, st);
#define TAMOE_ROUTE(KK)                                                               \
    do {                                                                              \
        if (table) launch_route_table<KK>(a, st); else launch_route_copy<KK>(a, st);  \
    } while (0)
        if (a.k == 1) TAMOE_ROUTE(1);
        else if (a.k == 2) TAMOE_ROUTE(2);
        else if (a.k == 3) TAMOE_ROUTE(3);
        else if (a.k == 4) TAMOE_ROUTE(4);
        else TAMOE_ROUTE(0);
#undef TAMOE_ROUTE
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
