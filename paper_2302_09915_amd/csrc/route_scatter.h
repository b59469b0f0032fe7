// Kernels of the scatter, shared by the translation units that instantiate them (route.hip, route_given.hip).
#pragma once

#include <type_traits>

#include "gate_tile.h"
#include "internal.h"
#include "scan128.h"

namespace tamoe {

constexpr int kCopyThreads = 256;

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
    uint32_t k_magic;           // ceil(2^32 / k), k > 1
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
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

template <int TH>
struct TableLds {
    uint32_t part[TH / 64][64][8];                           // by wavefront and column: all tiles, tiles before blk0
    int32_t before[TAMOE_MAX_K * TAMOE_MAX_EXPERTS];         // pairs of e that precede choice j of tile blk0, at j*N + e
    int32_t total[TAMOE_MAX_K * TAMOE_MAX_EXPERTS];          // pairs of (e, j), where a thread has one choice
    int32_t pairs[TAMOE_MAX_EXPERTS], kept[TAMOE_MAX_EXPERTS];
    unsigned char rank[kGivenTokens * TAMOE_MAX_K];          // of a given routing: see count_given
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

// The same from a routing that is given, for the tokens from t0 on (B == 0): every workgroup counts all pairs itself, in the two
// halves of a word all of them and those of tokens before t0 (both fit: kGivenPairs is below 2^16), and ranks those of its own
// tokens t0 .. t1 - 1 (64 at a time, one ballot per bit of the expert, as finish_block does).  An index outside [0, N) is no pair.
// With one copy of the counts, pairs that meet in an expert were up to 64 turns of an LDS addition (16384 x 128 bytes, most of
// them to few experts: 24.5 us for the calls that take 12.0 now).
template <int TH, int KK, class Body>
__device__ __forceinline__ void count_given(const RouteArgs& a, int t0, int t1, TableLds<TH>& t, Body while_waiting) {
    constexpr int kWaves = TH / 64, kTurns = (TAMOE_MAX_K + kWaves - 1) / kWaves, kGroups = kGivenTokens / 64;
    const int k = KK > 0 ? KK : a.k, n = (int)a.S * k, N = a.N;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WordBuffer idx(a.topk_idx, n);
    const int32_t cap_e = WordBuffer(a.cap, a.cap != nullptr ? N : 0).load<int32_t>(tid);
    int32_t v[kGivenBatch], own[kTurns][kGroups];
    auto request = [&](int from) {
#pragma unroll
        for (int i = 0; i < kGivenBatch; ++i) v[i] = idx.load<int32_t>(from + tid + i * TH);
    };
    request(0);
#pragma unroll
    for (int q = 0; q < kTurns; ++q)
#pragma unroll
        for (int h = 0; h < kGroups; ++h) own[q][h] = idx.load<int32_t>((t0 + h * 64 + lane) * k + wave + q * kWaves);
    __builtin_amdgcn_sched_barrier(0);
    while_waiting();
    // several counts of each, by lane: additions to one place in LDS are done one after the other
    uint32_t* const hist = &t.part[0][0][0];
    const int bins = k * N, pitch = bins + 1;
    int copies = 16;
    while (copies * pitch > (int)(sizeof(t.part) / 4)) copies >>= 1;
    for (int i = tid; i < copies * pitch; i += TH) hist[i] = 0;
    for (int i = tid; i < bins; i += TH) t.before[i] = 0;
    uint32_t* const mine_of = hist + (lane & (copies - 1)) * pitch;
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    for (int from = 0;;) {
        int p0 = from + tid;
        // With more than four choices the compiler would keep all sixteen sums with i * TH, in scratch memory in part (71 registers
        // so, 128 without); with fewer they fit and save time (8192 x 512 bytes, two: 12.6 us, 13.7 so).
        if constexpr (KK == 0) asm("" : "+v"(p0));
#pragma unroll
        for (int i = 0; i < kGivenBatch; ++i) {
            const int p = p0 + i * TH;
            if (p < n && (uint32_t)v[i] < (uint32_t)N) {
                const int tok = KK > 0 ? p / (KK > 0 ? KK : 1) : (int)__umulhi((uint32_t)p, a.k_magic);
                const int j = p - tok * k;
                __hip_atomic_fetch_add(mine_of + j * N + v[i], tok < t0 ? 0x10001u : 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        from += kGivenBatch * TH;
        if (from >= n) break;
        request(from);
    }
#pragma unroll
    for (int q = 0; q < kTurns; ++q) {
        const int j = wave + q * kWaves;
        if (j >= k) break;
#pragma unroll
        for (int h = 0; h < kGroups; ++h) {
            const int tok = t0 + h * 64 + lane;
            if (h > 0 && t0 + h * 64 >= t1) break;   // uniform
            const int mine = tok < t1 && (uint32_t)own[q][h] < (uint32_t)N ? own[q][h] : -1;
            uint64_t same = __ballot(mine >= 0);
#pragma unroll
            for (int b = 0; b < 7; ++b) {
                const bool bit = (mine >> b) & 1;
                const uint64_t with_bit = __ballot(bit);
                same &= bit ? with_bit : ~with_bit;
            }
            const int earlier = __popcll(same & ((1ull << lane) - 1ull));
            if (mine >= 0) {
                int32_t* cnt = t.before + j * N + mine;   // pairs of the groups before, this wavefront's alone so far
                const int32_t c = *cnt;
                t.rank[(tok - t0) * k + j] = (unsigned char)(c + earlier);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (earlier == 0) *cnt = c + __popcll(same);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    __syncthreads();
    for (int i = tid; i < bins; i += TH) {
        uint32_t w = hist[i];
#pragma unroll 4
        for (int c = 1; c < copies; ++c) w += hist[c * pitch + i];
        t.total[i] = (int32_t)w;
    }
    __syncthreads();
    if (tid < N) {
        int32_t run = 0;
#pragma unroll
        for (int j = 0; j < (KK > 0 ? KK : TAMOE_MAX_K); ++j) {
            if (KK == 0 && j >= k) break;
            const uint32_t w = (uint32_t)t.total[j * N + tid];
            t.before[j * N + tid] = run + (int32_t)(w >> 16);
            run += (int32_t)(w & 0xffffu);
        }
        const int32_t lim = pair_limit(cap_e, a.cap != nullptr, a.pad_C);
        t.pairs[tid] = run;
        t.kept[tid] = run < lim ? run : lim;
    }
    __syncthreads();
}
// Tiles before blk0 (B > 0), or tokens before t0 of a given routing (B == 0).
template <int TH, int KK, int B, class Body>
__device__ __forceinline__ void count_pairs(const RouteArgs& a, int blk0, int t0, int t1, TableLds<TH>& t, Body while_waiting) {
    if constexpr (B == 0) count_given<TH, KK>(a, t0, t1, t, while_waiting);
    else scan_counts<TH, KK, B>(a, blk0, t, while_waiting);
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
        count_pairs<TH, KK, B>(a, 0, 0, 0, *t, [&] {
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
        count_pairs<TH, KK, B>(a, 0, 0, 0, t, [] {});
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
    int t1 = 0;   // of a given routing: past the workgroup's last token
    if constexpr (B == 0) {
        int last, c1;
        if constexpr (ROWU) split_wave(first_unit + TH / 64 * U - 1, a.wpr, a.shift, last, c1);
        else split_chunk((int64_t)(first_unit + TH / 64 * U) * 64 - 1, total, cpr, a.shift, last, c1);
        t1 = last + 1 < (int)a.S ? last + 1 : (int)a.S;
    }
    // Slot of choice j of token tok, from its expert and position; -1: none, or dropped.  All lanes call.
    auto slot_of = [&](const WaveOffsets& wo, int32_t e, int32_t pos, int tok, int j, bool there) {
        const bool ok = there && (uint32_t)e < (uint32_t)N;
        e = ok ? e : 0;
        const int at = j * N + e;
        if constexpr (B == 0) {
            pos = t.before[at] + t.rank[ok ? (tok - t0) * k + j : 0];
        } else {
            pos += t.before[at];
            for (int b = blk0; b < tok >> a.tile_shift; ++b) pos += counts[(size_t)b * a.stride + at];   // tiles that begin inside this workgroup
        }
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
        const int32_t e = topk_idx[p], pos = B == 0 ? 0 : local_pos[p];
        int tok[U], seg[U];
        split_wave(unit0, a.wpr, a.shift, tok[0], seg[0]);
#pragma unroll
        for (int u = 1; u < U; ++u) {
            const bool next = seg[u - 1] + 1 == a.wpr;
            tok[u] = tok[u - 1] + next;
            seg[u] = next ? 0 : seg[u - 1] + 1;
        }
        // An offset for each unit is U registers, for which there is no room beside 16 rows of the table, or 16 indices and eight choices: a
        // row went to scratch memory as soon as it was there, ahead of the sums (8192 x 2 KiB, four choices, 64 experts 37.7 us, now
        // 36.7; 2048 x 8 KiB, eight, separate calls 76.7, 71.9).  There a unit's 64 chunks are a buffer of their own, with one offset
        // for all (elsewhere that is slower: separate calls of 16384 x 4 KiB, one choice 50.2, 50.4).
        constexpr bool kOwnBuffer = B > kTableBatch || (B == 0 && KK == 0);
        const auto begin = [&](int u) { return kOwnBuffer ? seg[u] * 64 : 0; };
        const auto col = [&](int u) { return kOwnBuffer ? lane : seg[u] * 64 + lane; };
        count_pairs<TH, KK, B>(a, blk0, t0, t1, t, [&] {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = tok[u] < a.S;
                v[u] = RowBuffer(x + (size_t)(in ? tok[u] : 0) * cpr + begin(u), cpr - begin(u), in).template load<LD>(col(u));
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
                RowBuffer(send + (size_t)(to >= 0 ? to : 0) * cpr + begin(u), cpr - begin(u), to >= 0).template store<ST>(col(u), v[u]);
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
                pos[u][j] = B == 0 ? 0 : local_pos[p];
            }
        }
        count_pairs<TH, KK, B>(a, blk0, t0, t1, t, [&] {
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

// How rows are moved: by whole wavefronts or flat, x loaded for the caches to keep or not, and how rows are stored.
struct RowPolicies {
    bool by_wave, keep;
    StorePolicy store;
};
// Launches for complete arguments, each in a translation unit of its own: with a table of pair counts, by choices, and with a
// routing that the scatter ranks itself (through L2, or flat rows from it).
void launch_route_table_few(const RouteArgs& a, const RowPolicies& how, hipStream_t st);
void launch_route_table_many(const RouteArgs& a, const RowPolicies& how, hipStream_t st);
void launch_route_given(const RouteArgs& a, const RowPolicies& how, hipStream_t st);

}  // namespace tamoe
