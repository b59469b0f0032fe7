// tamoe_regroup: the step right after the global exchange (paper Section 3.1: each expert
// receives a combined batch of tokens).  The receive buffer holds one chunk per source device,
// each chunk grouped by local expert; the experts need one contiguous batch each.  Regrouping is
// a permutation of P*E contiguous row segments (and its inverse before the return exchange): a
// pure copy, bound by HBM (2 * R * d * b bytes for R rows).
//
// One launch: two wavefronts of every workgroup turn the P*E <= 128 counts into the two offset tables
// (source-major and expert-major, two entries per lane) with a few lane operations; a kernel of its own for
// that took 5 us in front of every call.  (Every wavefront for itself, without LDS and barrier, reads half
// as many bytes of counts as of rows: 2 GiB 308 -> 325 us.)
#include "internal.h"
#include "scan128.h"

namespace tamoe {

constexpr int kThreads = 256;
constexpr int kMaxSeg = TAMOE_MAX_EXPERTS;  // P * E <= 128

// x / P for 0 <= x < 256 and 1 <= P <= 128, with magic = ceil(65536 / P).
__device__ __forceinline__ int small_div(int x, int magic) { return (x * magic) >> 16; }

// The counts and how they lie; magic numbers for small_div.
struct Segments {
    const int32_t* cnt;
    int P, E, magic_P, magic_E;
};
// segment g of the `from` order -> the same segment in the `to` order
__device__ __forceinline__ int other_order(const Segments& sg, int g, bool to_expert_major) {
    if (to_expert_major) {               // g = s*E + e -> e*P + s
        const int s = small_div(g, sg.magic_E);
        return (g - s * sg.E) * sg.P + s;
    }
    const int e = small_div(g, sg.magic_P);
    return (g - e * sg.P) * sg.E + e;
}

// Exclusive offsets of the segments in both orders (entry n = P*E: the number of rows) in LDS, and the
// expert offsets by workgroup 0.  Every thread calls; ends with a barrier.
__device__ __forceinline__ void offset_tables(const Segments& sg, bool to_expert_major, int32_t* from_off, int32_t* to_off,
                                              int32_t* __restrict__ expert_offset) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = sg.P * sg.E;
    if (wave < 2) {   // one order each
        const bool expert_major = (wave == 0) != to_expert_major;
        int32_t c[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int h = lane + 64 * i;
            const int g = expert_major ? other_order(sg, h, false) : h;   // place in the counts
            const int32_t v = h < n ? sg.cnt[g] : 0;
            c[i] = v < 0 ? 0 : v;
        }
        const int32_t i0 = wave_inclusive_scan(c[0]);
        const int32_t i1 = wave_inclusive_scan(c[1]) + __builtin_amdgcn_readlane(i0, 63);
        const int32_t off[2] = {i0 - c[0], i1 - c[1]};
        int32_t* tab = wave == 0 ? from_off : to_off;
        const bool write = expert_major && linear_block() == 0 && expert_offset != nullptr;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int h = lane + 64 * i;
            if (h < n) tab[h] = off[i];
            const int e = small_div(h, sg.magic_P);
            if (write && h < n && e * sg.P == h) expert_offset[e] = off[i];
        }
        if (lane == 63) {
            tab[n] = i1;
            if (write) expert_offset[sg.E] = i1;
        }
    }
    __syncthreads();
}

// Rows by whole wavefronts, U segments of 64 chunks each; a row's segment of the table is found
// by counting the offsets that do not exceed it (one ballot per 64).
template <int U, int ST, int LD>
__global__ __launch_bounds__(kThreads) void regroup_copy_kernel(const vec16* __restrict__ in, const Segments sg,
                                                                int64_t cap_rows, int cpr, int wpr, int shift,
                                                                int to_expert_major, vec16* __restrict__ out,
                                                                int32_t* __restrict__ expert_offset) {
    __shared__ int32_t from_off[kMaxSeg + 1], to_off[kMaxSeg + 1];
    const int lane = threadIdx.x & 63, n = sg.P * sg.E;
    const uint32_t wave = linear_block() * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    offset_tables(sg, to_expert_major, from_off, to_off, expert_offset);
    const int32_t f0 = lane < n ? from_off[lane] : 0x7fffffff, f1 = lane + 64 < n ? from_off[lane + 64] : 0x7fffffff;
    const int32_t rows = __builtin_amdgcn_readfirstlane(from_off[n]);
    const int64_t R = rows < cap_rows ? rows : cap_rows;
    vec16 v[U];
    int32_t drow[U];
    int col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        int row, seg;
        split_wave(wave * U + u, wpr, shift, row, seg);
        col[u] = seg * 64 + lane;
        drow[u] = -1;
        if (row < R) {   // the same for the whole wavefront
            // largest g with from[g] <= row (empty segments are skipped)
            const int g = __popcll(__ballot(f0 <= row)) + __popcll(__ballot(f1 <= row)) - 1;
            drow[u] = __builtin_amdgcn_readfirstlane(to_off[other_order(sg, g, to_expert_major)] + (row - from_off[g]));
        }
        if (drow[u] >= cap_rows) drow[u] = -1;
        v[u] = RowBuffer(in + (size_t)(drow[u] >= 0 ? row : 0) * cpr, cpr, drow[u] >= 0).template load<LD>(col[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        RowBuffer(out + (size_t)(drow[u] >= 0 ? drow[u] : 0) * cpr, cpr, drow[u] >= 0).template store<ST>(col[u], v[u]);
}

// Other rows: chunks flat over the lanes, a chunk's segment by binary search over the offsets in LDS.
template <int U, int ST, int LD>
__global__ __launch_bounds__(kThreads) void regroup_flat_kernel(const vec16* __restrict__ in, const Segments sg,
                                                                int64_t cap_rows, int cpr, int shift, int to_expert_major,
                                                                vec16* __restrict__ out,
                                                                int32_t* __restrict__ expert_offset) {
    __shared__ int32_t from_off[kMaxSeg + 1], to_off[kMaxSeg + 1];
    const int n = sg.P * sg.E;
    offset_tables(sg, to_expert_major, from_off, to_off, expert_offset);
    const int64_t R = from_off[n] < cap_rows ? from_off[n] : cap_rows;
    const int64_t total = R * cpr;
    const int64_t base = (int64_t)linear_block() * (kThreads * U) + threadIdx.x;
    vec16 v[U];
    int64_t dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = base + (int64_t)u * kThreads;
        dst[u] = -1;
        if (c < total) {
            int row, col;
            split_chunk(c, total, cpr, shift, row, col);
            int lo = 0, hi = n;  // largest lo with from_off[lo] <= row (empty segments are skipped)
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (from_off[mid] <= row) lo = mid; else hi = mid;
            }
            const int64_t drow = (int64_t)to_off[other_order(sg, lo, to_expert_major)] + (row - from_off[lo]);
            if (drow < cap_rows) {
                dst[u] = drow * cpr + col;
                v[u] = load_chunk<LD>(in + c);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (dst[u] >= 0) store_chunk<ST>(out + dst[u], v[u]);
}

}  // namespace tamoe

using namespace tamoe;

extern "C" int tamoe_regroup(const void* in, const int32_t* recv_count, int P, int E, int dtype, int d,
                             int64_t cap_rows, int to_expert_major, void* out, int32_t* expert_offset, void* ws,
                             size_t ws_bytes, void* stream) {
    const char* fn = "tamoe_regroup";
    clear_error();
    int rc;
    if (P <= 0 || E <= 0) return fail(TAMOE_INVALID_ARG, "%s: P = %d and E = %d must be positive", fn, P, E);
    if ((int64_t)P * E > kMaxSeg)
        return fail(TAMOE_UNSUPPORTED, "%s: P*E = %lld exceeds the limit of %d segments", fn, (long long)P * E, kMaxSeg);
    if (cap_rows < 0 || cap_rows >= ((int64_t)1 << 31))
        return fail(TAMOE_INVALID_ARG, "%s: cap_rows = %lld outside [0, 2^31)", fn, (long long)cap_rows);
    int cpr = 0;   // 16-byte chunks per row
    if ((rc = check_rows(fn, dtype, d, &cpr)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "recv_count", recv_count, 4)) != TAMOE_OK) return rc;
    if ((rc = check_ptr(fn, "ws", ws, 256)) != TAMOE_OK) return rc;
    // the tables lie in LDS, ws is not touched; what it had to be when it held them is still asked for
    const size_t need = 2 * (kMaxSeg + 1) * sizeof(int32_t);
    if (ws_bytes < need) return fail(TAMOE_WORKSPACE_TOO_SMALL, "%s: workspace has %zu bytes, %zu needed", fn, ws_bytes, need);
    if (cap_rows > 0) {
        if ((rc = check_ptr(fn, "in", in, 16)) != TAMOE_OK) return rc;
        if ((rc = check_ptr(fn, "out", out, 16)) != TAMOE_OK) return rc;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    // two chunks per thread: the tables are made once per 8 KiB instead of once per 4 KiB
    // (2 GiB: 377 -> 341 us; four chunks: 350 us)
    constexpr int U = 2;
    // Rows that are no multiple of a line (128 bytes): flat, the wavefronts write whole lines across the ends of
    // rows; by wavefront every row ends in a partial line and, but for a multiple of 1 KiB, in idle lanes.  200000
    // x 1040 bytes, both ways: 166 us by wavefront, 145 flat; 60000 x 4112 174, 164; 40000 x 12016 321, 312.  Below 24 MiB
    // latency counts, and the search for a chunk's segment is longer flat: 3000 x 3184 12.5, 14.0.  Whole
    // lines go by wavefront at any size: 76288 x 7680 381, 406.
    const bool rowu = rows_by_wave(cpr) && (cpr % 8 == 0 || cap_rows * cpr * 16 <= (int64_t)24 << 20);
    const int wpr = row_waves(cpr);
    int64_t blocks = rowu ? ceil_div(cap_rows * wpr, kThreads / 64 * U) : ceil_div(cap_rows * cpr, kThreads * U);
    if (blocks > 0x7fffffff) return fail(TAMOE_UNSUPPORTED, "%s: the buffer is too large for one launch", fn);
    if (blocks == 0) {   // no rows: only the offsets, if they are asked for
        if (expert_offset == nullptr) return TAMOE_OK;
        blocks = 1;
    }
    const StorePolicy policy = regroup_store(row_lines(out, cpr), cap_rows, cpr);
    const Segments sg{recv_count, P, E, (65536 + P - 1) / P, (65536 + E - 1) / E};
    const vec16* src = static_cast<const vec16*>(in);
    vec16* dst = static_cast<vec16*>(out);
    const dim3 grid = grid_of(blocks, kThreads), block(kThreads);
    TraceScope tr("regroup_copy_kernel", st);
#define TAMOE_REGROUP(ST, LD)                                                                                      \
    do {                                                                                                           \
        if (rowu)                                                                                                  \
            launch_kernel(regroup_copy_kernel<U, ST, LD>, grid, block, st, src, sg, cap_rows, cpr, wpr, pow2_shift(wpr),    \
                                                                   to_expert_major, dst, expert_offset);           \
        else                                                                                                       \
            launch_kernel(regroup_flat_kernel<U, ST, LD>, grid, block, st, src, sg, cap_rows, cpr, pow2_shift(cpr),         \
                                                                   to_expert_major, dst, expert_offset);           \
    } while (0)
    if (policy == kStoreStream) TAMOE_REGROUP(kStoreStream, kLoadStream);
    else if (policy == kStoreBack) TAMOE_REGROUP(kStoreBack, kLoadStream);
    else if (regroup_load(cap_rows, cpr) == kLoadKeep) TAMOE_REGROUP(kStoreThrough, kLoadKeep);
    else TAMOE_REGROUP(kStoreThrough, kLoadStream);
#undef TAMOE_REGROUP
    return check_launch(fn, "regroup_copy_kernel");
}
