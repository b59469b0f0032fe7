// Internal declarations shared by the translation units of libtamoe (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstddef>
#include <cstdint>
#include <tuple>
#include <type_traits>

#include "route_rules.h"
#include "store_rules.h"
#include "tamoe.h"

namespace tamoe {

// 16 bytes as a native vector, the unit of every row copy (global_load/store_dwordx4).
typedef uint32_t vec16 __attribute__((ext_vector_type(4)));

// Records the message returned by tamoe_last_error() and passes `code` through.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline int elem_bytes(int dtype) { return dtype == TAMOE_F32 ? 4 : 2; }

// ---- launch geometry (host side; the kernels receive what they need as arguments) ----------

// Upper bound of the number of gate workgroups over every choice of tile.
inline int64_t gate_blocks_max(int64_t S) { return ceil_div(S, 32); }

// tamoe_dispatch_static: pairs are counted per "count tile" of kCountTile tokens.
constexpr int kCountTile = 1024;
inline int64_t count_tiles(int64_t S) { return ceil_div(S, kCountTile); }

// ---- workspace layout -----------------------------------------------------------------------
// Row pitch of the gate's pair-count table for `blocks` gate workgroups: a multiple of 64 entries, so
// that every expert's row starts on a 256-byte boundary and can be read in 16-byte pieces.
inline int64_t pair_pitch(int k, int64_t blocks) { return (int64_t)align_up((size_t)((int64_t)k * blocks), 64); }

struct Workspace {
    size_t m_part;      // float  [N][gate blocks]        per-workgroup sums of gate probabilities
    size_t tile_pairs;  // int32  [N][pair_pitch]         pairs per (expert; choice, token tile), then their
                        //                                exclusive prefix in priority order; or GateStats::counts
    size_t local_pos;   // int32  [S][k]                  position of a pair among those of its token tile
    size_t total;
};
Workspace workspace_layout(int64_t S, int N, int k);

// Where the block-wide results of the selection go (device memory, the caller's workspace).
struct GateStats {
    float* m_part;        // [N][n_blocks]      sums of gate probabilities per workgroup
    int32_t* tile_pairs;  // [N][pitch]         pairs per (expert; choice j, workgroup b) at [e*pitch + j*n_blocks + b]
    int32_t* local_pos;   // [S][k]             earlier pairs of the same workgroup with the same expert and choice
    int n_blocks;
    int pitch;
    uint16_t* counts;     // [n_blocks][stride] instead of tile_pairs, if not NULL: the pairs of (e, j) at j*N + e;
                          // m_part is then [n_blocks][sum_stride(N)]
    int stride;           // count_stride(N, k)
};
// Entries per row of m_part then and of `counts`: whole pieces of 16 bytes, a power of two of them.
__host__ __device__ constexpr int sum_stride(int N) {
    int pieces = 1;
    while (pieces * 4 < N) pieces *= 2;
    return pieces * 4;
}

// What the gate stage left in the workspace for the stages behind it.
struct GateRun {
    GateStats stats;
    int tile_tokens;      // tokens per gate workgroup: token t belongs to workgroup t / tile_tokens
};
// The gate's kernels up to the per-workgroup partial results (no finalize).  compact: the pair counts go to
// stats.counts, for a scatter that scans them itself.  Arguments are those of
// tamoe_gate / tamoe_select, already checked.
int run_gate_stage(const char* fn, const void* x, const void* w, int dtype, int64_t S, int d, int N, int k,
                   float* logits, int32_t* topk_idx, float* topk_w, bool compact, void* ws, const Workspace& lay,
                   hipStream_t st, GateRun* run);
GateStats stats_in(void* ws, const Workspace& lay, int N, int k, int64_t blocks, bool compact);
int run_select_stage(const char* fn, const float* logits, int64_t S, int N, int k, int32_t* topk_idx, float* topk_w,
                     void* ws, const Workspace& lay, hipStream_t st, GateRun* run);
// The dispatch of a routing that is given, arguments already checked: packed rows (pad_C == 0) or pad_C rows
// per expert (then expert_offset and send_count_dev may be NULL).  ws: laid out as `lay`.
int run_dispatch(const char* fn, const void* x, const int32_t* topk_idx, const int32_t* cap, int64_t S, int cpr, int N,
                 int P, int k, int pad_C, void* send, int32_t* slot, int32_t* kept_expert,
                 int32_t* expert_offset, int32_t* send_count_dev, void* ws, const Workspace& lay, hipStream_t st);
int check_select_outputs(const char* fn, int64_t S, int32_t* topk_idx, float* topk_w, float* m, int32_t* c_expert,
                         int32_t* c_device, void* ws, size_t ws_bytes, const Workspace& lay);

// Workgroups of a launch as a grid.  HIP takes fewer than 2^32 threads along a dimension: 16 777 216 workgroups of
// 256 are an invalid configuration, and of a few more only those run, without an error.  More go into rows
// of 2^20 workgroups, the last of which may have workgroups without work.  blocks < 2^31.
constexpr int kGridRowShift = 20;
inline dim3 grid_of(int64_t blocks, int threads) {
    if (blocks * threads < (int64_t)1 << 32) return dim3((unsigned)blocks);
    return dim3(1u << kGridRowShift, (unsigned)ceil_div(blocks, (int64_t)1 << kGridRowShift));
}
__device__ __forceinline__ uint32_t linear_block() { return blockIdx.x + (blockIdx.y << kGridRowShift); }

// log2(v) if v is a power of two, else -1.
inline int pow2_shift(int v) {
    if (v <= 0 || (v & (v - 1)) != 0) return -1;
    int s = 0;
    while ((1 << s) < v) ++s;
    return s;
}

// Chunk index -> (row, column) for a matrix of `cpr` 16-byte chunks per row.
__device__ __forceinline__ void split_chunk(int64_t c, int64_t total, int cpr, int shift, int& row, int& col) {
    if (shift >= 0) {
        row = (int)(c >> shift);
        col = (int)c & (cpr - 1);
    } else if (total <= 0xffffffffll) {
        const uint32_t r = (uint32_t)c / (uint32_t)cpr;
        row = (int)r;
        col = (int)((uint32_t)c - r * (uint32_t)cpr);
    } else {
        const int64_t r = c / cpr;
        row = (int)r;
        col = (int)(c - r * cpr);
    }
}

// Wavefront wv of a launch -> row and segment of 64 chunks in it.  shift: pow2_shift(wpr).  The rows of one
// device's memory are fewer than 2^31 wavefronts.
__device__ __forceinline__ void split_wave(uint32_t wv, int wpr, int shift, int& row, int& seg) {
    const uint32_t r = shift >= 0 ? wv >> shift : wv / (uint32_t)wpr;
    row = (int)r;
    seg = (int)(wv - r * (uint32_t)wpr);
}

// Pairs of expert e that may be kept: its capacity (none given: unlimited), and in the fixed-size
// layout (pad_C > 0) at most the pad_C rows that every expert owns.
__device__ __forceinline__ int32_t pair_limit(int32_t cap_e, bool has_cap, int pad_C) {
    int32_t c = has_cap ? (cap_e < 0 ? 0 : cap_e) : 0x7fffffff;
    if (pad_C > 0 && c > pad_C) c = pad_C;
    return c;
}
__device__ __forceinline__ int32_t pair_limit(const int32_t* __restrict__ cap, int e, int pad_C) {
    return pair_limit(cap != nullptr ? cap[e] : 0, cap != nullptr, pad_C);
}

// Rows that a slot can name: the kernels compare slots as unsigned numbers, so that one comparison leaves out a dropped
// pair (-1) too, whatever bound the caller gives.
inline int64_t slot_bound(int64_t K_rows) { return K_rows < (int64_t)1 << 31 ? K_rows : (int64_t)1 << 31; }

// A chunk by address, with one of the policies.  (s_nop: a vector instruction must not overwrite the data of a store of
// more than 8 bytes in the two wait states behind it, and the compiler looks at its own stores only.)
template <int ST>
__device__ __forceinline__ void store_chunk(vec16* p, vec16 v) {
    if constexpr (ST == kStoreThrough) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
    else if constexpr (ST == kStoreOut) asm volatile("global_store_dwordx4 %0, %1, off sc0 nt sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
    else if constexpr (ST == kStoreStream) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// A chunk by address, with one of the policies.
template <int LD>
__device__ __forceinline__ vec16 load_chunk(const vec16* p) {
    if constexpr (LD == kLoadStream) return __builtin_nontemporal_load(p);
    else return *p;
}

// A row as a buffer resource: the hardware returns zeros for a load and drops a store outside its `cpr`
// chunks, and a row that is not there (present == false) has none.  Lanes beyond the end of a row and
// dropped pairs need no branch then, and cost no memory access.  With a branch around each load the k
// rows of a token are requested one after the other: the compiler waits for the slot of the next between
// them.  row and present must be the same in every lane.
struct RowBuffer {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ RowBuffer(const void* row, int cpr, bool present)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), 0, present ? cpr * 16 : 0, 0x00020000)) {}
    template <int LD>
    __device__ __forceinline__ vec16 load(int col) const {
        return __builtin_bit_cast(vec16, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)((uint32_t)col * 16u), 0, LD));
    }
    template <int ST>
    __device__ __forceinline__ void store(int col, vec16 v) const {
        typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rsrc, (int)((uint32_t)col * 16u), 0, ST);
    }
};

// Common argument checks.  Return TAMOE_OK or a failure already recorded with fail().
int check_shape(const char* fn, int64_t S, int N, int P, int k);
int check_rows(const char* fn, int dtype, int d);
// check_rows for the row movers, with the number of 16-byte chunks per row: below 2^27 (a RowBuffer and its
// byte offsets hold less than 2 GiB).
int check_rows(const char* fn, int dtype, int d, int* cpr);
int check_ptr(const char* fn, const char* name, const void* p, size_t align);
int check_launch(const char* fn, const char* kernel);

// Launches kernel k without dynamic LDS; check_launch tells how it went.  (<<<>>> and hipGetLastError behind it are 2.4 us on the host,
// this 2.15; calls on small tensors are bound by it.)
void note_launch_error(hipError_t e);
template <class... P, class... A>
inline void launch_kernel(void (*k)(P...), dim3 grid, dim3 block, hipStream_t st, const A&... args) {
    static_assert(sizeof...(P) == sizeof...(A), "the kernel's arguments");
    std::tuple<std::remove_cv_t<P>...> values(static_cast<P>(args)...);
    std::apply(
        [&](auto&... v) {
            void* pointers[] = {const_cast<void*>(static_cast<const void*>(&v))...};
            const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(k), grid, block, pointers, 0, st);
            if (__builtin_expect(e != hipSuccess, 0)) note_launch_error(e);
        },
        values);
}

// Brackets one kernel launch with a pair of events while a trace is running (tamoe_trace_start);
// a single branch otherwise.
extern std::atomic<bool> g_trace_on;
bool trace_begin(const char* kernel, hipStream_t st);
void trace_end(hipStream_t st);
struct TraceScope {
    hipStream_t st;
    bool on;
    TraceScope(const char* kernel, hipStream_t s) : st(s), on(false) {
        if (g_trace_on.load(std::memory_order_relaxed)) on = trace_begin(kernel, st);
    }
    ~TraceScope() {
        if (on) trace_end(st);
    }
};

}  // namespace tamoe
