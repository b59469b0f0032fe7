// How the scatter is launched, by sizes.  Host code without HIP: the rules can be compiled and looked at anywhere.
#pragma once

#include <cstdint>

namespace tamoe {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- how rows lie on wavefronts, and tables in memory
// Rows of at least 64 chunks (1 KiB) are moved by whole wavefronts: a row takes row_waves(cpr) of them, the
// last one with idle lanes unless the row is a multiple of 1 KiB.  A wavefront then has one token, whose
// slots and weights go through the scalar unit, nothing is divided per lane, and a row is a buffer of its
// own (RowBuffer).  A flat layout of chunks over lanes has none of this, and gains only where most of a
// wavefront would idle (shorter rows).
inline bool rows_by_wave(int cpr) { return cpr >= 64; }
inline int row_waves(int cpr) { return (cpr + 63) / 64; }
// S rows just over one or two wavefronts, the last of which has fewer than `lanes` lanes and costs what the others
// cost, in a launch that is bound by that.  (Below 8192 wavefronts it is latency, and neither is better throughout: 2000
// rows of 1040 bytes, dispatch with one choice 6.6 us by wavefront, 6.9 flat, with three 9.1 and 8.6.)
inline bool poor_last_wave(int64_t S, int cpr, int lanes) {
    return row_waves(cpr) <= 3 && cpr % 64 > 0 && cpr % 64 < lanes && S * row_waves(cpr) >= 8192;
}
// Entries per row of the pair counts of a token tile: whole pieces of 16 bytes, a power of two of them.
inline int count_stride(int N, int k) {
    int pieces = 1;
    while (pieces * 8 < N * k) pieces *= 2;
    return pieces * 8;
}

// Gate: tokens per workgroup (32, 64, 128 or 256).
int gate_tile_tokens(int64_t S, int N);

// ---- a routing that is given: tokens of a workgroup that ranks it
// Few tiles keep the table of counts small; but with 512 tokens whatever k, the wavefronts did k turns one after the
// other in a handful of workgroups.  Two turns each (512 tokens, from three choices 256, from five 128), while an
// expert's counts stay within the 1024 that route_expert_kernel takes in one pass: 600 tokens, k = 8 9.5 -> 4.1 us,
// 16384, k = 8 10.9 -> 6.2, 5003, k = 4 6.6 -> 4.6, 65536, k = 4 6.1 -> 5.1 (512 tokens throughout -> now).
// Never below the gate's tiles, for which the table has room.
inline int rank_tokens(int64_t S, int N, int k) {
    int tok = k <= 2 ? 512 : k <= 4 ? 256 : 128;
    while (tok < 512 && (tok < gate_tile_tokens(S, N) || k * ceil_div(S, tok) > 1024)) tok *= 2;
    return tok;
}

// ---- how rows are moved
constexpr int copy_units(int k) { return k == 1 ? 2 : 1; }   // chunks per thread

// By wavefront or flat?  Flat with a poor last wavefront: 65536 rows of 2064 bytes, two choices 107.8 us by wavefront,
// 100.7 flat, 1040 bytes 53.4 and 51.5, one choice 31.9 and 28.6, whole calls on 8000 x 1040
// with two 14.9 and 13.4, on 8000 x 1184 with one 11.3 and 10.4; from 12 lanes on, or 4 behind two full wavefronts, the
// other way round (2288 bytes 47.6 and 49.2, 3184 bytes 78.7 and 85.3, calls on 30000 x 2176 43.5 and 45.5).  And flat with more than four choices, for
// which a wavefront keeps eight of everything, if a tenth of its lanes would idle and rows are no whole lines: 16500 x
// 2064, eight choices 105.6 and 96.7, 11520 x 6368 166.9 and 161.7; but 9000 x 4000, six choices (2 % idle) 2.9 us less
// by wavefront, and 1536 bytes (whole lines, 25 % idle) 5 us less behind the gate, 5 more on its own.
inline bool scatter_by_wave(int64_t S, int cpr, int k) {
    if (!rows_by_wave(cpr)) return false;
    if (poor_last_wave(S, cpr, row_waves(cpr) == 2 ? 12 : 4)) return false;
    const int lanes = row_waves(cpr) * 64;
    return k <= 4 || cpr % 8 == 0 || (lanes - cpr) * 10 <= lanes || S * row_waves(cpr) < 8192;
}

// Units of 64 chunks: of one row each, or anywhere (flat).
inline int64_t move_units(int64_t S, int cpr, int k) {
    return scatter_by_wave(S, cpr, k) ? S * row_waves(cpr) : ceil_div(S * (int64_t)cpr, 64);
}

// ---- who sums the table of pair counts, or counts a given routing
constexpr int kTableThreads = 512;   // or half as many (table_threads)
constexpr int kTableBatch = 8;   // rows per lane, requested together (one in the smallest tables, twice as many in large ones)

// Of a scatter that ranks a given routing itself: most pairs, those a thread requests at a time, most tokens of a workgroup.
constexpr int kGivenPairs = 16384, kGivenBatch = 16, kGivenTokens = 128;

// Units (64 chunks) per wavefront with which the scatter sums the table itself (route_table_kernel); 0: with
// route_expert_kernel and route_copy_kernel.
// The table has to be one batch of scan_counts: a second one is a second memory round trip (5003 x 2000 bytes, 157 tiles
// of 192 counts: 65.9 us for a training pass, 65.7 with the launch).  A batch of twice the pieces takes nearly all registers, which pays by wavefront
// while all workgroups are resident (forward calls with the launch and without: that size 29.8, 28.4, 3000 x 1 KiB, four choices, 126 experts 19.6,
// 18.2, 8192 x 2 KiB, four 39.0, 37.3 (36.3 with every register in its place); 32768 units 48.5, 49.0, 65536 of them 128.6, 134.0, flat 6000 x 512 18.1, 18.2).  Units: as many as leave a workgroup per compute
// unit, since each one sums the table (small_forward, 4096 units: with two 14.8, with one 17.5; gpt_moe_forward, 32768: with
// eight 43.0, with four 45.3; 6681 x 3456 bytes, eight choices, 26724: with eight 71.9, with two 75.0, with the launch 75.2); beyond 65536 of
// them (64 MiB of x) the launch that is saved counts for little (31106 x 2304, three, 93318: 102.4 with it, 99.9 without), and for a
// routing that is given, behind which x does not come from the last-level cache, beyond 32768 (skewed_separate, 65536: 53.7 with the
// launch, 54.7 without; fused, 16384 x 4 KiB, one choice 59.7 and 56.7).  Flat rows have the work of a slot in every lane, and
// at most two units (60623 x 256, one choice, 15156: 23.6 with the launch, 24.6 with two, 28.7 with one).
inline int table_units(int64_t S, int cpr, int N, int k, int tile_tokens, bool behind_gate) {
    // 16 bits hold the sums of a wavefront's share of the tiles, whatever the routing: with R = 512 / C rows of C pieces requested at a
    // time it has ceil(tiles / R) times max(1, 64 / C) tiles, (S + tile) / 8 + 64 * tile / C tokens at most (S / 4 + tile for C = 128), which
    // are 57 832 for S = 200 000, C = 1 and tiles of 512, and a token counts once per expert and choice
    const int64_t pieces = ceil_div(S, tile_tokens) * (count_stride(N, k) / 8);
    if (S > 200000 || pieces > 2 * kTableBatch * kTableThreads) return 0;
    const bool by_wave = scatter_by_wave(S, cpr, k);
    const int64_t units = move_units(S, cpr, k);
    if (units > (!by_wave ? 8192 : behind_gate ? 65536 : 32768)) return 0;
    int U = 1;
    while (U < (by_wave ? 8 : 2) && units >= kTableThreads / 64 * U * 2 * 256) U *= 2;
    // (one choice, and two of so few units, do not have as many pieces: no instances)
    if (pieces > kTableBatch * kTableThreads && (!by_wave || units >= 32768 || k == 1 || (k == 2 && U == 1))) return 0;
    return U;
}

// Units per wavefront with which the scatter counts a given routing itself, and its threads; 0: behind a launch that ranks it.
// A launch is 2.4 us on the host and 3 or more on the device.  Renormalisation, dispatch_padded and combine, us with it and without:
// 4096 x 128 bytes, two choices 14.6, 11.4, 4096 x 1 KiB, two 17.6, 11.2, 1024 x 1 KiB, eight 15.1, 12.8, 8192 x 512, two 17.7, 13.4, 6144 x 2 KiB, two, half of
// it padding 26.2, 22.4, 4096 x 4 KiB, two 28.7, 23.3; separate calls of 8192 x 256, two 37.5, 33.0, 16384 x 4 KiB, one 68.2, 61.8, 8192 x 8 KiB, two 91.3, 86.8.  Every workgroup reads all pairs:
// beyond kGivenPairs that takes longer than the launch (with 30000, 10000 x 256, three 15.8, 23.5).  It should be one of at most
// 256, as many units to a wavefront as that takes (5003 x 2000, three: 626 workgroups 23.0, 313 21.1; 3200 x 1 KiB, five 19.0, 16.1).
// It reads the rows of dropped tokens too, which the launch behind a ranking leaves out: with one choice and two of five pairs dropped it loses
// beyond 48 MiB of x what it gains where few are (renormalisation, dispatch_padded and combine of 16384 x 4 KiB 45.6, 47.6, none dropped 54.0, 51.6; separate
// calls of 12000 x 8 KiB 74.7, 77.7, none dropped 96.0, 91.0; of 16384 x 4 KiB 55.0, 50.5).
inline int given_units(int64_t S, int cpr, int N, int k, int* threads) {
    const int64_t units = move_units(S, cpr, k);
    const bool by_wave = scatter_by_wave(S, cpr, k);
    if (S <= 0 || S * k > kGivenPairs || units > (by_wave ? 131072 : 8192)) return 0;
    const bool half = units < kTableThreads / 64 * 256 && S * k <= kGivenBatch * kTableThreads / 2;
    *threads = half ? kTableThreads / 2 : kTableThreads;
    int U = 1;
    while (!half && U < (by_wave ? 8 : 2) && units > kTableThreads / 64 * U * 256) U *= 2;
    // flat: whole rows, or two more in part; by wavefront a unit is a row at most
    const int chunks = *threads * U;
    const int tokens = by_wave ? *threads / 64 * U : chunks % cpr == 0 ? chunks / cpr : (chunks - 2) / cpr + 2;
    return tokens <= kGivenTokens ? U : 0;
}

// Threads of a workgroup that sums the table: half as many where workgroups of 512 would be fewer than the compute units, as
// long as the table is one batch of theirs (forward calls, us with 512 and 256: 435 x 400 bytes, four choices 15.0, 14.4; 704 x 128,
// four 13.5, 12.7; 1024 x 1 KiB, 72 experts 14.9, 14.5; fixed-size layout, 704 x 352, eight 17.1, 15.7; 128 threads are no better: 1958 x
// 1792 13.8, 256 13.1).
inline int table_threads(int64_t S, int cpr, int k, int64_t pieces) {
    constexpr int kHalf = kTableThreads / 2;
    // a fourth of the tiles per wavefront: fits 16 bits, as in table_units
    return move_units(S, cpr, k) < kTableThreads / 64 * 256 && S <= 100000 && pieces <= kTableBatch * kHalf ? kHalf : kTableThreads;
}

}  // namespace tamoe
