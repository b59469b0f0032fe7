// How the row movers store their rows, and how they load them: a cache policy by size, by how rows lie on lines and by what comes next.  Host
// code without HIP: the rules can be compiled and looked at anywhere.
#pragma once

#include <cstdint>

namespace tamoe {

// Cache policies of the row stores (the bits of a buffer store).  A line that is dirty in an L2 when the kernel ends is
// written back then, with nothing to overlap, and evictions before that come in L2's order and not in that of the rows.
// Each row mover has a rule of its own, with what it measured.
enum StorePolicy {
    kStoreBack = 0,      // ordinary: the line waits in L2 until it is evicted or the kernel ends
    kStoreStream = 2,    // nt: the last-level cache does not keep the line
    kStoreThrough = 16,  // sc1: straight through L2; the last-level cache keeps the line
    kStoreOut = 19       // nt sc1 sc0: straight through L2, not kept
};

// Cache policies of the row loads.
enum LoadPolicy {
    kLoadKeep = 0,    // ordinary
    kLoadStream = 2   // nt: the caches let go of the line first
};

// How rows of cpr chunks of 16 bytes that begin at base lie on the lines of 128 bytes.  A line that a row shares with
// another is written in two parts, which only L2 can merge.  The length alone does not say it: buffers are aligned to 16
// bytes.  (Rows of whole lines in buffers that begin 48 bytes into one, us of a pass stored as if they were aligned, and
// now: regroup 17407 x 3200 bytes, four choices 171.8, 143.7, 10171 x 5632, two 92.8, 79.6; forward 11008 x 5376, eight
// 281.4, 228.6, 48222 x 3584, two 215.0, 187.9; backward 15009 x 4 KiB, two 95.4, 93.9.)
enum RowLines { kWholeLines, kHalfLines, kSharedLines };
inline RowLines row_lines(const void* base, int cpr) {
    const uintptr_t ends = reinterpret_cast<uintptr_t>(base) | (uintptr_t)cpr * 16;
    return ends % 128 == 0 ? kWholeLines : ends % 64 == 0 ? kHalfLines : kSharedLines;
}

// The scatter: how `rows` rows of send are written.  What decides is whether the last-level cache (256 MB) keeps them for whoever
// reads them next, and who merges the lines that a row shares with its neighbours.  Us of a whole forward call (recv = send)
// with ordinary / streaming / through stores:
//  - rows of whole lines go straight through L2 as long as they fit the last-level cache (576 x 7680 bytes, two choices (8 MiB)
//    25.8 / 25.1 / 25.3; 1919 x 3456, two 19.7 / 19.7 / 19.0; 30720 x 2 KiB, two 44.5 / 46.4 / 43.7; 23706 x 5504, two (249 MiB) - /
//    134.1 / 124.0, 29440 x 4608, two (259) - / 186.3 / 195.1; one choice, which leaves x less room to need, up to 360 MiB: 44244
//    x 7936 (335) - / 289.1 / 281.1), and beyond past that too (nt sc1 sc0, against nt alone: 65536 x 8 KiB, two 623.2 and
//    625.0, 65536 x 4 KiB, three 393.1 and 395.7; other rows lose by it, 30000 x 6368 258.7 and 247.5).  Flat ones behind the gate come
//    from L2 below 16 MiB (2123 x 256, four 14.2 / 15.0 / 14.4; 1280 x 384, four 15.0 / 15.9 / 16.2; 16640 x 640, two (20 MiB) 26.4 / 27.9 /
//    25.8), behind a routing that is given they gain nothing by it;
//  - rows of half lines stream beyond 16 MiB, also flat (9920 x 2112, four 64.5 / 60.7 / 63.3, 2880 x 2240, six 32.2 / 30.9 / 33.1;
//    41280 x 576, two 46.4 / 43.7 / 45.3, 45504 x 832, three 79.6 / 72.2 / 78.4, 33344 x 1600, eight 230.9 / 215.8 / 228.9);
//  - other rows by wavefront: through (9830 x 4000, two 45.8 / 46.1 / 44.9; 47185 x 2000, two 134.5 / 137.6 / 132.2), with many choices
//    and for large buffers of three and more from L2, which merges their lines (2496 x 2032, six 26.1 / 27.4 / 26.8, 11320 x 6368,
//    eight 273 / 287 / 286, 42567 x 4208, four (683 MiB) 384 / 397 / 390; 15440 x 5648, three, a training pass 337 / 349 / 336);
//  - other flat ones from L2 (57974 x 1040, four 111 / 136 / 121; 115651 x 272, two 61 / 65 / 65; 131072 x 880, eight (880 MiB) 422 / 441 /
//    453), streaming beyond 32 MiB with one choice (86016 x 544 57.7 / 54.3 / 58.0, 131072 x 720 108.1 / 100.1 / 108.2)
//    and beyond 240 with two (64384 x 2096 155.6 / 142.1 / -; 126256 x 688 (166 MiB) 133.9 / 141.2 / 143.3);
//  - the fixed-size layout goes by the rows that pairs can name (the padding between them is stored by fill_streams), which
//    nobody reads in the calls that were timed: beyond 128 MiB they leave the last-level cache to others (10880 x 6400, three (199 MiB) - /
//    112.0 / 115.0, 45284 x 2304, two (199) - / 127.5 / 130.4, 13248 x 2960, eight (299) 144.6 / 139.0 / -; 5333 x 4 KiB, two,
//    three of four rows padding (42) 55.6 / 62.4 / 55.4, 7245 x 2304, two, as many (32) 44.1 / 49.7 / 43.7, 1920 x 7984, eight (117) 79.4 / 87.7 /
//    82.0), and flat rows go through L2 from 4 to 24 MiB (3712 x 512, eight (14) 24.9 / 22.5 / 22.4, 12822 x 384, two
//    20.2 / - / 19.1, 7552 x 416, four (12) 19.9 / 18.1 / 18.3, those that share lines with more than four choices from 12 MiB: 2336 x
//    880, six (15) 22.1 / 20.1 / 20.7, but 4008 x 272, six (6) 18.4 / - / 19.1; 320 x 512, eight (1) 15.7 / - / 16.5, 13376 x 256, eight (26) 27.8 / - /
//    29.0, 30531 x 512, two (30) 31.3 / - / 31.9).
inline StorePolicy scatter_store(RowLines lines, int64_t rows, int cpr, int k, bool by_wave, bool behind_gate, bool padded) {
    const int64_t bytes = rows * cpr * 16, MiB = (int64_t)1 << 20;
    const bool leave = padded && bytes > 128 * MiB;
    if (padded && !by_wave && bytes <= 24 * MiB) return bytes < (k > 4 && lines == kSharedLines ? 12 : 4) * MiB ? kStoreBack : kStoreThrough;
    if (lines == kWholeLines) {
        if (!by_wave && (padded ? !leave : behind_gate && bytes < 16 * MiB)) return kStoreBack;
        return leave || bytes > (k == 1 ? 360 : 240) * MiB ? kStoreOut : kStoreThrough;
    }
    if (lines == kHalfLines && bytes > 16 * MiB) return kStoreStream;
    if (!by_wave) return !padded && ((k == 1 && bytes > 32 * MiB) || (k == 2 && bytes > 240 * MiB)) ? kStoreStream : kStoreBack;
    if (leave) return kStoreStream;
    if (bytes <= (k <= 4 ? 240 : 24) * MiB) return kStoreThrough;
    return k > 2 ? kStoreBack : kStoreStream;
}

// Where a mover finds everything it touches in the last-level cache, rows are loaded so that they stay there; beyond, what is read
// makes room for the rest.  Us of whole calls over the buffers of three layers in turn, with streaming / ordinary loads of the
// one mover.
// The scatter, x.  Behind the gate, which has just read x, in forward calls: 34176 x 288 bytes, one choice (19 MiB with the rows) 27.0 /
// 26.1, 2528 x 7232, eight (24) 42.7 / 39.0, 9486 x 2432, two (66) 41.6 / 39.8, 1007 x 8176, eight (71) 58.9 / 50.6, 15950 x 2432, two
// (111) 56.7 / 54.8; beyond 128 MiB either way (63985 x 768, two (141) 63.6 / 62.5, 6784 x 7552, two (147) 76.3 / 77.4, 65536 x 8 KiB, two 625
// / 637).  Of a routing that is given, in the fixed-size layout with ordinary loads of the combine: 39168 x 256, two (27) 24.3 / 22.6, 20098 x
// 512, three (39) 26.2 / 24.9, 3648 x 4608, two (48) 27.8 / 26.0; streaming ones there: 8926 x 2432, two (62) 34.8 / 36.1, 3693 x 8960, one (63) 38.5 /
// 41.4, 28736 x 1536, two (126) 59.5 / 62.6.  The rows are those of the buffer: 6144 x 2 KiB, two, half of 48 MiB padding 25.65 / 26.2, 11776 x 1 KiB, two,
// as much 31.6 / 34.2, 9856 x 1 KiB, two (47) 27.3 / 24.9.
// Ranked by the scatter itself, which waits for the counts meanwhile: 8192 x 4 KiB, one (72) 31.4 / 27.9, 3770 x 5888, two (62)
// 29.9 / 26.4, 1150 x 16 KiB, two, half padding (92) 32.2 / 29.0; 8192 x 4 KiB, two (96) 40.9 / 44.7, 5300 x 7 KiB, two (118) 46.4 / 49.2, 16384 x 4 KiB, one (140) 52.7 / 56.4.  Where
// the combine keeps the rows that come back, which lie in another buffer (combine_load), there is room for less beside them: streaming / ordinary
// 3481 x 4 KiB, two, half padding (68) 22.8 / 27.2, 7130 x 2000, two, half (68) 25.4 / 29.3, 5802 x 4 KiB, one, half (68) 24.7 / 26.9, 1820 x 4 KiB, four,
// half (64) 22.9 / 25.0, 3072 x 4 KiB, two, half (60) 20.3 / 21.5; 4437 x 4 KiB, one, half (52) 21.7 / 19.4, 2218 x 8 KiB, one, half (52) 21.4 / 19.5,
// 1331 x 8 KiB, two, half (52) 18.2 / 18.8.
constexpr int kKeepBehindGate = 128, kKeepRanking = 88, kKeepBoth = 54, kKeepGiven = 48;   // MiB of x and the rows sent
inline LoadPolicy scatter_load(int64_t S, int64_t rows, int cpr, bool behind_gate, bool ranks = false, bool combine_keeps = false) {
    const int most = behind_gate ? kKeepBehindGate : !ranks ? kKeepGiven : combine_keeps ? kKeepBoth : kKeepRanking;
    return (S + rows) * cpr * 16 <= (int64_t)most << 20 ? kLoadKeep : kLoadStream;
}

// Padding of the fixed-size layout: zeros stream where they would take the place of its rows in the last-level cache, which is in
// buffers of more than 96 MiB, and beyond 64 if they are not most of it; elsewhere they are stored as the rows are.  Us of a call
// streamed / as the rows: 1388 x 3840 bytes, 15 of 16 rows padding (81 MiB) 28.9 / 22.4, 673 x 3872, as many (80) 29.5 / 22.1, 25024 x
// 384, three of four (73) 34.6 / 31.3, 9152 x 640, seven of eight (89) 32.0 / 27.6; 5120 x 4304, half (84) 41.5 / 43.2, 40250 x 304, a
// fifth (87) 59.5 / 62.8, 8576 x 1920, half (94) 41.5 / 42.6; 2829 x 10 KiB, three of four (110) 43.7 / 49.6, 5333 x 4 KiB, three of
// four (167) 55.4 / 74.9, 53902 x 1536, half 78 / 86.
inline bool fill_streams(int64_t buffer_rows, int64_t rows, int cpr) {
    const int64_t bytes = buffer_rows * cpr * 16, MiB = (int64_t)1 << 20;
    return bytes > 96 * MiB || (bytes > 64 * MiB && 3 * rows > buffer_rows);
}

// The combine and its transpose: y goes straight through L2 and is not kept: ordinary stores are written back behind the last wavefront, and streaming
// ones still wait in L2 for their turn (the whole forward call on 16384 x 2 KiB, two choices: 47.8 us with ordinary
// stores, 47.5 streaming, 46.5 straight through; 65536 x 8 KiB 663, 625, 626).  Rows that are no whole lines only with three
// and more choices (18970 x 1520, four 75.2 streaming, 73.5; 23592 x 2000, four 109.3, 105.7); with two what is gained on rows
// from the last-level cache is lost on others (28835 x 2000 86.0, 84.5; fixed-size layout, 24898 x 5488 169.8, 171.9), with
// one all of it (28050 x 4112: 113.8, 116.6); and flat rows not at all (fixed-size layout, 15808 x 640, two 28.3, 28.8).
inline StorePolicy combine_store(RowLines lines, int64_t S, int cpr, int k, bool by_wave) {
    return by_wave && (k > 2 || lines == kWholeLines) && S * cpr * 16 <= (int64_t)256 << 20 ? kStoreOut : kStoreStream;
}

// The combine, the rows it reads (with what it writes): 768 x 7216, two choices (16 MiB) forward 18.6 / 17.5, 1664 x 4912, four (39)
// forward 34.4 / 32.5, 20098 x 512, three (39) fixed-size layout 26.8 / 24.9; forward 16159 x 1792, two (83) 34.8 / 34.6, 31936 x 640, four (98) 50.6 /
// 54.6, fixed-size layout 8926 x 2432, two (62) 34.8 / 36.1, 3693 x 8960, one (63) 38.5 / 42.7.  The buffer they lie in
// counts too: 6144 x 2 KiB, two, half of 48 MiB padding 26.2 / 25.4, 21193 x 768, two, half of 62 MiB 34.8 / 37.5.
// Above 40 MiB it depends on how the rows lie (42 to 47 MiB, streaming / kept): those that share lines gain whatever the call, as the
// line is wanted again (forward 6484 x 1520, four 30.0 / 26.8, 2737 x 2000, eight 29.9 / 28.0; separate calls 10807 x 1520, two 40.3 / 37.6, 2464 x 4000,
// four 37.6 / 35.0; training passes 6160 x 2000, three 59.1 / 56.4); others gain with up to three choices in training and with padding, and lose less
// in separate calls (14336 x 1 KiB, two 48.2 / 47.0; 10752 x 1 KiB, three, a fifth padding 27.1 / 25.9; 5312 x 2 KiB, three 31.1 / 32.1); with four
// and more those lose (8499 x 1 KiB, four 35.2 / 37.0, 2124 x 4 KiB, four 30.7 / 32.7, 1180 x 4 KiB, eight 32.4 / 36.4) what padding gains (8499 x 1 KiB,
// four 28.8 / 28.0).  And buffers beyond 48 MiB lose (half padding, 3788 x 4 KiB, two (59) 24.3 / 26.1, 30037 x 512, two (59) 34.4 / 36.3; 3520 x 2000, six, a
// fifth (50) 30.5 / 31.6).
inline LoadPolicy combine_load(int64_t S, int64_t buffer_rows, int cpr, int k, RowLines lines = kWholeLines) {
    const int64_t row = cpr * 16, MiB = (int64_t)1 << 20, own = S * (k + 1) * row;
    if (own > 40 * MiB && ((k > 3 && lines != kSharedLines) || buffer_rows > 48 * MiB / row)) return kLoadStream;
    return own <= 48 * MiB && buffer_rows <= 60 * MiB / row ? kLoadKeep : kLoadStream;
}
// Its transpose reads what combine_bwd has left there either way.  Rows that share lines gain, as the line is wanted again, up to 120 MiB of
// them: us of the three backward calls on 16448 x 2224, two (70 MiB) 50.5 / 46.9, 9791 x 4016, two (75) 60.2 / 56.8, 39321 x 2000, one (75) 75.5 / 72.2,
// 6867 x 8016, two (105) 79.4 / 77.7, 15697 x 8016, one (120) 109.7 / 107.7; but 15665 x 4016, two (120) 91.3 / 92.3, 8829 x 8016, two (135) 101.2 / 105.6,
// 45613 x 2000, two (174) 137 / 150, 45431 x 4016, one (174) 165 / 176.  (Passes of forward and backward with nothing between them over the buffers of
// three layers lose from 60 MiB on: 31457 x 2000, one 130.0 / 132.8, 6867 x 8016, two (105) 164.4 / 167.1.)  Not with three
// choices and more (10 to 188 MiB of rows of 1040 to 8016 bytes, either way within 1 %: 6640 x 2000, three 33.5 / 33.5, 8388 x 2000,
// four 48.6 / 48.5; 9168 x 8928, eight (625) 411 / 471), nor rows of whole lines (18911 x 1792, three 68.0 / 71.3, 25000 x 1536, two 45.5 / 45.6).
inline LoadPolicy dispatch_bwd_load(RowLines lines, int64_t S, int cpr, int k, bool by_wave) {
    return by_wave && k <= 2 && lines == kSharedLines && S * k * cpr * 16 <= (int64_t)120 << 20 ? kLoadKeep : kLoadStream;
}

// combine_bwd: d_recv goes straight through L2, whose last-level cache keeps what fits of it for the kernel that reads it
// next, and no dirty line is left for the end of this one.  Us of combine_bwd, dispatch_bwd and gate_bwd, rows with ordinary /
// streaming / through stores: 58880 x 2 KiB, two choices (combine_bwd and dispatch_bwd) 159 / 194 / 155, 25600 x 8 KiB, two 276 / 304 /
// 272, 65536 x 8 KiB, two 782 / 795 / 770; 1664 x 7296, two (23 MiB) 22.5 / 24.2 / 22.2, 2696 x 1536, four 16.7 / 16.8 / 16.4.  But
//  - flat rows of whole lines that fill their group of lanes are merged in L2, in buffers of up to 16 MiB: 2624 x 512 bytes, six
//    choices 14.6 / 15.6 / 15.4, 12838 x 512, two 15.2 / 15.7 / 15.6, 34682 x 256, two (17 MiB) 20.8 / 22.4 / 21.0; not 5760 x 640, two
//    13.1 / - / 12.2, 5893 x 768, two 13.5 / 12.9 / 12.6, 17498 x 384, three (19 MiB) 20.8 / 20.4 / 19.7, nor 10752 x 336, three 18.0 /
//    16.6 / 16.5;
//  - with one choice rows of half lines of up to 1.5 KiB stream beyond 48 MiB (107142 x 1344 142.7 / 132.2 / 139.0, 450000 x
//    320 168.1 / 154.2 / 165.7, but 58752 x 3520 182.9 / 186.1 / 180.1; two choices, 27200 x 3648 148.0 / 154.4 / 146.1), and so do
//    rows just over one wavefront, which two wavefronts write (129055 x 1040 148.4 / 139.6 / 145.3, 60000 x 1040 75.2 / 71.0 /
//    72.5, but 80000 x 1104 97.7 / 97.9 / 95.6).
inline StorePolicy combine_bwd_store(RowLines lines, int64_t S, int cpr, int k) {
    const int64_t bytes = S * k * cpr * 16;
    if (cpr < 64 && (cpr & (cpr - 1)) == 0 && lines == kWholeLines && bytes <= (int64_t)16 << 20) return kStoreBack;
    if (k == 1 && bytes > (int64_t)48 << 20 && (lines == kHalfLines ? cpr <= 96 : cpr > 64 && cpr < 68)) return kStoreStream;
    return kStoreThrough;
}

// combine_bwd, dy and recv (with the rows it writes), us of the three backward calls: 7762 x 768, two (28 MiB) 13.25 / 12.3, 6920 x 512, eight
// (57) 24.7 / 22.5, 12736 x 1152, two (70) 24.2 / 23.6; beyond 72 MiB either way (31931 x 640, two, 12 experts (97) 34.4 / 32.3, 32448 x 512, two, 128 experts,
// whose scores take as much again (79) 32.4 / 33.9, 11494 x 2304, two (126) 40.1 / 41.8, 19489 x 2048, four (343) 74.5 / 77.7).  Not short rows
// that share lines: 59392 x 224, two (63) 30.2 / 31.4; and flat rows, which have more scores to them, only up to 60 MiB: 57472 x 256,
// two, 72 experts (70) 31.7 / 32.0.
inline LoadPolicy combine_bwd_load(RowLines lines, int64_t S, int cpr, int k) {
    return S * (2 * k + 1) * cpr * 16 <= (int64_t)(cpr < 64 ? 60 : 72) << 20 && (cpr >= 64 || lines != kSharedLines) ? kLoadKeep : kLoadStream;
}

// The regroup: straight through L2 while the buffer fits the last-level cache, which keeps it for the experts (or the exchange),
// and streaming beyond; rows that share lines stream earlier.  Small buffers of flat rows are merged in L2 instead.  Us of one call
// with ordinary / streaming / through stores: 20480 x 2 KiB 28.3 / 30.1 / 27.0, 117760 x 2 KiB 146 / 142 / 139, 44800 x 8 KiB 230 / 213 / 220;
// 20971 x 2000 32.0 / 32.8 / 30.8, 34000 x 2320 (75 MiB) - / 53.6 / 50.0, 47185 x 2000 64.3 / 63.2 / 64.7, 120586 x 2000 155 / 148 / 174.  Both
// ways: 1340 x 384 7.4 / 7.4 / 8.0, 4852 x 384 (2 MiB) 6.9 / 7.0 / 7.2, 5120 x 176 7.9 / 8.4 / 8.5; 10551 x 512 (5 MiB) 10.1 / 9.7 / 9.7, 6480 x 608 (4
// MiB) 9.7 / - / 9.3, 27904 x 176 (5 MiB) 10.5 / - / 9.9, 19200 x 608 (11 MiB) 12.3 / 12.9 / 12.0.
inline StorePolicy regroup_store(RowLines lines, int64_t rows, int cpr) {
    const int64_t bytes = rows * cpr * 16, MiB = (int64_t)1 << 20;
    if (cpr < 64 && bytes <= 3 * MiB) return kStoreBack;
    return bytes > (lines == kSharedLines ? 80 : 256) * MiB ? kStoreStream : kStoreThrough;
}

// Its loads, us there and back streaming / ordinary: 1115 x 1280, four (5 MiB) 7.9 / 7.9, 4958 x 896, two (8.5) 11.3 / 10.3, 3328 x 1776, four (22.5)
// 21.8 / 17.7, 22.9 MiB of 1280 bytes 18.9 / 17.3; 31 MiB of 1 KiB 23.0 / 23.0, 40 of 512 bytes 32.1 / 32.8, 52 of 4864 bytes 33.9 / 38.0; 1893 x
// 256, six (3) 7.7 / 8.0.
inline LoadPolicy regroup_load(int64_t rows, int cpr) {
    const int64_t bytes = rows * cpr * 16, MiB = (int64_t)1 << 20;
    return bytes > 4 * MiB && bytes <= 24 * MiB ? kLoadKeep : kLoadStream;
}

}  // namespace tamoe
