"""How the scatter is launched (csrc/route_rules.h, csrc/store_rules.h, host code): the sizes of test_gpu_route_instances.py reach
every instance that any sizes reach, up to how rows are stored."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_09915_amd", "csrc")

# The instance that run_dispatch and run_copy choose, as a number: choices (0: more than four), units, rows by wavefront, threads, x kept,
# rows of the table requested together (0: a routing ranked by the scatter); 0 behind the per-expert launch.
RULES = """
#include <cmath>
#include <random>
#include <set>
#include "route_rules.h"
#include "store_rules.h"
using namespace tamoe;
static int key(int gate, int ranks, int k, int units, bool by_wave, int threads, bool keep, int batch) {
    return ((((((1 + 2 * gate + ranks) * 8 + (k <= 4 ? k : 0)) * 16 + units) * 2 + by_wave) * 2 + (threads == kTableThreads)) * 2 + keep) * 32 + batch;
}
extern "C" int instance(int64_t S, int cpr, int N, int k, int64_t C, int gate) {
    const bool by_wave = scatter_by_wave(S, cpr, k);
    const int64_t pairs = S * k, room = N * C, rows = C > 0 && room < pairs ? room : pairs, buffer = C > 0 ? room : rows;
    const RowLines lines = row_lines(nullptr, cpr);   // buffers that begin with a line
    const bool keeps = combine_load(S, buffer, cpr, k, lines) == kLoadKeep;
    int threads = 0, units = gate ? 0 : given_units(S, cpr, N, k, &threads);
    if (units > 0) {
        const StorePolicy s = scatter_store(lines, rows, cpr, k, by_wave, false, C > 0);
        if (s == kStoreThrough || (s == kStoreBack && !by_wave))
            return key(0, 1, k, units, by_wave, threads, units < 4 || !by_wave || scatter_load(S, buffer, cpr, C == 0, true, keeps) == kLoadKeep, 0);
    }
    const int tile = gate ? gate_tile_tokens(S, N) : rank_tokens(S, N, k);
    if ((units = table_units(S, cpr, N, k, tile, gate)) == 0) return 0;
    const int64_t pieces = ceil_div(S, tile) * (count_stride(N, k) / 8);
    threads = table_threads(S, cpr, k, pieces);
    const int batch = pieces > kTableBatch * threads ? 2 * kTableBatch : units == 1 && pieces <= threads ? 1 : kTableBatch;
    return key(gate, 0, k, units, by_wave, threads, units == 1 || scatter_load(S, buffer, cpr, C == 0) == kLoadKeep, batch);
}
// sizes drawn over the whole range: an instance and sizes for it, n of them at most
extern "C" int reach(int draws, int n, int64_t* out) {
    std::mt19937_64 rng(7);
    const auto log = [&](double lo, double hi) { return (int64_t)std::exp(std::uniform_real_distribution<>(std::log(lo), std::log(hi + 1))(rng)); };
    std::set<int> seen;
    for (int i = 0; i < draws; ++i) {
        const int k = 1 + (int)(rng() % 8), some[] = {(int)log(1, 128), 128, 64, k};
        const int N = std::max(k, some[rng() % 4]), lens[] = {(int)log(1, 2048), (int)log(1, 70), 64 * (1 + (int)(rng() % 16)), 65};
        const int64_t S = log(1, 200000), cpr = lens[rng() % 4], part[] = {1, 2, 4, 5, 8, 32};
        const int64_t C = rng() % 2 ? 0 : std::max<int64_t>(1, S * k * part[rng() % 6] / 4 / N);
        const int gate = C == 0 && rng() % 2;
        const int id = (S * (k + 1) + N * C) * cpr * 16 > (int64_t)8 << 30 ? 0 : instance(S, (int)cpr, N, k, C, gate);
        if (id == 0 || !seen.insert(id).second || (int)seen.size() > n) continue;
        const int64_t row[] = {id, S, cpr, N, k, C, gate};
        std::copy(row, row + 7, out + 7 * (seen.size() - 1));
    }
    return (int)seen.size();
}
"""


def test_gpu_tests_reach_every_instance(tmp_path):
    import paper_2302_09915_amd as T
    from test_gpu_route_instances import DISPATCH, GATE

    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    T.lib()
    home = os.path.dirname(T.LIB_PATH)
    src, so = tmp_path / "rules.cpp", tmp_path / "rules.so"
    src.write_text(RULES)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so), "-L", home, "-ltamoe",
                    f"-Wl,-rpath,{home}"], check=True)
    rules = ctypes.CDLL(str(so))
    rules.instance.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3 + [ctypes.c_int64, ctypes.c_int]
    tested = {rules.instance(S, cpr, N, k, 0, 1) for S, cpr, N, k in GATE} | {rules.instance(*s, 0) for s in DISPATCH}
    assert 0 not in tested
    found = (ctypes.c_int64 * (7 * 1000))()
    count = rules.reach(3000000, 1000, found)
    assert 150 < count <= 1000
    missed = [tuple(found[7 * i + 1:7 * i + 7]) for i in range(count) if found[7 * i] not in tested]
    assert not missed, missed
