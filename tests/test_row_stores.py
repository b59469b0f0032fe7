"""How rows are stored: what the compiler makes of store_chunk (csrc/internal.h), and the rules that choose a cache
policy (csrc/store_rules.h, host code)."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_09915_amd", "csrc")

PROBE = """
#include "internal.h"
using namespace tamoe;
template <int ST> __global__ void probe(vec16* p, uint32_t z) {
    vec16 v = {threadIdx.x, z, z, z};
    p += threadIdx.x;
    for (int i = 0; i < 4; ++i) {
        store_chunk<ST>(p, v);
        __builtin_amdgcn_sched_barrier(0);
        v.w ^= v.x;   // into the register that was stored, nothing else between
        v.x += v.y;
        asm volatile("" ::: "memory");
    }
}
template __global__ void probe<kStoreBack>(vec16*, uint32_t);
template __global__ void probe<kStoreStream>(vec16*, uint32_t);
template __global__ void probe<kStoreThrough>(vec16*, uint32_t);
template __global__ void probe<kStoreOut>(vec16*, uint32_t);
"""


def _gaps(lines):
    """Wait states between each 16-byte store and the first instruction that writes its data registers."""
    out = []
    for i, line in enumerate(lines):
        m = re.match(r"global_store_dwordx4 \S+ v\[(\d+):(\d+)\],", line)
        if m is None:
            continue
        data, states = range(int(m[1]), int(m[2]) + 1), 0
        for after in lines[i + 1:]:
            nop = re.match(r"s_nop (\d+)", after)
            w = re.match(r"v_\w+ v(?:(\d+)|\[(\d+):(\d+)\]),", after)
            if w and any(r in data for r in range(int(w[1] or w[2]), int(w[1] or w[3]) + 1)):
                out.append(states)
                break
            states += int(nop[1]) + 1 if nop else 1
    return out


def test_data_of_a_store_is_not_overwritten_early(tmp_path):
    """A store of 16 bytes still reads its data in the two wait states behind it.  The compiler keeps them free behind
    its own stores; behind those it does not see, as many have to be part of them."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True, timeout=300)
    gaps = {}
    for name, body in re.findall(r"^_Z5probeILi(\d+)E\w+:(.*?)s_endpgm", asm.read_text(), flags=re.S | re.M):
        lines = [s.split(";")[0].strip() for s in body.splitlines()]
        gaps[int(name)] = _gaps([s for s in lines if re.match(r"(v|s|global)_", s)])
    assert sorted(gaps) == [0, 2, 16, 19] and all(len(g) >= 3 for g in gaps.values()), gaps
    need = min(gaps[0])   # the compiler's own
    assert need >= 2 and all(min(g) >= need for g in gaps.values()), gaps


BACK, STREAM, THROUGH, OUT = 0, 2, 16, 19
MIB = 1 << 20
RULES = """
#include "store_rules.h"
using namespace tamoe;
extern "C" {
int scatter(uint64_t base, int64_t rows, int cpr, int k, int by_wave, int behind_gate, int padded) {
    return scatter_store(row_lines((const void*)base, cpr), rows, cpr, k, by_wave, behind_gate, padded);
}
int combine(uint64_t base, int64_t S, int cpr, int k, int by_wave) { return combine_store(row_lines((const void*)base, cpr), S, cpr, k, by_wave); }
int combine_bwd(uint64_t base, int64_t S, int cpr, int k) { return combine_bwd_store(row_lines((const void*)base, cpr), S, cpr, k); }
int fill(int64_t buffer_rows, int64_t rows, int cpr) { return fill_streams(buffer_rows, rows, cpr); }
int regroup(uint64_t base, int64_t rows, int cpr) { return regroup_store(row_lines((const void*)base, cpr), rows, cpr); }
int scatter_ld(int64_t S, int64_t rows, int cpr, int kind) { return scatter_load(S, rows, cpr, kind == 1, kind == 2); }
int combine_ld(int64_t S, int64_t rows, int cpr, int k) { return combine_load(S, rows, cpr, k); }
int dispatch_bwd_ld(uint64_t base, int64_t S, int cpr, int k, int by_wave) { return dispatch_bwd_load(row_lines((const void*)base, cpr), S, cpr, k, by_wave); }
int combine_bwd_ld(uint64_t base, int64_t S, int cpr, int k) { return combine_bwd_load(row_lines((const void*)base, cpr), S, cpr, k); }
int regroup_ld(int64_t rows, int cpr) { return regroup_load(rows, cpr); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(RULES)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, str(d / "rules.cpp"),
                    "-o", str(d / "rules.so")], check=True, timeout=120)
    lib = ctypes.CDLL(str(d / "rules.so"))
    i64, u64, i32 = ctypes.c_int64, ctypes.c_uint64, ctypes.c_int
    lib.scatter.argtypes = [u64, i64] + [i32] * 5
    lib.combine.argtypes = [u64, i64] + [i32] * 3
    lib.combine_bwd.argtypes = [u64, i64] + [i32] * 2
    lib.fill.argtypes = [i64, i64, i32]
    lib.regroup.argtypes = [u64, i64, i32]
    lib.scatter_ld.argtypes = [i64, i64, i32, i32]
    lib.combine_ld.argtypes = [i64, i64, i32, i32]
    lib.dispatch_bwd_ld.argtypes = [u64, i64, i32, i32, i32]
    lib.combine_bwd_ld.argtypes = [u64, i64, i32, i32]
    lib.regroup_ld.argtypes = [i64, i32]
    return lib


@pytest.mark.parametrize("cpr", [8, 64, 128, 256, 320])
def test_rows_share_lines_where_the_buffer_is_not_aligned(rules, cpr):
    """A whole number of lines per row is not enough: in a buffer that begins inside a line every row shares its first and
    last with its neighbours, and is stored as rows of other lengths are."""
    at, off = 1 << 20, (1 << 20) + 48
    rows = 200 * MIB // (cpr * 16)
    assert rules.regroup(at, rows, cpr) == THROUGH and rules.regroup(off, rows, cpr) == STREAM == rules.regroup(at, rows, cpr + 1)
    for k in (1, 2, 4, 8):
        S = rows // k
        for by_wave in ((1, 0) if cpr >= 64 else (0,)):
            for n in (rows // 6, rows, 3 * rows):
                assert rules.scatter(off, n, cpr, k, by_wave, 1, 0) == rules.scatter(at, n * cpr // (cpr + 1), cpr + 1, k, by_wave, 1, 0)
            assert rules.combine(off, S, cpr, k, by_wave) == rules.combine(at, S, cpr + 1, k, by_wave)
        if cpr >= 64:
            assert rules.combine(at, S, cpr, k, 1) == OUT and rules.combine(off, S, cpr, k, 1) == (OUT if k > 2 else STREAM)
    assert rules.scatter(at + 64, rows, cpr, 2, 1, 1, 0) == rules.scatter(at, rows, cpr + 4, 2, 1, 1, 0)   # half lines


@pytest.mark.parametrize("S,cpr,k,policy", [
    (2624, 32, 6, BACK), (12838, 32, 2, BACK), (16 * MIB // (32 * 16 * 2), 32, 2, BACK),                        # flat, whole lines, small
    (16 * MIB // (32 * 16 * 2) + 1, 32, 2, THROUGH), (5760, 40, 2, THROUGH), (10752, 21, 3, THROUGH), (5000, 36, 1, THROUGH),
    (1000, 512, 2, THROUGH), (600, 512, 4, THROUGH), (1664, 456, 2, THROUGH), (65536, 512, 2, THROUGH),          # by wavefront
    (107142, 84, 1, STREAM), (66666, 60, 2, THROUGH), (58752, 220, 1, THROUGH), (20000, 84, 1, THROUGH),         # half lines
    (129055, 65, 1, STREAM), (60000, 67, 1, STREAM), (60000, 69, 1, THROUGH), (60000, 65, 2, THROUGH), (40000, 65, 1, THROUGH)])
def test_gradient_rows(rules, S, cpr, k, policy):
    """Where each policy of combine_bwd's rows begins and ends."""
    assert rules.combine_bwd(1 << 20, S, cpr, k) == policy


def _at(mib, cpr):
    """Rows of cpr chunks in mib MiB."""
    return mib * MIB // (cpr * 16)


@pytest.mark.parametrize("mib,cpr,k,by_wave,behind_gate,policy", [
    (8, 480, 2, 1, 1, THROUGH), (12, 216, 2, 1, 1, THROUGH), (20, 64, 4, 1, 1, THROUGH), (240, 256, 2, 1, 1, THROUGH),   # whole lines
    (241, 256, 2, 1, 1, OUT), (360, 256, 1, 1, 1, THROUGH), (361, 256, 1, 1, 1, OUT), (240, 32, 8, 0, 1, THROUGH), (241, 32, 8, 0, 1, OUT),
    (15, 32, 2, 0, 1, BACK), (16, 32, 2, 0, 1, THROUGH), (20, 32, 4, 0, 1, THROUGH), (2, 24, 4, 0, 1, BACK), (15, 32, 8, 0, 0, THROUGH),
    (15, 132, 2, 1, 1, THROUGH), (17, 132, 2, 1, 1, STREAM), (30, 140, 6, 1, 1, STREAM), (300, 300, 4, 1, 1, STREAM),    # half lines
    (15, 36, 2, 0, 1, BACK), (17, 36, 2, 0, 1, STREAM), (400, 100, 8, 0, 1, STREAM), (500, 220, 6, 0, 1, STREAM),
    (20, 125, 8, 1, 1, THROUGH), (25, 125, 8, 1, 1, BACK), (100, 125, 2, 1, 1, THROUGH), (100, 125, 4, 1, 1, THROUGH),     # others, by wavefront
    (241, 125, 2, 1, 1, STREAM), (241, 125, 3, 1, 1, BACK), (700, 263, 4, 1, 1, BACK), (700, 397, 8, 1, 1, BACK),
    (31, 45, 1, 0, 1, BACK), (33, 45, 1, 0, 1, STREAM), (240, 45, 2, 0, 1, BACK), (257, 131, 2, 0, 1, STREAM), (880, 55, 8, 0, 1, BACK)])
def test_scattered_rows(rules, mib, cpr, k, by_wave, behind_gate, policy):
    """Where each policy of the scatter's rows begins and ends."""
    assert rules.scatter(1 << 20, _at(mib, cpr), cpr, k, by_wave, behind_gate, 0) == policy


@pytest.mark.parametrize("mib,cpr,k,by_wave,policy", [
    (3, 32, 8, 0, BACK), (4, 32, 8, 0, THROUGH), (24, 32, 2, 0, THROUGH), (25, 32, 2, 0, BACK), (128, 32, 8, 0, BACK), (129, 32, 8, 0, OUT),
    (3, 256, 2, 1, THROUGH), (128, 256, 2, 1, THROUGH), (129, 256, 2, 1, OUT), (129, 256, 1, 1, OUT), (17, 132, 2, 1, STREAM), (300, 300, 6, 1, STREAM),
    (24, 125, 8, 1, THROUGH), (25, 125, 8, 1, BACK), (128, 125, 8, 1, BACK), (129, 125, 8, 1, STREAM), (128, 125, 2, 1, THROUGH), (129, 125, 4, 1, STREAM),
    (3, 53, 2, 0, BACK), (5, 53, 4, 0, THROUGH), (11, 53, 6, 0, BACK), (13, 53, 6, 0, THROUGH), (5, 48, 6, 0, THROUGH), (24, 53, 8, 0, THROUGH), (25, 53, 8, 0, BACK), (51, 53, 1, 0, BACK), (300, 45, 2, 0, BACK),
    (20, 36, 2, 0, THROUGH), (25, 36, 2, 0, STREAM)])
def test_rows_of_the_fixed_size_layout(rules, mib, cpr, k, by_wave, policy):
    """The rows go by their own size, whatever the padding between them."""
    assert rules.scatter(1 << 20, _at(mib, cpr), cpr, k, by_wave, 0, 1) == policy


@pytest.mark.parametrize("mib,part,streams", [
    (64, 1.0, 0), (65, 1.0, 1), (65, 0.5, 1), (96, 0.25, 0), (96, 1 / 16, 0), (97, 0.25, 1), (97, 0, 1), (10, 0, 0)])
def test_padding(rules, mib, part, streams):
    """Zeros stream in buffers beyond 96 MiB, and beyond 64 MiB unless most rows are padding."""
    for cpr in (1, 60, 240, 512):
        rows = _at(mib, cpr)
        assert rules.fill(rows, int(part * rows), cpr) == streams


@pytest.mark.parametrize("rows,cpr,off,policy", [
    (1340, 24, 0, BACK), (6144, 32, 0, BACK), (6145, 32, 0, THROUGH), (5120, 11, 0, BACK), (16384, 26, 0, THROUGH),      # flat
    (6000, 24, 48, BACK), (27810, 24, 48, THROUGH), (1024, 128, 0, THROUGH), (1000, 65, 0, THROUGH), (500, 128, 48, THROUGH),
    (_at(256, 128), 128, 0, THROUGH), (_at(257, 128), 128, 0, STREAM), (_at(256, 100), 100, 0, THROUGH), (_at(80, 145), 145, 0, THROUGH),
    (_at(81, 145), 145, 0, STREAM), (_at(81, 128), 128, 48, STREAM), (_at(300, 32), 32, 0, STREAM)])
def test_regrouped_rows(rules, rows, cpr, off, policy):
    """Where each policy of the regroup begins and ends."""
    assert rules.regroup((1 << 20) + off, rows, cpr) == policy


@pytest.mark.parametrize("units,U,by_wave", [(2047, 0.5, 1), (2047, 0.5, 0), (4095, 1, 1), (4095, 1, 0), (8191, 2, 1), (8192, 2, 0), (16383, 4, 1), (65536, 8, 1)])
def test_policies_of_the_scatter_that_sums_the_table(rules, units, U, by_wave):
    """launch_route_table_u leaves out the policies that no call of its size asks for: units of at most 1 KiB of x, times k."""
    base = {0: 1 << 20, 1: (1 << 20) + 64, 2: (1 << 20) + 48}
    for k in range(1, 9):
        most = int((64 if U == 8 else 4 * U) * (k if k <= 4 else 8))   # MiB of rows that the launch reckons with
        there = {THROUGH} | ({STREAM} if most > 16 else set())
        if not by_wave or (k > 4 and most > 24) or (k == 4 and most > 240):
            there.add(BACK)
        if by_wave and most > 128:
            there.add(OUT)
        cprs = (64, 96, 100, 128, 200, 512) if by_wave else (1, 8, 24, 36, 60, 63)
        for cpr in cprs:
            waves = (cpr + 63) // 64 if by_wave else cpr / 64
            for S in sorted({int(units / waves * f / 40) for f in range(1, 41)}):
                for lines in base:
                    for gate, padded in ((1, 0), (0, 0), (0, 1)):
                        assert rules.scatter(base[lines], S * k, cpr, k, by_wave, gate, padded) in there, (k, cpr, S, lines, gate, padded)


def test_gpu_tests_reach_every_policy(rules):
    """The shapes at which the GPU tests move rows are stored as they say, in every way there is."""
    from test_gpu_row_movers import PADDING_SHAPES, STORE_SHAPES

    for S, cpr, k, by_wave, policy in STORE_SHAPES:
        assert rules.scatter(1 << 20, S * k, cpr, k, by_wave, 0, 0) == policy, (S, cpr, k)
    for S, cpr, k, C, by_wave, policy, fill in PADDING_SHAPES:
        assert rules.scatter(1 << 20, min(S * k, 16 * C), cpr, k, by_wave, 0, 1) == policy, (S, cpr, k, C)
        assert rules.fill(16 * C, min(S * k, 16 * C), cpr) == fill, (S, cpr, k, C)
    for shapes, at in ((STORE_SHAPES, 3), (PADDING_SHAPES, 4)):
        for by_wave in (0, 1):
            assert {s[at + 1] for s in shapes if s[at] == by_wave} == {BACK, STREAM, THROUGH, OUT}
    for call, seen in (("combine", {OUT, STREAM}), ("combine_bwd", {BACK, STREAM, THROUGH}), ("regroup", {BACK, STREAM, THROUGH})):
        got = set()
        for S, cpr, k, by_wave, _ in STORE_SHAPES:
            got.add({"combine": lambda: rules.combine(1 << 20, S, cpr, k, by_wave), "combine_bwd": lambda: rules.combine_bwd(1 << 20, S, cpr, k),
                     "regroup": lambda: rules.regroup(1 << 20, S * k, cpr)}[call]())
        assert got == seen, call


KEEP = 0   # rows are loaded with ordinary loads; STREAM: with streaming ones


@pytest.mark.parametrize("cpr", [1, 16, 64, 125, 512])
def test_loaded_rows(rules, cpr):
    """Where the movers cease to load rows for the caches to keep, in MiB of what they touch."""
    for k in (1, 2, 3, 8):
        S = lambda mib, per: mib * MIB // (per * cpr * 16)   # noqa: E731  tokens of per rows each
        for gate, most in ((1, 128), (0, 48), (2, 88)):   # behind a gate, behind a ranking, ranking itself
            assert [rules.scatter_ld(S(m, k + 1), S(m, k + 1) * k, cpr, gate) for m in (most, most + 1)] == [KEEP, STREAM]
        most = 40 if k > 4 else 48
        assert [rules.combine_ld(S(m, k + 1), S(m, k + 1) * k, cpr, k) for m in (1, most, most + 1)] == [KEEP, KEEP, STREAM]
        assert [rules.combine_ld(100, rows, cpr, k) for rows in (0, _at(60, cpr), _at(61, cpr), 1 << 31)] == [KEEP, KEEP, STREAM, STREAM]
        at, off = 1 << 20, (1 << 20) + 48
        short = cpr < 64
        most = 60 if short else 72
        assert [rules.combine_bwd_ld(at, S(m, 2 * k + 1), cpr, k) for m in (most, most + 1)] == [STREAM if short and cpr % 4 else KEEP, STREAM]
        assert rules.combine_bwd_ld(off, S(most, 2 * k + 1), cpr, k) == (STREAM if short else KEEP)
        for m, by_wave in ((120, 1), (121, 1), (100, 0)):
            shared = KEEP if by_wave and k <= 2 and m <= 120 else STREAM
            assert rules.dispatch_bwd_ld(off, S(m, k), cpr, k, by_wave) == shared
            assert rules.dispatch_bwd_ld(at, S(m, k), cpr, k, by_wave) == (STREAM if cpr % 4 == 0 else shared)
    assert [rules.regroup_ld(_at(m, cpr), cpr) for m in (3, 5, 24, 25)] == [STREAM, KEEP, KEEP, STREAM]


def test_gpu_tests_reach_every_load_policy(rules):
    from test_gpu_row_movers import PADDING_SHAPES, STORE_SHAPES

    seen = {"scatter": set(), "padded": set(), "combine": set(), "dispatch_bwd": set(), "combine_bwd": set(), "regroup": set()}
    for S, cpr, k, C, by_wave, _, _ in PADDING_SHAPES:
        if S * k > 16384:   # not ranked by the scatter itself
            seen["padded"].add((by_wave, rules.scatter_ld(S, 16 * C, cpr, 0)))
    for S, cpr, k, by_wave, _ in STORE_SHAPES:   # packed: as behind a gate
        seen["scatter"].add((by_wave, rules.scatter_ld(S, S * k, cpr, 1)))
        seen["combine"].add((by_wave, rules.combine_ld(S, S * k, cpr, k)))
        seen["combine_bwd"].add((by_wave, rules.combine_bwd_ld(1 << 20, S, cpr, k)))
        seen["dispatch_bwd"].add((by_wave, rules.dispatch_bwd_ld(1 << 20, S, cpr, k, by_wave)))
        seen["regroup"].add((by_wave, rules.regroup_ld(S * k, cpr)))
    both = {(b, p) for b in (0, 1) for p in (KEEP, STREAM)}
    assert seen.pop("dispatch_bwd") == both - {(0, KEEP)}
    assert all(s == both for s in seen.values()), seen


def test_x_is_kept_beside_what_the_combine_keeps(rules, tmp_path):
    """A scatter that ranks the routing itself keeps x up to 88 MiB, or up to 54 where the combine keeps rows as well."""
    src, so = tmp_path / "both.cpp", tmp_path / "both.so"
    src.write_text("""#include "store_rules.h"
extern "C" int both(int64_t S, int64_t rows, int cpr, int keeps) { return tamoe::scatter_load(S, rows, cpr, false, true, keeps); }""")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    both = ctypes.CDLL(str(so)).both
    both.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    for cpr, k in ((64, 1), (125, 2), (512, 4)):
        S = lambda mib: mib * MIB // ((k + 1) * cpr * 16)   # noqa: E731
        for keeps, most in ((0, 88), (1, 54)):
            assert [both(S(m), S(m) * k, cpr, keeps) for m in (most, most + 1)] == [KEEP, STREAM]
        # half of the rows padding: what the combine reads decides
        for m in (50, 60, 80, 90):
            s = m * MIB // ((2 * k + 1) * cpr * 16)
            keeps = rules.combine_ld(s, 2 * s * k, cpr, k) == KEEP
            assert both(s, 2 * s * k, cpr, keeps) == (KEEP if m <= (54 if keeps else 88) else STREAM), (m, k)


def test_rows_the_combine_keeps_beyond_40_mib(rules, tmp_path):
    """Between 40 and 48 MiB it matters whether rows share lines, and how large the buffer is."""
    src, so = tmp_path / "lines.cpp", tmp_path / "lines.so"
    src.write_text("""#include "store_rules.h"
using namespace tamoe;
extern "C" int lines(int64_t S, int64_t rows, int cpr, int k, uint64_t base) { return combine_load(S, rows, cpr, k, row_lines((const void*)base, cpr)); }""")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    load = ctypes.CDLL(str(so)).lines
    load.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_uint64]
    whole, half, shared = 1 << 20, (1 << 20) + 64, (1 << 20) + 16
    for cpr in (16, 64, 512):
        for k in (1, 3, 4, 8):
            S = lambda mib: mib * MIB // ((k + 1) * cpr * 16)   # noqa: E731
            for base in (whole, half, shared):
                most = 40 if k > 3 and base != shared else 48
                assert [load(S(m), S(m) * k, cpr, k, base) for m in (1, 40, most, most + 1, 60)] == [KEEP, KEEP, KEEP, STREAM, STREAM]
                # a buffer of more rows than pairs
                assert [load(S(39), _at(m, cpr), cpr, k, base) for m in (48, 60, 61)] == [KEEP, KEEP, STREAM]
                assert [load(S(44), _at(m, cpr), cpr, k, base) for m in (48, 49)] == [KEEP if most == 48 else STREAM, STREAM]
