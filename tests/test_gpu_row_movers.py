"""The row movers on an MI355X at the edges of their layouts: rows of less than, exactly and just over a
wavefront's 1 KiB, rows longer than the largest workgroup, every compiled number of choices, dropped pairs,
slots beyond the receive buffer and an empty receive buffer; against the oracle or 64-bit sums."""
import numpy as np
import pytest
import torch

import tamoe_workloads as W
from test_gpu_parity import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2302_09915_amd as pkg

    pkg.lib()
    return pkg


def _case(seed, S, d, dtype, k, K_rows):
    rng = np.random.default_rng(seed)
    recv = W.to_storage(rng.standard_normal((max(K_rows, 1), d)).astype(np.float32), dtype)
    dy = W.to_storage(rng.standard_normal((S, d)).astype(np.float32), dtype)
    w = rng.uniform(0.01, 1.0, (S, k)).astype(np.float32)
    slot = np.full(S * k, -1, np.int32)
    kept = rng.permutation(S * k)[:K_rows]
    slot[kept] = rng.permutation(K_rows).astype(np.int32)
    dropped = np.flatnonzero(slot < 0)
    slot[dropped[::3]] = K_rows + 5                 # beyond the buffer: ignored like a dropped pair
    return recv, dy, w, slot.reshape(S, k)


@pytest.mark.parametrize("dtype", [W.BF16, W.F16, W.F32])
@pytest.mark.parametrize("S,chunks,k", [
    (1, 1, 1), (37, 3, 2), (130, 63, 3), (67, 64, 1), (66, 65, 2), (33, 125, 4), (31, 192, 5), (9, 256, 2), (65, 208, 8),
    (5, 1024, 2), (5, 1025, 3), (3, 2300, 1), (700, 8, 6), (257, 31, 4),
    (131, 65, 1), (67, 65, 3), (66, 65, 4), (45, 79, 2), (45, 80, 2), (37, 129, 4), (33, 143, 1), (33, 129, 5), (29, 144, 2), (29, 193, 2),
    (4095, 65, 2), (4096, 65, 2), (4100, 67, 1), (4100, 68, 3), (2731, 129, 2), (2731, 131, 4), (2731, 129, 1)])
def test_combine_and_backward_layouts(T, oracle, dtype, S, chunks, k):
    d = chunks * (4 if dtype == W.F32 else 8)
    for K_rows in (0, max(1, (S * k * 2) // 3)):
        recv, dy, w, slot = _case(S + chunks + k, S, d, dtype, k, K_rows)
        r64, g64 = W.storage_to_f64(recv, dtype), W.storage_to_f64(dy, dtype)
        use = (slot >= 0) & (slot < K_rows)
        rows = r64[np.where(use, slot, 0)]                                          # [S,k,d]
        terms = np.where(use[..., None], w[..., None].astype(np.float64) * rows, 0.0)
        sl, wd = torch.from_numpy(slot).cuda(), torch.from_numpy(w).cuda()
        rd, gd = to_dev(recv, dtype)[:K_rows], to_dev(dy, dtype)
        y = to_host(T.combine(rd, K_rows, sl, wd, d=d), dtype)
        exact = terms.sum(1)
        mag = np.abs(terms).sum(1)
        ulp = {W.F32: 2.0 ** -23, W.BF16: 2.0 ** -8, W.F16: 2.0 ** -11}[dtype]
        tiny = 2.0 ** -24 if dtype == W.F16 else 0.0                               # subnormal spacing of half precision
        bound = ulp * np.abs(exact) + tiny + 4 * k * 2.0 ** -24 * mag + 1e-40
        assert (np.abs(W.storage_to_f64(y, dtype) - exact) <= bound).all()
        # unit weights
        dx = torch.empty((S, d), dtype=gd.dtype, device="cuda")
        T.tamoe_dispatch_bwd(rd, K_rows, sl, dx)
        ones = np.where(use[..., None], rows, 0.0)
        e1, m1 = ones.sum(1), np.abs(ones).sum(1)
        b1 = ulp * np.abs(e1) + tiny + 4 * k * 2.0 ** -24 * m1 + 1e-40
        assert (np.abs(W.storage_to_f64(to_host(dx, dtype), dtype) - e1) <= b1).all()
        # backward: rows that no slot names stay as they were
        d_recv = torch.full((max(K_rows, 1), d), 7.0, dtype=gd.dtype, device="cuda")
        d_w = torch.full((S, k), 7.0, device="cuda")
        T.tamoe_combine_bwd(gd, rd, K_rows, sl, wd, d_recv[:K_rows], d_w)
        dots = np.where(use, (g64[:, None, :] * rows).sum(2), 0.0)
        dmag = np.where(use, np.abs(g64[:, None, :] * rows).sum(2), 0.0)
        assert (np.abs(d_w.cpu().numpy() - dots) <= d * 2.0 ** -24 * dmag).all()
        want = np.full((max(K_rows, 1), d), 7.0)
        t, j = np.nonzero(use)
        want[slot[t, j]] = w[t, j, None].astype(np.float64) * g64[t]
        got = W.storage_to_f64(to_host(d_recv, dtype), dtype)
        assert (np.abs(got - want) <= ulp * np.abs(want) + tiny + 1e-40).all()


@pytest.mark.parametrize("dtype", [W.BF16, W.F16, W.F32])
@pytest.mark.parametrize("k", range(1, 9))
def test_infinities_stay_with_their_pairs(T, dtype, k):
    """d_topk_w of a dropped pair is 0 whatever dy holds, and infinities, NaN and weights of one token reach no
    other and no dropped pair, on short rows (3 and 40 chunks), whole wavefronts (64) and several (130)."""
    tt = {W.BF16: torch.bfloat16, W.F16: torch.float16, W.F32: torch.float32}[dtype]
    for chunks in (3, 40, 64, 130):
        S, d = 24, chunks * (4 if dtype == W.F32 else 8)
        g = torch.Generator(device="cuda").manual_seed(chunks + k)
        dy = torch.randn(S, d, generator=g, device="cuda").to(tt)
        K_rows = S * k
        recv = torch.randn(K_rows, d, generator=g, device="cuda").to(tt)
        w = torch.rand(S, k, generator=g, device="cuda")
        slot = torch.randperm(K_rows, generator=g, device="cuda").int().reshape(S, k)
        slot[:6] = -1                                     # nothing kept
        slot[6:12, ::2] = -1                              # half of the choices
        slot[12:14, k - 1] = K_rows                       # beyond the buffer
        kept = (slot >= 0) & (slot < K_rows)
        for t, v in ((0, np.inf), (1, -np.inf), (2, np.nan), (6, np.inf), (7, np.nan), (12, -np.inf), (13, np.nan)):
            dy[t, [0, d // 2, d - 1][t % 3]] = v
        w[~kept] = float("nan")                           # a dropped pair's weight is not used either
        d_recv, d_w = torch.full_like(recv, 7.0), torch.full((S, k), 7.0, device="cuda")
        T.tamoe_combine_bwd(dy, recv, K_rows, slot, w, d_recv, d_w)
        rows = recv[slot.clamp(0, K_rows - 1).long()].double()
        terms = dy.double()[:, None, :] * rows
        want = torch.where(kept, terms.sum(2), 0.0).cpu()
        got = d_w.cpu().double()
        finite = torch.isfinite(want)
        assert torch.equal(torch.isfinite(got), finite) and torch.equal(torch.isnan(got), torch.isnan(want)), chunks
        assert torch.equal(got[~finite & ~torch.isnan(want)], want[~finite & ~torch.isnan(want)])
        bound = d * 2.0 ** -24 * torch.where(kept, terms.abs().sum(2), 0.0).cpu()
        assert ((got - want).abs()[finite] <= bound[finite]).all()
        assert (got[~kept.cpu()] == 0).all()
        t, j = torch.nonzero(kept, as_tuple=True)
        out = torch.full(recv.shape, 7.0, dtype=torch.float64, device="cuda")
        out[slot[t, j].long()] = w[t, j, None].double() * dy[t].double()
        there = torch.isfinite(out)
        assert torch.equal(torch.nan_to_num(d_recv.double()[~there], 5.0), torch.nan_to_num(out[~there], 5.0))
        # half an ulp is 2^-p of the value for p significant bits; one more rounding in fp32; half the subnormal
        # spacing of half precision
        half = {W.F32: 2.0 ** -24, W.BF16: 2.0 ** -8, W.F16: 2.0 ** -11}[dtype]
        assert ((d_recv.double() - out).abs()[there] <= ((half + 2.0 ** -23) * out.abs() + 2.0 ** -25)[there]).all()
        y = T.combine(recv, K_rows, slot, w)
        assert torch.isfinite(y).all() and (y[:6] == 0).all()


@pytest.mark.parametrize("chunks", [5, 64, 200])
def test_dropped_pairs_under_any_bound(T, chunks):
    """K_rows beyond the range of a slot (a caller without a bound): -1 and other negative slots stay dropped."""
    S, k, d = 33, 3, chunks * 8
    g = torch.Generator(device="cuda").manual_seed(chunks)
    recv = torch.randn(S * k, d, generator=g, device="cuda").bfloat16()
    dy = torch.randn(S, d, generator=g, device="cuda").bfloat16()
    w = torch.rand(S, k, generator=g, device="cuda")
    slot = torch.randperm(S * k, generator=g, device="cuda").int().reshape(S, k)
    slot[::2, 1], slot[::3, 0], slot[5] = -1, -(1 << 31), -7

    def run(K_rows):
        y, dx, d_recv, d_w = torch.empty_like(dy), torch.empty_like(dy), torch.full_like(recv, 7.0), torch.empty_like(w)
        L, st, p = T.lib(), torch.cuda.current_stream().cuda_stream, torch.Tensor.data_ptr
        assert L.tamoe_combine(p(recv), K_rows, p(slot), p(w), T.BF16, S, d, k, p(y), st) == T.OK
        assert L.tamoe_dispatch_bwd(p(recv), K_rows, p(slot), T.BF16, S, d, k, p(dx), st) == T.OK
        assert L.tamoe_combine_bwd(p(dy), p(recv), K_rows, p(slot), p(w), T.BF16, S, d, k, p(d_recv), p(d_w), st) == T.OK
        return y, dx, d_recv, d_w

    want = run(S * k)
    for bound in (1 << 31, 1 << 32, (1 << 32) + 5, (1 << 63) - 1):
        for a, b in zip(run(bound), want):
            assert torch.equal(a, b), bound


@pytest.mark.parametrize("P,E,chunks,mean", [(1, 1, 1, 3), (3, 2, 63, 4), (64, 2, 64, 3), (2, 64, 65, 2), (5, 7, 128, 0.3), (128, 1, 8, 5),
                                             (16, 4, 129, 20), (16, 4, 65, 400), (8, 3, 321, 250), (16, 4, 136, 190)])
@pytest.mark.parametrize("clip", [0, 7])
def test_regroup_layouts(T, P, E, chunks, mean, clip):
    rng = np.random.default_rng(P * 100 + chunks)
    cnt = rng.poisson(mean, (P, E)).astype(np.int32)               # empty segments among them
    cnt[rng.random((P, E)) < 0.1] = -3                              # counts as none
    c = np.maximum(cnt, 0)
    R = int(c.sum())
    rows = max(R - clip, 1) if clip else R + 3
    d = chunks * 8
    x = rng.integers(0, 1 << 15, (rows, d)).astype(np.int16)
    src = np.concatenate([[0], np.cumsum(c.reshape(-1))])           # source-major
    exp = np.concatenate([[0], np.cumsum(c.T.reshape(-1))])         # expert-major
    s_of, e_of = np.divmod(np.arange(P * E), E)
    to = np.full(max(R, rows), -1)
    for g in range(P * E):
        h = e_of[g] * P + s_of[g]
        to[src[g]:src[g + 1]] = exp[h] + np.arange(c[s_of[g], e_of[g]])
    want = np.full((rows, d), 9, np.int16)
    n = min(R, rows)
    ok = np.flatnonzero((to[:n] >= 0) & (to[:n] < rows))
    want[to[ok]] = x[ok]
    xd = torch.from_numpy(x).cuda().view(torch.bfloat16)
    out = torch.from_numpy(np.full((rows, d), 9, np.int16)).cuda().view(torch.bfloat16)
    off = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    ws = T.workspace(1, d, 1, 1, 1, T.BF16)
    cd = torch.from_numpy(cnt).cuda()
    T.tamoe_regroup(xd, cd, True, out, off, ws)
    np.testing.assert_array_equal(out.view(torch.int16).cpu().numpy(), want)
    np.testing.assert_array_equal(off.cpu().numpy(), exp[::P][:E + 1])
    if not clip:                                                    # and back
        back = torch.from_numpy(np.full((rows, d), 9, np.int16)).cuda().view(torch.bfloat16)
        T.tamoe_regroup(out, cd, False, back, off, ws)
        np.testing.assert_array_equal(back.view(torch.int16).cpu().numpy()[:R], x[:R])
        assert (back.view(torch.int16)[R:] == 9).all()
        np.testing.assert_array_equal(off.cpu().numpy(), exp[::P][:E + 1])


# (tokens, chunks per row, choices, whether the scatter takes the rows by wavefront, how it stores them): tests/test_row_stores.py
# holds this list and the next against the rules
BACK, STREAM, THROUGH, OUT = 0, 2, 16, 19
STORE_SHAPES = [
    (2048, 128, 2, 1, THROUGH), (5000, 64, 3, 1, THROUGH), (30720, 256, 2, 1, THROUGH), (30721, 256, 2, 1, OUT), (23040, 1024, 1, 1, THROUGH),
    (23041, 1024, 1, 1, OUT), (3000, 32, 2, 0, THROUGH), (61440, 32, 8, 0, THROUGH), (61441, 32, 8, 0, OUT),                       # whole lines
    (4000, 100, 2, 1, THROUGH), (21000, 100, 2, 1, STREAM), (60000, 84, 1, 1, STREAM), (10000, 36, 2, 0, BACK), (30000, 36, 2, 0, STREAM),   # half lines
    (11000, 137, 2, 1, THROUGH), (62914, 125, 2, 1, THROUGH), (62915, 125, 2, 1, STREAM), (31457, 125, 4, 1, THROUGH), (31458, 125, 4, 1, BACK),
    (2000, 125, 6, 1, THROUGH), (4000, 125, 6, 1, BACK), (21000, 125, 8, 1, BACK),                                                 # others, by wavefront
    (6000, 17, 3, 0, BACK), (32000, 65, 1, 0, BACK), (33000, 65, 1, 0, STREAM), (120989, 65, 2, 0, BACK), (120990, 65, 2, 0, STREAM)]   # flat
# (tokens, chunks, choices, rows per expert of 16, by wavefront, how rows are stored, whether padding streams)
PADDING_SHAPES = [
    (2000, 64, 2, 500, 1, THROUGH, 0), (9000, 128, 1, 2200, 1, THROUGH, 0), (20000, 128, 1, 2200, 1, THROUGH, 1), (9000, 128, 2, 3300, 1, THROUGH, 1),
    (70000, 128, 1, 4500, 1, OUT, 1), (16000, 128, 8, 9000, 1, OUT, 1), (9000, 125, 2, 2300, 1, THROUGH, 1), (8000, 125, 6, 3300, 1, BACK, 1),
    (70000, 125, 1, 4500, 1, STREAM, 1), (20000, 36, 2, 2600, 0, THROUGH, 0), (16000, 132, 4, 4100, 1, STREAM, 1), (1000, 8, 2, 200, 0, BACK, 0),
    (20000, 16, 2, 2600, 0, THROUGH, 0), (60000, 32, 2, 8000, 0, BACK, 0), (140000, 32, 2, 18000, 0, OUT, 1), (40000, 36, 2, 5100, 0, STREAM, 0),
    (9000, 64, 2, 1200, 1, THROUGH, 0)]


@pytest.mark.parametrize("S,chunks,k", [s[:3] for s in STORE_SHAPES])
def test_store_policies(T, S, chunks, k):
    """Rows scattered with every cache policy, on both sides of the sizes where one takes over from another, and what
    the other movers make of them."""
    g = torch.Generator(device="cuda").manual_seed(S + chunks)
    x = torch.randint(-32768, 32767, (S, chunks * 8), generator=g, device="cuda", dtype=torch.int16).view(torch.bfloat16)
    N = 16
    idx = torch.rand((S, N), generator=g, device="cuda").topk(k, 1).indices.int().contiguous()
    cap = torch.full((N,), S * k // N - 3, dtype=torch.int32, device="cuda")       # some pairs are dropped
    q = T.dispatch(x, idx, cap, N, N)
    slot, K = q["slot"], int(q["expert_offset"][-1])
    t, j = torch.nonzero(slot >= 0, as_tuple=True)
    assert t.numel() == K == int(q["kept_expert"].sum())
    same = lambda a, b: torch.equal(a.view(torch.int16), b.view(torch.int16))       # noqa: E731
    assert same(q["send"][slot[t, j].long()], x[t])
    # one row each: the transposes of the copy are copies too
    first = torch.full_like(slot, -1)
    first[:, 0] = slot[:, 0]
    there = first[:, 0] >= 0
    x0 = torch.where(there[:, None], x, torch.zeros_like(x)).nan_to_num(0.0, 0.0, 0.0)
    rows = q["send"].nan_to_num(0.0, 0.0, 0.0)
    y, dx = T.combine(rows, K, first, torch.ones((S, k), device="cuda")), torch.empty_like(x)
    T.tamoe_dispatch_bwd(rows, K, first, dx)
    assert torch.equal(y, x0) and torch.equal(dx, x0)
    d_recv, d_w = torch.full_like(rows, 7.0), torch.empty((S, k), device="cuda")
    T.tamoe_combine_bwd(x0, rows, K, first, torch.ones((S, k), device="cuda"), d_recv, d_w)
    want = torch.full_like(rows, 7.0)
    want[first[there, 0].long()] = x0[there]
    assert torch.equal(d_recv, want)
    # regrouping there and back
    cnt = torch.full((8, 2), S * k // 16, dtype=torch.int32, device="cuda")
    R = int(cnt.sum())
    by_expert, back = torch.empty_like(rows), torch.empty_like(rows)
    ws = T.workspace(1, chunks * 8, 16, 8, 1, T.BF16)
    T.tamoe_regroup(rows, cnt, True, by_expert, None, ws)
    assert torch.equal(by_expert[:R].view(2, 8, -1), rows[:R].view(8, 2, -1).transpose(0, 1))
    T.tamoe_regroup(by_expert, cnt, False, back, None, ws)
    assert torch.equal(back[:R], rows[:R])


@pytest.mark.parametrize("S,d,k,C", [(s[0], s[1] * 8, s[2], s[3]) for s in PADDING_SHAPES])
def test_padding_policies(T, S, d, k, C):
    """Rows of the fixed-size layout with every policy; unused rows are cleared whatever the size of the buffer."""
    g = torch.Generator(device="cuda").manual_seed(S + d)
    x = torch.randn((S, d), generator=g, device="cuda").bfloat16()
    N = 16
    idx = torch.rand((S, N), generator=g, device="cuda").topk(k, 1).indices.int().contiguous()
    cap = torch.full((N,), C, dtype=torch.int32, device="cuda")
    send = torch.full((N * C, d), 3.0, dtype=torch.bfloat16, device="cuda")
    slot, kept = torch.empty((S, k), dtype=torch.int32, device="cuda"), torch.empty(N, dtype=torch.int32, device="cuda")
    T.tamoe_dispatch_padded(x, idx, cap, N, N, C, send, slot, kept, T.workspace(S, d, N, N, k, T.BF16))
    want = torch.zeros_like(send)
    t, j = torch.nonzero(slot >= 0, as_tuple=True)
    want[slot[t, j].long()] = x[t]
    assert t.numel() == int(kept.sum()) and torch.equal(send, want)
