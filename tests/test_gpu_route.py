"""The stages behind a routing on an MI355X: the scatter that scans a small table of pair counts itself and the
one behind the per-expert kernel, at the sizes where one takes over from the other, on rows that are moved by
whole wavefronts and flat ones, packed and fixed-size; against the oracle and tamoe_dispatch_static, which
assigns slots with kernels of its own."""
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


@pytest.mark.parametrize("S,d,N,P,k", [
    (1, 8, 1, 1, 1), (511, 8, 3, 3, 1), (513, 520, 64, 8, 2), (1024, 512, 128, 64, 2), (1025, 512, 128, 64, 2),   # table / expert
    (4096, 512, 64, 64, 2), (4097, 512, 64, 64, 3), (3000, 16, 128, 2, 8), (70000, 8, 32, 4, 1),                   # blocks, tiles
    (2000, 1000, 48, 16, 4), (700, 512, 5, 5, 5), (9000, 1032, 128, 64, 8), (33, 4096, 16, 4, 6),
    (257, 8, 6, 3, 3), (129, 64, 10, 5, 5), (16384, 8, 16, 4, 8), (16385, 8, 16, 4, 8), (20000, 24, 128, 4, 5),    # tiles of the ranking
    (5000, 520, 16, 4, 1), (5000, 600, 16, 4, 2), (5000, 608, 16, 4, 2), (333, 1032, 16, 4, 3), (4000, 1112, 16, 4, 4),    # by wavefront
    (4000, 1120, 16, 4, 1), (900, 800, 16, 4, 5), (900, 1024, 16, 4, 6), (300, 1544, 16, 4, 2), (4095, 520, 16, 4, 2),     # or flat
    (8192, 64, 64, 64, 1), (8193, 64, 64, 64, 1), (4096, 64, 8, 8, 1), (4097, 64, 8, 8, 1), (1024, 72, 128, 64, 8), (1025, 72, 128, 64, 8),   # a routing ranked
    (512, 64, 128, 64, 8), (513, 64, 5, 5, 5), (1365, 56, 16, 4, 6), (1366, 128, 16, 4, 3), (2730, 1032, 10, 5, 3), (4096, 1024, 16, 4, 2), (8190, 512, 16, 4, 1), (2000, 32, 16, 4, 2),   # by the scatter
    (4096, 520, 16, 4, 2), (2731, 1048, 16, 4, 2), (2731, 1056, 16, 4, 2), (4200, 808, 16, 4, 5), (4096, 936, 16, 4, 5), (2800, 1032, 16, 4, 6)])
def test_dispatch_stages(T, oracle, S, d, N, P, k):
    rng = np.random.default_rng(S + d + N)
    x_np = W.to_storage(rng.standard_normal((S, d)).astype(np.float32), W.BF16)
    idx = W.random_routing(S + 3, S, N, k, skew=0.3).copy()
    idx[rng.random((S, k)) < 0.02] = -1                                        # no pair
    idx[rng.random((S, k)) < 0.02] = N                                         # out of range: no pair either
    cap = rng.integers(0, max(2, 2 * S * k // N), N).astype(np.int32)
    x, ix, cp = to_dev(x_np, W.BF16), torch.from_numpy(idx).cuda(), torch.from_numpy(cap).cuda()
    q = T.dispatch(x, ix, cp, N, P)
    s = {key: torch.empty_like(v) for key, v in q.items()}
    T.tamoe_dispatch_static(x, ix, cp, N, P, s["send"], s["slot"], s["kept_expert"], s["expert_offset"], s["send_count_dev"])
    torch.cuda.synchronize()
    K = int(q["expert_offset"][-1])
    for key in ("slot", "kept_expert", "expert_offset", "send_count_dev"):
        assert torch.equal(q[key], s[key]), key
    assert torch.equal(q["send"][:K].view(torch.int16), s["send"][:K].view(torch.int16))
    slot = q["slot"].cpu().numpy()
    np.testing.assert_array_equal(to_host(q["send"][:K], W.BF16), oracle.scatter(x_np, W.BF16, slot, K))
    # fixed-size layout: the same pairs in the same order, N * C rows, the unused ones zero
    C = max(1, int(cap.max()) // 2)
    ws = T.workspace(S, d, N, P, k, T.BF16)
    send = torch.full((N * C, d), 3.0, dtype=torch.bfloat16, device="cuda")
    slot_p, kept_p = torch.empty_like(q["slot"]), torch.empty_like(q["kept_expert"])
    T.tamoe_dispatch_padded(x, ix, cp, N, P, C, send, slot_p, kept_p, ws)
    torch.cuda.synchronize()
    off = q["expert_offset"].cpu().numpy()
    e = np.where(slot >= 0, np.searchsorted(off, slot, side="right") - 1, 0)
    pos = np.where(slot >= 0, slot - off[e], C)
    want = np.where((slot >= 0) & (pos < C), e * C + pos, -1)
    np.testing.assert_array_equal(slot_p.cpu().numpy(), want)
    np.testing.assert_array_equal(kept_p.cpu().numpy(), np.minimum(np.diff(off), C))
    rows = np.zeros((N * C, d), np.uint16)
    t, j = np.nonzero(want >= 0)
    rows[want[t, j]] = np.asarray(x_np).view(np.uint16)[t]
    np.testing.assert_array_equal(np.asarray(to_host(send, W.BF16)).view(np.uint16), rows)


@pytest.mark.parametrize("S,d,N,P,k", [(1, 8, 1, 1, 1), (600, 64, 8, 8, 1), (2048, 512, 32, 8, 2), (2049, 512, 32, 8, 2), (130, 1032, 128, 64, 8),
                                        (5000, 520, 16, 4, 1), (9000, 1032, 64, 8, 2), (777, 1000, 24, 3, 6)])
def test_fused_call_against_separate_calls(T, S, d, N, P, k):
    g = torch.Generator(device="cuda").manual_seed(S + d)
    x = torch.randn((S, d), generator=g, device="cuda").bfloat16()
    w = (torch.randn((N, d), generator=g, device="cuda") / d ** 0.5).bfloat16()
    pen = torch.rand(N, generator=g, device="cuda")
    cap = torch.randint(0, max(2, 2 * S * k // N), (N,), generator=g, device="cuda", dtype=torch.int32)
    f = T.gate_dispatch(x, w, P, k, pen, cap)
    a = T.gate(x, w, P, k)
    loss = T.aux_loss(a["m"], a["c_expert"], pen, P, S)
    q = T.dispatch(x, a["topk_idx"], cap, N, P)
    torch.cuda.synchronize()
    for key in ("logits", "topk_idx", "topk_w", "c_expert", "c_device"):
        assert torch.equal(f[key], a[key]), key
    for key in ("slot", "kept_expert", "expert_offset", "send_count_dev"):
        assert torch.equal(f[key], q[key]), key
    K = int(q["expert_offset"][-1])
    assert torch.equal(f["send"][:K].view(torch.int16), q["send"][:K].view(torch.int16))
    # sums of S (then N) 32-bit terms of one sign in another order
    torch.testing.assert_close(f["m"], a["m"], rtol=1e-5, atol=1e-9)
    torch.testing.assert_close(f["loss"], loss, rtol=1e-5, atol=0)


@pytest.mark.parametrize("S,d,N,P,k", [
    (33, 8, 2, 2, 2), (1000, 64, 3, 3, 1), (4095, 512, 16, 16, 2), (4096, 512, 16, 16, 2), (8191, 512, 40, 8, 2),        # units per wavefront
    (16390, 512, 40, 8, 1), (16384, 1024, 64, 64, 2), (16385, 1024, 33, 11, 3), (65536, 512, 16, 4, 2), (65537, 512, 16, 4, 2),   # and no more
    (3000, 1000, 64, 8, 4), (4128, 264, 64, 8, 4), (2000, 1544, 128, 8, 4), (2000, 264, 128, 8, 5), (1000, 1544, 128, 8, 8), (16384, 256, 16, 4, 2), (16385, 256, 16, 4, 2), (200000, 8, 8, 8, 2), (200001, 8, 8, 8, 2),  # columns
    (2047, 512, 16, 16, 2), (2048, 512, 16, 16, 2), (16376, 64, 8, 8, 2), (16385, 64, 8, 8, 2), (1024, 96, 64, 8, 8), (1025, 96, 64, 8, 8), (1030, 96, 128, 8, 2),   # smaller workgroups
    (256, 512, 128, 8, 4), (257, 512, 128, 8, 4), (31, 16, 128, 8, 8), (33, 64, 128, 8, 8),
    (16384, 512, 8, 8, 8), (16385, 512, 8, 8, 8), (8191, 512, 8, 8, 5), (8192, 512, 8, 8, 5), (16383, 512, 16, 4, 4), (16384, 512, 16, 4, 4), (9000, 1024, 16, 4, 3),   # a lane per pair
    (2047, 128, 64, 8, 8), (2049, 128, 64, 8, 8), (777, 136, 5, 5, 5), (513, 2056, 127, 127, 3)])
def test_table_summed_by_the_scatter(T, S, d, N, P, k):
    """The fused call and tamoe_dispatch on both sides of the rule that leaves out the per-expert launch, against
    tamoe_dispatch_static; some capacities keep nothing, some everything."""
    g = torch.Generator(device="cuda").manual_seed(S + d + N)
    x = torch.randn((S, d), generator=g, device="cuda").bfloat16()
    w = (torch.randn((N, d), generator=g, device="cuda") / d ** 0.5).bfloat16()
    pen = torch.rand(N, generator=g, device="cuda")
    cap = torch.randint(0, max(2, 2 * S * k // N), (N,), generator=g, device="cuda", dtype=torch.int32)
    cap[0], cap[N - 1] = 0, S
    f = T.gate_dispatch(x, w, P, k, pen, cap)
    q = T.dispatch(x, f["topk_idx"], cap, N, P)
    s = {key: torch.empty_like(v) for key, v in q.items()}
    T.tamoe_dispatch_static(x, f["topk_idx"], cap, N, P, s["send"], s["slot"], s["kept_expert"], s["expert_offset"], s["send_count_dev"])
    K = int(s["expert_offset"][-1])
    for key in ("slot", "kept_expert", "expert_offset", "send_count_dev"):
        assert torch.equal(q[key], s[key]), key
        assert torch.equal(f[key], s[key]), key
    assert torch.equal(q["send"][:K].view(torch.int16), s["send"][:K].view(torch.int16))
    assert torch.equal(f["send"][:K].view(torch.int16), s["send"][:K].view(torch.int16))
    count = torch.bincount(f["topk_idx"].reshape(-1).long(), minlength=N)
    assert torch.equal(f["c_expert"].long(), count) and torch.equal(f["c_device"].long(), count.view(P, -1).sum(1))
    # sums of S (then N) 32-bit terms of one sign
    m = torch.softmax(f["logits"].double(), 1).mean(0)
    torch.testing.assert_close(f["m"].double(), m, rtol=1e-5, atol=1e-9)
    torch.testing.assert_close(f["loss"].double().reshape(()), N * P / S * (pen.double() * m * count).sum(), rtol=1e-5, atol=0)


@pytest.mark.parametrize("S,d,k", [(200000, 8, 1), (200000, 8, 2), (199997, 16, 1), (100000, 8, 1), (100000, 8, 3), (65536, 32, 2), (131071, 8, 1), (4096, 512, 2)])
def test_all_tokens_to_the_same_experts(T, S, d, k):
    """The largest sums of pair counts that the scatter adds up 16 bits wide."""
    g = torch.Generator(device="cuda").manual_seed(S + k)
    x = torch.randint(-32768, 32767, (S, d), generator=g, device="cuda", dtype=torch.int16).view(torch.bfloat16)
    idx = torch.arange(k, device="cuda", dtype=torch.int32).flip(0).repeat(S, 1).contiguous()
    cap = torch.full((8,), S - 5, dtype=torch.int32, device="cuda")
    q = T.dispatch(x, idx, cap, 8, 8)
    s = {key: torch.empty_like(v) for key, v in q.items()}
    T.tamoe_dispatch_static(x, idx, cap, 8, 8, s["send"], s["slot"], s["kept_expert"], s["expert_offset"], s["send_count_dev"])
    for key in ("slot", "kept_expert", "expert_offset", "send_count_dev"):
        assert torch.equal(q[key], s[key]), key
    assert q["kept_expert"].tolist() == [S - 5] * k + [0] * (8 - k)
    K = k * (S - 5)
    assert torch.equal(q["send"][:K].view(torch.int16), s["send"][:K].view(torch.int16))
