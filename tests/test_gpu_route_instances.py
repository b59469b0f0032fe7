"""Every instance of the scatter that counts for itself on an MI355X, at the smallest sizes that reach it: the one that sums a table of pair
counts behind the gate or behind a ranking, and the one that ranks a given routing, with each number of units, threads and rows of the table,
on rows by wavefront and flat ones, x kept and streamed; against tamoe_dispatch_static, which has kernels of its own.
test_route_rules.py holds the sizes against the rules."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# tokens, 16-byte chunks per row, experts, choices
GATE = [
    (1, 1, 1, 1), (1, 64, 1, 1), (521, 64, 73, 1), (566, 1, 66, 1), (1024, 65, 1, 1), (1094, 65, 73, 1), (2050, 65, 1, 1), (2477, 53, 1, 1),
    (4132, 76, 1, 1), (4703, 1, 69, 1), (8194, 32, 1, 1), (9184, 76, 1, 1), (1, 1, 2, 2), (1, 64, 2, 2), (260, 1, 71, 2), (260, 64, 68, 2),
    (1024, 65, 2, 2), (1025, 65, 48, 2), (2048, 65, 2, 2), (2133, 1, 82, 2), (2981, 44, 2, 2), (4172, 64, 74, 2), (4248, 79, 2, 2),
    (4644, 76, 128, 2), (7943, 33, 2, 2), (8215, 77, 128, 2), (8464, 76, 18, 2), (14565, 192, 2, 2), (1, 1, 3, 3), (1, 64, 3, 3), (129, 65, 90, 3),
    (131, 1, 95, 3), (1024, 65, 3, 3), (1046, 65, 26, 3), (1065, 1, 97, 3), (2048, 65, 3, 3), (2087, 65, 100, 3), (2113, 64, 92, 3), (2124, 62, 3, 3),
    (4158, 76, 3, 3), (4274, 84, 64, 3), (7090, 37, 3, 3), (8249, 77, 48, 3), (8394, 78, 3, 3), (10923, 192, 3, 3), (1, 1, 4, 4), (1, 64, 4, 4),
    (129, 64, 65, 4), (143, 1, 65, 4), (1025, 65, 4, 4), (1045, 65, 18, 4), (1047, 1, 68, 4), (2049, 65, 4, 4), (2075, 64, 71, 4), (2080, 65, 72, 4),
    (2390, 55, 4, 4), (4103, 76, 4, 4), (4159, 79, 48, 4), (5746, 292, 48, 4), (7710, 34, 4, 4), (8204, 80, 64, 4), (8524, 77, 4, 4),
    (13110, 128, 4, 4), (1, 1, 5, 5), (1, 64, 5, 5), (65, 65, 106, 5), (513, 64, 128, 5), (1024, 65, 5, 5), (1025, 64, 128, 5), (2048, 65, 5, 5),
    (2050, 65, 64, 5), (3028, 152, 64, 5), (3290, 40, 5, 5), (4173, 80, 5, 5), (6031, 152, 48, 5), (7109, 37, 5, 5), (8285, 80, 5, 5),
    (2696, 446, 48, 6), (75, 1, 65, 8), (590, 1, 68, 8), (1766, 528, 8, 8), (3038, 308, 48, 8), (3292, 289, 10, 8),
]
# and rows per expert of the fixed-size layout, 0: packed
DISPATCH = [
    (1, 1, 1, 1, 0), (1, 2, 1, 1, 0), (1, 64, 1, 1, 0), (1024, 65, 1, 1, 0), (1025, 65, 1, 1, 0), (2050, 65, 1, 1, 0), (2477, 53, 1, 1, 0),
    (4132, 76, 1, 1, 0), (4153, 4, 1, 1, 0), (4358, 96, 1, 1, 34864), (6145, 64, 1, 1, 49160), (16388, 64, 1, 1, 0), (16456, 64, 2, 1, 16456),
    (16555, 1, 34, 1, 0), (19428, 18, 1, 1, 155424), (23847, 11, 1, 1, 0), (26220, 5, 1, 1, 0), (33902, 4, 35, 1, 0), (1, 1, 2, 2, 0),
    (1, 2, 2, 2, 0), (1, 64, 2, 2, 0), (1024, 65, 2, 2, 0), (1026, 65, 2, 2, 0), (2052, 65, 2, 2, 0), (2054, 4, 2, 2, 0), (2981, 44, 2, 2, 0),
    (3208, 65, 2, 2, 25664), (4248, 79, 2, 2, 0), (4620, 1, 65, 2, 0), (4737, 91, 16, 2, 2368), (8192, 512, 64, 2, 0), (8195, 64, 2, 2, 0),
    (8457, 76, 2, 2, 16914), (8464, 76, 18, 2, 0), (8784, 15, 2, 2, 0), (9834, 64, 2, 2, 19668), (13147, 20, 2, 2, 0), (16522, 8, 46, 2, 0),
    (34982, 10, 2, 2, 139928), (1, 1, 3, 3, 0), (1, 2, 3, 3, 0), (1, 64, 3, 3, 0), (364, 964, 3, 3, 0), (960, 527, 16, 3, 360), (1024, 65, 3, 3, 0),
    (1025, 65, 3, 3, 0), (1065, 1, 97, 3, 0), (1376, 4, 3, 3, 0), (2050, 65, 3, 3, 0), (2124, 62, 3, 3, 0), (2185, 65, 3, 3, 17480),
    (4158, 76, 3, 3, 0), (4226, 84, 16, 3, 0), (4227, 108, 16, 3, 1585), (5711, 23, 3, 3, 0), (7090, 37, 3, 3, 0), (7105, 64, 3, 3, 14210),
    (8394, 78, 3, 3, 0), (8461, 31, 16, 3, 6345), (8577, 1, 88, 3, 0), (9063, 76, 13, 3, 2614), (16451, 64, 100, 3, 0), (19821, 64, 128, 3, 232),
    (1, 1, 4, 4, 0), (1, 2, 4, 4, 0), (1, 64, 4, 4, 0), (1025, 64, 4, 4, 0), (1025, 65, 4, 4, 0), (1028, 4, 4, 4, 0), (1047, 1, 68, 4, 0),
    (2049, 65, 4, 4, 0), (2390, 55, 4, 4, 0), (2749, 136, 4, 4, 0), (3097, 135, 5, 4, 4955), (3221, 65, 4, 4, 12884), (4098, 32, 4, 4, 0),
    (4098, 64, 4, 4, 0), (4103, 76, 4, 4, 0), (4226, 95, 16, 4, 2113), (5389, 65, 4, 4, 10778), (5503, 64, 5, 4, 8804), (7710, 34, 4, 4, 0),
    (8385, 2, 70, 4, 0), (8406, 84, 64, 4, 525), (8524, 77, 4, 4, 0), (16405, 64, 66, 4, 0), (16449, 64, 128, 4, 257), (1, 1, 5, 5, 0),
    (1, 2, 5, 5, 0), (1, 64, 5, 5, 0), (1025, 65, 5, 5, 0), (1674, 585, 48, 5, 87), (2050, 65, 5, 5, 0), (2638, 50, 5, 5, 0), (2738, 192, 5, 5, 5476),
    (3004, 136, 5, 5, 0), (3290, 40, 5, 5, 0), (4101, 64, 125, 5, 0), (4143, 128, 128, 5, 161), (4173, 80, 5, 5, 0), (4416, 65, 6, 5, 7360),
    (4523, 64, 123, 5, 367), (4788, 80, 128, 5, 0), (5529, 80, 5, 5, 6911), (7109, 37, 5, 5, 0), (8285, 80, 5, 5, 0), (8437, 80, 64, 5, 0),
    (268, 1, 86, 6, 0), (2179, 65, 16, 6, 3268), (8216, 104, 48, 6, 513), (513, 64, 8, 8, 0), (515, 4, 8, 8, 0), (2050, 64, 8, 8, 0),
    (2050, 65, 8, 8, 0), (2084, 64, 18, 8, 0), (2108, 1, 73, 8, 0), (2651, 70, 8, 8, 5302),
]


@pytest.fixture(scope="module")
def T():
    import paper_2302_09915_amd as pkg

    pkg.lib()
    return pkg


def _static(T, x, idx, cap, N):
    S, k = idx.shape
    i32 = dict(dtype=torch.int32, device="cuda")
    s = {"send": torch.empty((S * k, x.shape[1]), dtype=x.dtype, device="cuda"), "slot": torch.empty((S, k), **i32), "kept_expert": torch.empty(N, **i32),
         "expert_offset": torch.empty(N + 1, **i32), "send_count_dev": torch.empty(1, **i32)}
    T.tamoe_dispatch_static(x, idx, cap, N, 1, *s.values())
    return s


def _same_dispatch(got, s):
    for key in ("slot", "kept_expert", "expert_offset", "send_count_dev"):
        assert torch.equal(got[key], s[key]), key
    K = int(s["expert_offset"][-1])
    assert torch.equal(got["send"][:K].view(torch.int16), s["send"][:K].view(torch.int16))


def _capacities(g, S, N, k):
    cap = torch.randint(0, max(2, 2 * S * k // N), (N,), generator=g, device="cuda", dtype=torch.int32)
    cap[N - 1] = S * k
    return cap


@pytest.mark.parametrize("S,cpr,N,k", GATE)
def test_behind_the_gate(T, S, cpr, N, k):
    g = torch.Generator(device="cuda").manual_seed(S + cpr + N)
    d = cpr * 8
    x = torch.randn((S, d), generator=g, device="cuda").bfloat16()
    w = (torch.randn((N, d), generator=g, device="cuda") / d ** 0.5).bfloat16()
    cap = _capacities(g, S, N, k)
    f = T.gate_dispatch(x, w, 1, k, None, cap)
    _same_dispatch(f, _static(T, x, f["topk_idx"], cap, N))
    count = torch.bincount(f["topk_idx"].reshape(-1).long(), minlength=N)
    assert torch.equal(f["c_expert"].long(), count)
    m = torch.softmax(f["logits"].double(), 1).mean(0)   # 32-bit sums of S terms of one sign
    torch.testing.assert_close(f["m"].double(), m, rtol=1e-5, atol=1e-9)


@pytest.mark.parametrize("S,cpr,N,k,C", DISPATCH)
def test_of_a_given_routing(T, S, cpr, N, k, C):
    g = torch.Generator(device="cuda").manual_seed(S + cpr + N)
    d = cpr * 8
    x = torch.randint(1, 30000, (S, d), generator=g, device="cuda", dtype=torch.int16).view(torch.bfloat16)
    idx = torch.argsort(torch.rand((S, N), generator=g, device="cuda") ** 2 + torch.arange(N, device="cuda") / N, dim=1)[:, :k].int()
    odd = torch.rand((S, k), generator=g, device="cuda")
    idx = torch.where(odd < 0.02, -1, torch.where(odd > 0.98, N, idx)).int().contiguous()   # no pairs
    cap = _capacities(g, S, N, k)
    s = _static(T, x, idx, cap, N)
    if C == 0:
        return _same_dispatch(T.dispatch(x, idx, cap, N, 1), s)
    send = torch.full((N * C, d), 3.0, dtype=torch.bfloat16, device="cuda")
    slot, kept = torch.empty_like(s["slot"]), torch.empty_like(s["kept_expert"])
    T.tamoe_dispatch_padded(x, idx, cap, N, 1, C, send, slot, kept, T.workspace(S, d, N, 1, k, T.BF16))
    assert torch.equal(kept, s["kept_expert"].clamp(max=C))
    at, e = s["slot"].long(), idx.clamp(0, N - 1).long()
    pos = at - s["expert_offset"].long()[e]
    want = torch.where((at >= 0) & (pos < C), e * C + pos, -1)
    assert torch.equal(slot.long(), want)
    t, j = torch.nonzero(want >= 0, as_tuple=True)
    assert torch.equal(send.view(torch.int16)[want[t, j]], x.view(torch.int16)[t])
    unused = torch.ones(N * C, dtype=torch.bool, device="cuda")
    unused[want[t, j]] = False
    assert not send.view(torch.int16)[unused].any()
