"""The gate's tile geometries on an MI355X: every tile size of every expert count and storage type at the
batch sizes where the rule changes (one tile more than compute units), with and without a tail of K, and
fp32 scores (three bfloat16 parts per value) against 64 bits over the exponent range."""
import math

import numpy as np
import pytest
import torch

import tamoe_workloads as W
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_2302_09915_amd as pkg

    pkg.lib()
    return pkg


@pytest.mark.parametrize("dtype", [W.BF16, W.F16, W.F32])
@pytest.mark.parametrize("S,d,N,P,k", [
    (31, 64, 32, 4, 1), (8192, 40, 31, 1, 2), (8193, 256, 32, 8, 3),                         # tiles of 32, 64
    (40, 256, 20, 4, 2), (40, 264, 20, 4, 2), (65, 1096, 31, 1, 3),                          # 32: short and long rows
    (33, 512, 64, 64, 2), (8192, 72, 33, 3, 4), (8193, 128, 64, 8, 1), (16385, 24, 48, 16, 2),   # 32, 64, 128
    (32, 8, 128, 64, 8), (8191, 136, 65, 5, 2), (8257, 64, 128, 32, 5), (16500, 32, 96, 8, 2),   # 32, 64, 128
    (32769, 24, 128, 64, 2), (33000, 64, 100, 4, 8),                                         # 256
    # steps of the small tiles: fewer, as many and more than wavefronts that share a row, a part of a step left over
    (1, 8, 1, 1, 1), (33, 64, 16, 4, 2), (95, 136, 16, 16, 8), (40, 256, 9, 3, 3), (40, 520, 16, 4, 2), (70, 1032, 16, 4, 2),
    (40, 1000, 17, 1, 2), (33, 1032, 32, 8, 2), (33, 2056, 32, 8, 2), (40, 128, 64, 8, 2), (40, 136, 33, 3, 2), (33, 1024, 48, 16, 4),
    (40, 1032, 64, 8, 2), (33, 3000, 64, 8, 2), (40, 512, 65, 5, 2), (33, 1016, 128, 8, 8), (33, 1040, 128, 8, 2),
    (8300, 64, 16, 4, 2), (8300, 264, 10, 5, 2), (16400, 40, 16, 4, 2), (8300, 72, 32, 8, 2), (8300, 600, 16, 4, 1),
    (8300, 504, 16, 4, 2), (8300, 512, 16, 4, 2), (16500, 520, 9, 3, 2), (32768, 136, 32, 8, 2), (8300, 128, 20, 4, 2),
    # shared steps and private ones: either side of the workgroups, steps and experts where one takes over
    (9700, 576, 16, 4, 2), (9600, 576, 16, 4, 2), (9700, 512, 16, 4, 2), (8300, 576, 32, 8, 2), (8800, 1600, 20, 4, 2), (8300, 1600, 20, 4, 2),
    (16500, 320, 32, 8, 2), (16500, 384, 32, 8, 2), (7700, 1152, 32, 8, 2), (7680, 1152, 32, 8, 2), (5760, 1664, 32, 8, 2),
    (5770, 1664, 32, 8, 2), (5770, 1536, 20, 4, 2), (5770, 1280, 17, 1, 1), (4700, 1088, 48, 8, 2), (4600, 1088, 48, 8, 2),
    (4700, 1152, 64, 8, 2), (6700, 1408, 50, 5, 2), (6600, 1408, 50, 5, 2), (70, 192, 64, 8, 2), (70, 288, 64, 8, 2), (70, 480, 64, 8, 2), (70, 576, 64, 8, 2),
    (70, 544, 64, 8, 2), (70, 608, 64, 8, 2), (70, 1216, 40, 8, 2), (70, 320, 128, 8, 2), (70, 352, 128, 8, 2), (70, 384, 100, 4, 2),
    (40, 524296, 16, 4, 2), (33, 524352, 20, 4, 2),                                          # rows of more than 1 MiB
])
def test_tile_edges(T, oracle, dtype, S, d, N, P, k):
    oracle.set_threads(oracle.max_threads())
    rng = np.random.default_rng(S * 7 + d)
    x = W.to_storage(rng.standard_normal((S, d)).astype(np.float32), dtype)
    w = W.to_storage((rng.standard_normal((N, d)) / math.sqrt(d)).astype(np.float32), dtype)
    beta = rng.uniform(1.0, 9.0, size=(P, P))
    _, pen, cap = T.tamoe_topo_pattern(beta, None, P, N, P // 2, k, S, 1.1, 1)
    full_parity(T, oracle, {"dtype": dtype, "N": N, "P": P, "k": k}, x, w, pen.astype(np.float64), cap)


@pytest.mark.parametrize("S,N", [(64, 32), (64, 64), (64, 128), (9000, 64), (33000, 128)])
def test_fp32_scores_over_the_exponent_range(T, S, N):
    """Rows of x scaled by powers of two from 2^-90 to 2^90.  A score is a 32-bit sum of d products with
    24-bit factors: error below d * 2^-24 of the sum of magnitudes in any order, and the parts left out of
    a product below 2^-21 of it."""
    d = 320
    g = torch.Generator().manual_seed(S + N)
    x = torch.randn((S, d), generator=g)
    w = torch.randn((N, d), generator=g) / math.sqrt(d)
    x *= torch.exp2(torch.linspace(-90, 90, S).round())[:, None]
    lg = T.gate(x.cuda(), w.cuda(), 1, 1)["logits"].cpu().double()
    ref = x.double() @ w.double().t()
    mag = x.double().abs() @ w.double().abs().t()
    assert ((lg - ref).abs() <= (d * 2.0 ** -24 + 2.0 ** -21) * mag).all()
    # and, in the 2-norm of a row, no more than a few roundings of the result
    rel = (lg - ref).norm(dim=1) / ref.norm(dim=1)
    assert rel.max() < 1e-6, rel.max()


@pytest.mark.parametrize("S,N,d", [(512, 8, 64), (2048, 8, 1024), (40000, 32, 512), (4096, 64, 1024), (16384, 64, 1024), (20000, 64, 264),
                                   (4096, 128, 256), (16384, 128, 512), (20000, 128, 1024), (33000, 128, 1024), (33000, 100, 200)])
def test_fp32_products_keep_their_bits(T, S, N, d):
    """Rows with one value: the score is one product, off by the rounding of the result (2^-24) and the terms left
    out (2^-22).  Rows of positive values: the errors of a 32-bit sum have either sign, so their mean over a batch
    is far below one rounding (2^-28: a sixteenth), where parts cut from every product would add up."""
    g = torch.Generator(device="cuda").manual_seed(S + d)
    w = torch.randn((N, d), generator=g, device="cuda")
    at = torch.randint(0, d, (S, 1), generator=g, device="cuda")
    one = torch.zeros((S, d), device="cuda").scatter_(1, at, torch.randn((S, 1), generator=g, device="cuda"))
    ref = one.double() @ w.double().t()
    err = (T.gate(one, w, 1, 1)["logits"].double() - ref).abs() / ref.abs()
    assert err.max() <= 2.0 ** -22 + 2.0 ** -24
    x, w = torch.rand((S, d), generator=g, device="cuda"), w.abs()
    ref = x.double() @ w.double().t()
    err = (T.gate(x, w, 1, 1)["logits"].double() - ref) / ref
    assert err.mean().abs() <= 2.0 ** -28
    # the roundings of a running sum of d / 8 partial products, 2^-24 at most each and a third of that in the mean
    assert err.norm() / math.sqrt(err.numel()) <= math.sqrt(d / 8) * 2.0 ** -24 / 3 + 2.0 ** -24


def _bf16_parts(v):
    """A 32-bit value as the sum of three bfloat16 values, each rounded to nearest."""
    parts, rest = [], v.clone()
    for _ in range(3):
        parts.append(rest.bfloat16().float())
        rest = rest - parts[-1]
    assert (rest == 0).all()
    return [p.double() for p in parts]


@pytest.mark.parametrize("S,N,d", [(33, 8, 64), (40, 16, 136), (40, 16, 1032), (100, 32, 512), (100, 31, 1032), (8300, 4, 256), (8300, 16, 264), (16500, 16, 1024),
                                   (8300, 32, 64), (16500, 20, 520), (40000, 32, 64), (20000, 64, 128), (33000, 128, 64),
                                   (40, 16, 262152), (33, 32, 262400)])                      # rows of more than 1 MiB
def test_fp32_terms_left_out(T, S, N, d):
    """What a product leaves out are its terms of the third order of parts that are rounded to nearest, of x and of W: seen in the
    difference of a product and its own value rounded to 32 bits, of which 24 bits cancel.  (Not in tiles of 32 tokens with
    more than 32 experts, where W's middle part is cut.)"""
    g = torch.Generator().manual_seed(S + d)
    e = torch.arange(N)
    tail = 2.0 ** -16 - 2.0 ** -23                            # of a middle part: 2^-16 once rounded, nothing when cut
    b = torch.where(e % 2 == 0, 1 + 2.0 ** -9 + tail + (e // 2) * 2.0 ** -15, 1 + torch.rand(N, generator=g))
    for a in (1 + 2.0 ** -8 - 2.0 ** -22, 1.0 + float(torch.rand(1, generator=g))):
        a = torch.tensor(a, dtype=torch.float32)
        x, w = torch.zeros((S, d)), torch.zeros((N, d))
        x[:, d - 2], x[:, d - 1] = a, 1.0
        w[:, d - 2], w[:, d - 1] = b, -(a.double() * b.double()).float()
        (_, am, al), (_, bm, bl) = _bf16_parts(a), _bf16_parts(b)
        left = am * bl + al * bm + al * bl
        exact = a.double() * b.double() + w[:, d - 1].double()
        got = T.gate(x.cuda(), w.cuda(), 1, 1)["logits"].cpu().double()
        # the products of first parts have 16 bits and their sum is exact; what they leave and the other terms are below
        # 2^-6, and a sum of those in 32 bits is off by 2^-31 at each of a dozen additions
        assert (got - (exact - left)).abs().max() <= 16 * 2.0 ** -30


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("S,N,d", [(40, 8, 40), (40, 8, 64), (40, 8, 192), (9000, 20, 72), (40, 64, 64), (9000, 48, 136), (20000, 64, 72),
                                   (40, 128, 192), (9000, 100, 200), (20000, 128, 40), (33000, 128, 72), (33000, 65, 128),
                                   (9000, 8, 1000), (40000, 32, 512), (9000, 64, 1024), (12160, 48, 832), (20000, 64, 1024), (70000, 128, 1024)])
def test_infinities_in_the_scores(T, dtype, S, N, d):
    """An expert masked with an infinite weight, infinities and NaN in x (the last elements of a row among them):
    the scores, and what follows from them, are those of the arithmetic itself."""
    k = 2
    g = torch.Generator(device="cuda").manual_seed(S + d)
    x = torch.randn((S, d), generator=g, device="cuda").to(dtype)
    w = (torch.randn((N, d), generator=g, device="cuda") / math.sqrt(d)).to(dtype)
    x[:, d - 1] = 1.0
    w[3, d - 1] = -math.inf                                      # expert 3 is masked
    odd = [5, 7, S - 3, S - 2]
    x[5, d - 2], x[S - 3, 0], x[7, 1], x[S - 2, d - 2] = math.inf, -math.inf, math.nan, math.inf
    r = T.gate(x, w, 1, k)
    lg = r["logits"].cpu().double()
    ref = x.cpu().double() @ w.cpu().double().t()
    assert torch.equal(torch.isnan(lg), torch.isnan(ref))
    inf = torch.isinf(ref)
    assert torch.equal(torch.isinf(lg), inf) and torch.equal(lg[inf], ref[inf])
    fin = torch.isfinite(ref)
    mag = torch.nan_to_num(x.cpu().double(), 0, 0, 0).abs() @ torch.nan_to_num(w.cpu().double(), 0, 0, 0).abs().t()
    assert ((lg - ref).abs()[fin] <= (d + 2) * 2.0 ** -24 * mag[fin]).all()
    plain = torch.ones(S, dtype=torch.bool)
    plain[odd] = False
    prob = torch.softmax(lg[plain], 1)
    idx, wgt = r["topk_idx"].cpu()[plain].long(), r["topk_w"].cpu()[plain].double()
    assert ((idx >= 0) & (idx < N) & (idx != 3)).all()
    assert (wgt - prob.gather(1, idx)).abs().max() < 1e-5
    assert (wgt - prob.topk(k, 1).values).abs().max() < 1e-5
    assert (r["c_expert"].sum().item(), r["c_expert"][3].item()) == (int((r["topk_idx"] >= 0).sum()), int((r["topk_idx"] == 3).sum()))
    # the same without the odd tokens: the masked expert has no share
    m = T.gate(x[torch.tensor([t for t in range(S) if t not in odd], device="cuda")].contiguous(), w, 1, k)["m"].cpu().double()
    assert m[3] == 0 and (m - prob.mean(0)).abs().max() < 1e-5


@pytest.mark.parametrize("S,N,d", [(100, 8, 64), (9000, 32, 264), (500, 64, 64), (9000, 64, 136), (20000, 64, 512), (500, 128, 64), (9000, 128, 72),
                                   (20000, 100, 128), (33000, 128, 136)])
def test_fp32_scores_of_the_largest_values(T, S, N, d):
    """Values whose rounding to 8 bits overflows (above (1 - 2^-8) * 2^128), and products and partial sums that do, in
    a few tokens: finite scores stay finite and right, sums beyond the range are infinite."""
    g = torch.Generator(device="cuda").manual_seed(S + d)
    x = torch.randn((S, d), generator=g, device="cuda")
    w = torch.randn((N, d), generator=g, device="cuda") / math.sqrt(d)
    big = torch.finfo(torch.float32).max
    w[:, 0], w[:, 1] = 2.0 ** -20 * w[:, 2], 2.0
    x[:, :2] = 0.0
    x[3, 0], x[S // 2, 0], x[S - 1, 0] = big, -big, big * 0.999
    x[5, 1], x[6, 1] = big, -big
    lg = T.gate(x, w, 1, 2)["logits"].cpu().double()
    ref = x.cpu().double() @ w.cpu().double().t()
    mag = x.cpu().double().abs() @ w.cpu().double().abs().t()
    over = ref.abs() > big
    assert over.sum() == 2 * N and torch.equal(torch.isfinite(lg), ~over) and torch.equal(lg[over].sign(), ref[over].sign())
    assert ((lg - ref).abs()[~over] <= ((d + 4) * 2.0 ** -24 * mag)[~over]).all()
