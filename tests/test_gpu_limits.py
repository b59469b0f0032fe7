"""Sizes beyond what the oracle can follow on the CPU: a token matrix of more than 2^32 16-byte
chunks (64 GiB), where the kernels' chunk indices need 64 bits.  Inputs are seeded and generated on
the device; the results are checked through properties that hold at any size (kept counts, the slot
permutation, token order inside an expert, bit-exact rows, the one-term combine), evaluated with
plain tensor operations on the device."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def T():
    if not torch.cuda.is_available():
        pytest.fail("these tests need a GPU")
    import paper_2302_09915_amd as T

    T.lib()
    return T


def test_more_than_2_to_32_chunks(T):
    dev = torch.device("cuda:0")
    if torch.cuda.mem_get_info()[0] < 215 * 2 ** 30:
        pytest.skip("needs 215 GiB of free device memory (three 64 GiB matrices)")
    print("64 GiB case: dispatch on given routing", flush=True)
    S, d, N, P, k = (1 << 21) + 3, 16384, 8, 8, 1
    assert S * d * 2 // 16 > 1 << 32
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    x = torch.empty((S, d), dtype=torch.bfloat16, device=dev)
    for s0 in range(0, S, 1 << 16):
        n = min(1 << 16, S - s0)
        x[s0:s0 + n] = torch.randn((n, d), generator=g, device=dev, dtype=torch.float32).to(torch.bfloat16)
    idx = torch.randint(0, N, (S, k), generator=g, device=dev, dtype=torch.int32)
    w = torch.rand((S, k), generator=g, device=dev, dtype=torch.float32) + 0.25
    cap = torch.full((N,), S, dtype=torch.int32, device=dev)
    cap[3] = 1000                                        # one expert drops most of its pairs
    ws = T.workspace(S, d, N, P, k, T.BF16, dev)
    send = torch.empty((S * k, d), dtype=torch.bfloat16, device=dev)
    slot = torch.empty((S, k), dtype=torch.int32, device=dev)
    kept = torch.empty((N,), dtype=torch.int32, device=dev)
    off = torch.empty((N + 1,), dtype=torch.int32, device=dev)
    scd = torch.empty((P,), dtype=torch.int32, device=dev)
    T.tamoe_dispatch(x, idx, cap, N, P, send, slot, kept, off, scd, ws, None)
    torch.cuda.synchronize()

    cnt = torch.bincount(idx.flatten().long(), minlength=N)
    exp_kept = torch.minimum(cnt, cap.long())
    assert torch.equal(kept.long(), exp_kept)
    assert torch.equal(off.long(), torch.cat([torch.zeros(1, dtype=torch.long, device=dev), exp_kept.cumsum(0)]))
    assert torch.equal(scd.long(), exp_kept)              # one expert per device
    K = int(off[-1].item())
    live = slot[:, 0] >= 0
    assert int(live.sum().item()) == K
    sl = slot[:, 0][live].long()
    assert int(sl.max().item()) == K - 1 and torch.unique(sl).numel() == K      # a permutation of 0..K-1
    for e in (0, 3, 7):                                   # token order inside an expert, drops at the end
        s_e = slot[:, 0][idx[:, 0] == e]
        n_e = int(exp_kept[e].item())
        assert bool((s_e[:n_e] >= 0).all()) and bool((s_e[n_e:] < 0).all())
        assert torch.equal(s_e[:n_e].long(), torch.arange(int(off[e].item()), int(off[e].item()) + n_e, device=dev))
    tok = torch.nonzero(live).flatten()
    bad = 0
    for s0 in range(0, tok.numel(), 1 << 14):             # every kept row arrived bit-exact
        t = tok[s0:s0 + (1 << 14)]
        bad += int((send[slot[t, 0].long()].view(torch.int16) != x[t].view(torch.int16)).any(dim=1).sum().item())
    assert bad == 0

    y = torch.empty((S, d), dtype=torch.bfloat16, device=dev)
    T.tamoe_combine(send, K, slot, w, y, None)
    torch.cuda.synchronize()
    bad = 0
    for s0 in range(0, S, 1 << 14):                       # k = 1: y = round(w * x), zero row for a dropped token
        n = min(1 << 14, S - s0)
        ref = (w[s0:s0 + n, :1] * x[s0:s0 + n].float()).to(torch.bfloat16)
        ref = torch.where(live[s0:s0 + n, None], ref, torch.zeros_like(ref))
        bad += int((ref.view(torch.int16) != y[s0:s0 + n].view(torch.int16)).any(dim=1).sum().item())
    assert bad == 0
    del y
    torch.cuda.empty_cache()

    # The gate and the fused call on the same 64 GiB matrix: tamoe_gate_dispatch must give the bits of
    # tamoe_gate + tamoe_dispatch (whose slot logic was checked above), and the gate's scores must agree
    # with a library matrix product on a sample of rows.
    print("64 GiB case: gate, then the fused call against the separate calls", flush=True)
    N2, k2 = 8, 2
    wg = (torch.randn((N2, d), generator=g, device=dev, dtype=torch.float32) / d ** 0.5).to(torch.bfloat16)
    cap2 = torch.full((N2,), S // 6, dtype=torch.int32, device=dev)      # below the mean load 2S/8: drops
    ws2 = T.workspace(S, d, N2, P, k2, T.BF16, dev)
    sep = T.gate(x, wg, P, k2, want_logits=True, ws=ws2)
    rows = torch.randint(0, S, (4096,), generator=g, device=dev)
    ref = x[rows].float() @ wg.float().t()
    assert (sep["logits"][rows] - ref).abs().max().item() <= 1e-3 * ref.abs().max().item()
    assert int(sep["c_expert"].sum().item()) == S * k2
    del send, sep
    torch.cuda.empty_cache()
    # rows of d/2 elements (the first half of every row of x) keep two send buffers of k = 2 within the
    # memory of the 64 GiB case; 8193 gate workgroups: the per-expert scans of the fused call run over
    # several pieces
    xh = x.view(S * 2, d // 2)[::2].contiguous()
    del x
    torch.cuda.empty_cache()
    wh = wg[:, : d // 2].contiguous()
    slot_a = torch.empty((S, k2), dtype=torch.int32, device=dev)
    kept_a, off_a, scd_a = torch.empty_like(kept), torch.empty_like(off), torch.empty_like(scd)
    send_a = torch.empty((S * k2, d // 2), dtype=torch.bfloat16, device=dev)
    sep = T.gate(xh, wh, P, k2, want_logits=False, ws=ws2)
    T.tamoe_dispatch(xh, sep["topk_idx"], cap2, N2, P, send_a, slot_a, kept_a, off_a, scd_a, ws2, None)
    pen = torch.full((N2,), 1.0 / N2, device=dev)
    fz = T.gate_dispatch(xh, wh, P, k2, pen, cap2, want_logits=False, ws=ws2)
    torch.cuda.synchronize()
    for name, a, b in (("topk_idx", sep["topk_idx"], fz["topk_idx"]), ("topk_w", sep["topk_w"], fz["topk_w"]),
                       ("c_expert", sep["c_expert"], fz["c_expert"]), ("slot", slot_a, fz["slot"]),
                       ("kept", kept_a, fz["kept_expert"]), ("off", off_a, fz["expert_offset"]),
                       ("scd", scd_a, fz["send_count_dev"])):
        assert torch.equal(a, b), name
    K2 = int(off_a[-1].item())
    assert 0 < K2 < S * k2                                                # capacity dropped some pairs
    bad = 0
    for r0 in range(0, K2, 1 << 15):
        r1 = min(K2, r0 + (1 << 15))
        bad += int((send_a[r0:r1].view(torch.int16) != fz["send"][r0:r1].view(torch.int16)).any(dim=1).sum().item())
    assert bad == 0
    del xh, send_a, fz
    torch.cuda.empty_cache()


def test_launches_of_2_to_32_threads(T):
    """Rows just over 1 KiB take two wavefronts each: 2^25 of them are 2^32 threads, more than a launch takes along
    one dimension.  Few rows are kept, so that the reference stays small."""
    dev = torch.device("cuda:0")
    S, d, N, P, k = (1 << 25) + 5, 520, 8, 4, 2
    row = d * 2
    if torch.cuda.mem_get_info()[0] < 5 * S * row:
        pytest.skip("needs 175 GB of free device memory")
    g = torch.Generator(device=dev)
    g.manual_seed(9)
    x = torch.empty((S, d), dtype=torch.bfloat16, device=dev)
    for s0 in range(0, S, 1 << 20):
        n = min(1 << 20, S - s0)
        x[s0:s0 + n] = torch.randn((n, d), generator=g, device=dev, dtype=torch.float32).to(torch.bfloat16)
    w = (torch.randn((N, d), generator=g, device=dev) / d ** 0.5).to(torch.bfloat16)
    cap = torch.full((N,), 1000, dtype=torch.int32, device=dev)
    f = T.gate_dispatch(x, w, P, k, None, cap, want_logits=False)
    torch.cuda.synchronize()
    K = N * 1000
    assert int(f["expert_offset"][-1]) == K and torch.equal(f["kept_expert"], cap)
    assert int(f["c_expert"].sum()) == S * k

    def check_slots(r):   # the first 1000 pairs of every expert, in the order of first choices, then second ones
        for e in range(N):
            t = torch.nonzero(r["topk_idx"][:, 0] == e).flatten()[:1000]
            assert torch.equal(r["slot"][t, 0], torch.arange(e * 1000, e * 1000 + 1000, dtype=torch.int32, device=dev))
            assert torch.equal(r["send"][e * 1000:e * 1000 + 1000].view(torch.int16), x[t].view(torch.int16))
        assert int((r["slot"] >= 0).sum()) == K

    check_slots(f)
    send = f.pop("send")
    f["send"] = send
    send[:K] = 0
    ws = T.workspace(S, d, N, P, k, T.BF16, dev)
    slot, kept = torch.empty_like(f["slot"]), torch.empty_like(f["kept_expert"])
    off, scd = torch.empty_like(f["expert_offset"]), torch.empty_like(f["send_count_dev"])
    T.tamoe_dispatch(x, f["topk_idx"], cap, N, P, send, slot, kept, off, scd, ws)
    torch.cuda.synchronize()
    assert torch.equal(slot, f["slot"])
    check_slots(f)
    # the last tokens too: y and the gradients of tokens with a kept pair, zeros elsewhere
    slot[(slot >= 0) & (slot < 3) | (slot == K - 1)] = -1
    slot[S - 3:] = torch.tensor([[0, 1], [2, -1], [-1, K - 1]], dtype=torch.int32, device=dev)
    recv = send[:K].clone()
    live = torch.nonzero((slot >= 0).any(1)).flatten()
    rows = recv[slot[live].clamp(min=0).long()].float() * (slot[live] >= 0)[..., None]
    wgt = f["topk_w"]
    y = send[:S]
    T.tamoe_combine(recv, K, slot, wgt, y)
    assert torch.allclose(y[live].float(), (rows * wgt[live][..., None]).sum(1), rtol=2.0 ** -7, atol=1e-6)
    y[live] = 0
    assert not any(bool(y[s0:s0 + (1 << 20)].any()) for s0 in range(0, S, 1 << 20))
    T.tamoe_dispatch_bwd(recv, K, slot, y)
    assert torch.allclose(y[live].float(), rows.sum(1), rtol=2.0 ** -7, atol=1e-6)
    y[live] = 0
    assert not any(bool(y[s0:s0 + (1 << 20)].any()) for s0 in range(0, S, 1 << 20))
    d_recv, d_w = torch.empty_like(recv), torch.full_like(wgt, 7.0)
    T.tamoe_combine_bwd(x, recv, K, slot, wgt, d_recv, d_w)
    dots = (rows * x[live].float()[:, None, :]).sum(2)
    assert torch.allclose(d_w[live], dots, rtol=1e-4, atol=1e-3)
    d_w[live] = 0
    assert not bool(d_w.any())
    t, j = torch.nonzero(slot >= 0, as_tuple=True)
    assert t.numel() == K
    want = wgt[t, j][:, None] * x[t].float()
    assert torch.allclose(d_recv[slot[t, j].long()].float(), want, rtol=2.0 ** -7, atol=1e-6)
    del d_w, slot, f, y
    torch.cuda.empty_cache()

    # two buffers of 2^26 rows
    rows_in, rows_out = send, torch.empty_like(send)
    rows_in[:K] = recv
    cnt = torch.randint(0, 2 * K // 64, (8, 4), generator=g, device=dev, dtype=torch.int32)
    R = int(cnt.sum())
    assert 0 < R <= K
    rows_out[:R + 5] = 3.0
    off = torch.empty(5, dtype=torch.int32, device=dev)
    T.tamoe_regroup(rows_in, cnt, True, rows_out, off, ws)
    torch.cuda.synchronize()
    c = cnt.cpu()
    src = torch.cat([torch.zeros(1, dtype=torch.long), c.flatten().cumsum(0)])
    order = torch.cat([torch.arange(int(src[s * 4 + e]), int(src[s * 4 + e + 1])) for e in range(4) for s in range(8)])
    assert torch.equal(off.cpu().long(), torch.cat([torch.zeros(1, dtype=torch.long), c.sum(0).cumsum(0)]))
    assert torch.equal(rows_out[:R].view(torch.int16), rows_in[order.to(dev)].view(torch.int16))
    assert bool((rows_out[R:R + 5] == 3.0).all())
