"""The fp32 matrix-instruction kernel against the oracle, every row, at the sizes where its tiling can go wrong:
token counts around the two tile heights (32 and 64), widths that are no multiple of a stage (32 columns) or of a
chunk (32 or 64 units), every count of score blocks per wave, one workgroup per token tile (r of one chunk: softmax
and top-k inside the kernel) and several (scores through the workspace).  Tolerance: 1e-5 of the row's score scale,
the bound of tests/parity.py for fp32 storage."""
import pytest

from test_gpu_predict import _run_and_check, _rand_layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,r,E,k,L,act,bias", [
    (1, 8, 8, 1, 1, 1, "none", False),
    (1, 2048, 256, 64, 6, 2, "none", True),
    (31, 264, 72, 130, 9, 2, "silu", True),                # small tile, remainders of d and r, 2 blocks per wave
    (32, 1000, 40, 1000, 32, 1, "gelu", True),             # small tile, 8 blocks per wave
    (32, 96, 32, 300, 7, 3, "none", False),                # small tile, one chunk: epilogue in the kernel
    (33, 264, 72, 64, 6, 2, "silu", True),                 # large tile, one row in its second block
    (65, 544, 200, 128, 8, 2, "gelu", True),               # 2 blocks per wave
    (130, 256, 64, 16, 2, 3, "none", True),                # one chunk: epilogue in the kernel
    (150, 72, 40, 256, 12, 2, "none", True),               # 4 blocks per wave
    (70, 520, 136, 1000, 32, 1, "silu", True),             # 16 blocks per wave
    (70, 40, 64, 1000, 17, 2, "none", False),              # ... and the epilogue in the kernel
    (8193, 32, 128, 40, 3, 4, "none", True),               # more tiles than workgroups wanted: two chunks per workgroup
])
def test_f32_kernel_edges(T, d, r, E, k, L, act, bias):
    x, W1, W2, b1, b2 = _rand_layers(900 + T + d, L=L, T=T, d=d, r=r, E=E, dtype="f32", bias=bias)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "f32", act=act, what=f"f32 T={T} d={d} r={r} E={E}")
    assert out.path == "simple"


def test_f32_shared_tokens_margin_and_counts():
    import torch
    import oracle
    from paper_2511_10676_amd import binding as B
    from test_gpu_predict import _dev
    x, W1, W2, b1, b2 = _rand_layers(77, L=3, T=45, d=320, r=136, E=48, dtype="f32", bias=True)
    counts = torch.zeros((3, 48), dtype=torch.int32, device="cuda")
    o = B.predict(_dev(x[:1], "f32"), _dev(W1, "f32"), _dev(W2, "f32"), 5, b1=_dev(b1, "f32"), b2=_dev(b2, "f32"),
                  want_logits=True, want_margin=True, counts=counts)
    torch.cuda.synchronize()
    z = o.logits.sort(dim=2, descending=True).values
    assert torch.equal(o.margin, z[:, :, 4] - z[:, :, 5])
    idx = o.idx.cpu().numpy()
    for l in range(3):
        ref = oracle.group_by_expert(idx[l], 48)[0]
        assert counts[l].cpu().numpy().tolist() == ref.tolist()


@pytest.mark.parametrize("T", [20, 100])
def test_f32_without_a_workspace_keeps_r_in_one_workgroup(T):
    """fp32 calls never needed a workspace: a missing one costs the split of r, not the call.  The two runs add the
    same products in another order: 1e-5 of the row's score scale, the bound for fp32 storage."""
    import torch
    from paper_2511_10676_amd import binding as B
    from test_gpu_predict import _dev
    x, W1, W2, _, _ = _rand_layers(5, L=2, T=T, d=264, r=520, E=64, dtype="f32", bias=False)
    args = _dev(x, "f32"), _dev(W1, "f32"), _dev(W2, "f32"), 6
    a = B.predict(*args, want_logits=True)
    b = B.predict(*args, want_logits=True, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    scale = a.logits.abs().amax(dim=2, keepdim=True)
    assert ((a.logits - b.logits).abs() <= 2e-5 * scale).all()
    assert torch.equal(b.idx.long(), torch.sort(b.logits, dim=2, descending=True, stable=True).indices[:, :, :6])


@pytest.mark.parametrize("L,T,d,r,E", [(1, 16, 2048, 2048, 64), (1, 512, 2048, 2048, 64), (4, 8192, 2048, 2048, 64),
                                       (2, 64, 256, 64, 16), (2, 300, 4096, 1024, 64), (1, 33, 768, 512, 8)])
def test_f32_scores_are_as_close_to_float64_as_a_lane_split_sum(L, T, d, r, E):
    """A dot product of n terms split over 64 lanes and added up by a butterfly rounds n / 64 times in a lane, on sums
    that grow towards their end (n / 128 full roundings in the variance), and 6 times between the lanes; a rounding errs
    by up to 2^-24 of the value, half of that as a standard deviation.  Both layers together:
    2^-25 * sqrt((d + r) / 128 + 12) of the scores' norm."""
    import torch
    from paper_2511_10676_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(d + T)
    x = torch.randn((L, T, d), device="cuda", generator=g)
    W1 = torch.randn((L, r, d), device="cuda", generator=g) / d ** 0.5
    W2 = torch.randn((L, E, r), device="cuda", generator=g) / r ** 0.5
    z = B.predict(x, W1, W2, min(6, E), want_logits=True).logits.double()
    exact = torch.stack([(x[l].double() @ W1[l].double().T) @ W2[l].double().T for l in range(L)])
    err = float((z - exact).norm() / exact.norm())
    print(f"f32 {L} x {T} x ({d}, {r}, {E}): {err:.2e}", flush=True)
    assert err <= 2.0 ** -25 * ((d + r) / 128 + 12) ** 0.5


@pytest.mark.parametrize("T,r", [(3, 40), (70, 40), (70, 200)])
def test_f32_infinite_token_does_not_meet_the_padding_of_r(T, r):
    """Positive weights and one token with an infinity: its scores are infinities, not NaN, although r is no multiple of
    a chunk; the other tokens' scores are what they are without it."""
    import torch
    from paper_2511_10676_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(T)
    x, W1, W2 = (torch.rand(s, device="cuda", generator=g) + 0.1 for s in ((1, T, 48), (1, r, 48), (1, 20, r)))
    plain = B.predict(x, W1, W2, 3, want_logits=True).logits
    x[0, 1, 7] = float("inf")
    z = B.predict(x, W1, W2, 3, want_logits=True).logits
    assert bool((z[0, 1] == float("inf")).all())
    keep = torch.arange(T, device="cuda") != 1
    assert torch.equal(z[0, keep], plain[0, keep])


@pytest.mark.parametrize("T,E,k", [(70, 16, 15), (70, 40, 16), (31, 17, 16), (33, 200, 1), (100, 64, 7)])
@pytest.mark.parametrize("prob", ["softmax", "softmax_topk", "sigmoid"])
def test_f32_rows_finished_in_the_kernel(T, E, k, prob):
    """One chunk of r, so softmax and top-k run there: lists of up to 16 keys (the margin needs one more) by several lanes per
    row, longer ones by a wave.  Against the definition in float64 on the kernel's own scores; probabilities to 2e-5 of their value,
    the bound of tests/parity.py for the same comparison."""
    import torch
    from paper_2511_10676_amd import binding as B
    from test_gpu_predict import _dev
    x, W1, W2, b1, b2 = _rand_layers(T + E, L=2, T=T, d=72, r=32, E=E, dtype="f32", bias=True)
    o = B.predict(_dev(x, "f32"), _dev(W1, "f32"), _dev(W2, "f32"), k, b1=_dev(b1, "f32"), b2=_dev(b2, "f32"), act="silu",
                  prob=prob, want_logits=True, want_margin=True)
    srt, order = torch.sort(o.logits, dim=2, descending=True, stable=True)
    assert torch.equal(o.idx.long(), order[:, :, :k])
    assert torch.equal(o.margin, srt[:, :, k - 1] - srt[:, :, k])
    z = srt.double()
    want = torch.sigmoid(z) if prob == "sigmoid" else torch.softmax(z[:, :, :k] if prob == "softmax_topk" else z, dim=2)
    want = want[:, :, :k]
    assert ((o.probs.double() - want).abs() <= 2e-5 * want).all()


@pytest.mark.parametrize("prob,bar", [("softmax", 6.2e-8), ("softmax_topk", 6.0e-8)])
def test_f32_probabilities_are_rounded_as_by_a_wave_per_row(prob, bar):
    """Eight of 256 probabilities of 16384 rows that are finished in the kernel, against float64 on the row's own scores, rms: a sum
    in pairs and a division, as a wave per row makes them, give 5.9e-8 (of all scores) and 5.3e-8 (of the selected ones); a product
    with the reciprocal has a rounding more, a sum of eight one after the other twice as many in a row, 6.5e-8 and 6.8e-8 (both seen;
    of 131072 values, so good to half a percent).  The bars stand between."""
    import torch
    from paper_2511_10676_amd import binding as B
    L, T, d, r, E, k = 4, 4096, 256, 64, 256, 8
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, W1, W2 = rnd(L, T, d), rnd(L, r, d) / d ** 0.5, rnd(L, E, r) / r ** 0.5
    o = B.predict(x, W1, W2, k, prob=prob, want_logits=True)
    srt = torch.sort(o.logits.double(), dim=2, descending=True).values
    want = torch.softmax(srt[:, :, :k] if prob == "softmax_topk" else srt, dim=2)[:, :, :k]
    assert float(((o.probs.double() - want) / want).square().mean().sqrt()) <= bar
