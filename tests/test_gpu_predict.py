"""GPU parity of paep_predict with the CPU oracle, through the C ABI.
Small cases span several tiles and ragged tails on every kernel family and are
checked on every row.  The paper-shaped cases run at full token count with as
many layers as it takes for the launcher to choose the tile configuration and
r split it chooses for the whole model (the choice is asserted through
paep_predict_plan), and are checked on seeded row samples -- on every row for
the DeepSeek-V2-Lite shape."""
import numpy as np
import pytest
import torch

from paper_2511_10676_amd import binding as B
from paper_2511_10676_amd import configs, datagen

import oracle
import parity

pytestmark = pytest.mark.gpu
ACT_ID = {"none": 0, "silu": 1, "gelu": 2}


def _dev(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype == "bf16":
        t = t.to(torch.bfloat16)
    return t.cuda()


def _rand_layers(seed, L, T, d, r, E, dtype, bias=False, outliers=True):
    g = np.random.default_rng(seed)
    x = g.standard_normal((L, T, d)).astype(np.float32)
    if outliers and d >= 8:
        x[:, :, g.choice(d, 4, replace=False)] *= 8
    W1 = (g.standard_normal((L, r, d)) / np.sqrt(d)).astype(np.float32)
    W2 = (g.standard_normal((L, E, r)) / np.sqrt(r)).astype(np.float32)
    b1 = (0.3 * g.standard_normal((L, r))).astype(np.float32) if bias else None
    b2 = (0.5 * g.standard_normal((L, E))).astype(np.float32) if bias else None
    rs = lambda a: None if a is None else datagen.round_to_storage(a, dtype)
    return rs(x), rs(W1), rs(W2), rs(b1), rs(b2)


def _run_and_check(x, W1, W2, b1, b2, k, dtype, act="none", path="auto", rows=None, what="", workspace=None):
    L = W1.shape[0]
    out = B.predict(_dev(x, dtype), _dev(W1, dtype), _dev(W2, dtype), k,
                    b1=None if b1 is None else _dev(b1, dtype), b2=None if b2 is None else _dev(b2, dtype),
                    act=act, path=path, want_logits=True, workspace=workspace)
    torch.cuda.synchronize()
    idx, probs, z = out.idx.cpu().numpy(), out.probs.cpu().numpy(), out.logits.cpu().numpy()
    tot, tot_m = parity.RowReport(), parity.RowReport()
    for l in range(L):
        xl = x[l] if x.shape[0] == L else x[0]
        rep, rep_m = parity.check_layer(xl, W1[l], W2[l], None if b1 is None else b1[l],
                                        None if b2 is None else b2[l], ACT_ID[act], k, dtype,
                                        idx[l], probs[l], z[l], rows=rows, what=f"{what} layer {l}")
        tot.add(rep)
        if rep_m:
            tot_m.add(rep_m)
    print(f"{what}: path={out.path} rows={tot.rows} strict={tot.strict} exempt={tot.exempt} "
          f"exempt_differ={tot.exempt_differ} max_err={tot.max_logit_err:.2e}*s_t prob_rel_err={tot.max_prob_rel_err:.2e} "
          f"(vs own scores {tot.max_prob_rel_err_own:.2e}, idx = rule(own scores) on {tot.own_topk_rows} rows) | "
          f"vs bf16-hidden oracle: strict={tot_m.strict} differ={tot_m.exempt_differ} "
          f"max_err={tot_m.max_logit_err:.2e}*s_t prob_rel_err={tot_m.max_prob_rel_err:.2e}", flush=True)
    assert tot.own_topk_rows == tot.rows
    return out, tot, tot_m


def _plan(T, d, r, E, k, L):
    return B.predict_plan(B.make_desc(T, d, r, E, k, L, B.BF16))


# ------------------------------------------------------------------ toy / simple path
def test_toy_fp32_all_rows():
    w = configs.get("toy")
    lay = datagen.make_layer(w, 0, w.prefill_T[0])
    out, tot, _ = _run_and_check(lay.x[None], lay.W1[None], lay.W2[None], None, None, w.k, "f32", what="toy")
    assert out.path == "simple"
    assert tot.exempt_differ == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("act", ["none", "silu", "gelu"])
def test_simple_path_odd_shapes(dtype, act):
    x, W1, W2, b1, b2 = _rand_layers(1, L=2, T=37, d=72, r=40, E=13, dtype=dtype, bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, 5, dtype, act=act, path="simple", what=f"simple {dtype} {act}")
    assert out.path == "simple"


def test_simple_path_large_k_and_E():
    x, W1, W2, b1, b2 = _rand_layers(2, L=1, T=9, d=64, r=128, E=1000, dtype="f32")
    _run_and_check(x, W1, W2, None, None, 32, "f32", path="simple", what="simple E=1000 k=32")
    _run_and_check(x[:, :, :], W1, W2[:, :7], None, None, 7, "f32", path="simple", what="simple k=E=7")


# ------------------------------------------------------------------ decode path
@pytest.mark.parametrize("T", [1, 5, 16, 17, 33, 64])
def test_decode_path_small(T):
    x, W1, W2, b1, b2 = _rand_layers(10 + T, L=3, T=T, d=512, r=192, E=48, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, 6, "bf16", path="decode", what=f"decode T={T}")
    assert out.path == "decode"


@pytest.mark.parametrize("E,k,act", [(40, 8, "none"), (16, 2, "silu"), (250, 12, "gelu"), (8, 8, "none")])
def test_decode_path_ragged_experts(E, k, act):
    x, W1, W2, b1, b2 = _rand_layers(30 + E, L=2, T=7, d=256, r=128, E=E, dtype="bf16", bias=True)
    _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, path="decode", what=f"decode E={E} k={k} {act}")


@pytest.mark.parametrize("T,d,r,E,k,act,L", [
    # r in whole slices of 128: a workgroup takes 128 hidden units, its waves split the rows and share the tokens
    # through a ring of LDS stages of 128 columns (otherwise: slices of 64, waves split d, covered by the cases
    # above).  The ring has three stages in calls of fewer than 384 slices (the cases with 3 layers) and two
    # beyond (the first two cases); d = 128 is a single stage, d = 384 and 640 a ragged last round, 250 experts
    # give a wave two expert blocks; up to 32 tokens a stage holds 32 token rows, beyond that 64
    (1, 256, 1024, 48, 6, "none", 48), (16, 384, 512, 48, 6, "gelu", 96), (17, 384, 256, 48, 6, "none", 3),
    (32, 640, 128, 48, 6, "silu", 3), (33, 384, 256, 250, 12, "gelu", 3), (48, 1024, 384, 64, 6, "none", 3),
    (64, 640, 256, 48, 8, "none", 3), (64, 128, 128, 16, 2, "silu", 3),
])
def test_decode_row_split_kernel(T, d, r, E, k, act, L):
    x, W1, W2, b1, b2 = _rand_layers(70 + T + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, path="decode", what=f"decode rows T={T} d={d} r={r} E={E}")
    assert out.path == "decode"


def test_decode_shared_tokens_across_layers():
    x, W1, W2, _, _ = _rand_layers(50, L=4, T=3, d=256, r=64, E=32, dtype="bf16")
    _run_and_check(x[:1], W1, W2, None, None, 4, "bf16", path="decode", what="decode shared x")
    # the same through the row-split kernel (r = 256), no biases, both token-block sizes
    for T in (20, 50):
        x, W1, W2, _, _ = _rand_layers(52 + T, L=4, T=T, d=256, r=256, E=32, dtype="bf16")
        _run_and_check(x[:1], W1, W2, None, None, 4, "bf16", path="decode", what=f"decode rows shared x T={T}")


# Few hidden units in all (L * r <= 4096, or 8192 up to 16 tokens, r a multiple of 128) and d long enough: slices of 16 or
# 32 units, the stages of 128 columns dealt to eight waves.  Fewer stages than waves, ragged shares, two, four and six
# stages a wave, token counts around a block of 16, expert counts around a block of 16 and 8 blocks, both slice widths.
@pytest.mark.parametrize("T,d,r,E,k,act,L", [
    (1, 512, 128, 1, 1, "none", 1), (16, 640, 128, 16, 3, "silu", 4), (17, 1152, 256, 17, 4, "none", 2),
    (32, 2048, 256, 128, 8, "gelu", 1), (33, 2048, 128, 120, 6, "none", 2), (64, 1664, 384, 64, 16, "silu", 2),
    (1, 5120, 128, 64, 6, "none", 1), (31, 4096, 128, 64, 6, "none", 1), (9, 2176, 128, 33, 6, "none", 2),
    (1, 2176, 128, 129, 5, "none", 3), (16, 4096, 128, 255, 32, "silu", 1), (15, 1152, 2048, 64, 6, "none", 3),
    (2, 2304, 1152, 250, 9, "gelu", 2), (16, 1536, 8192, 16, 2, "none", 1), (1, 1920, 4096, 16, 2, "none", 1),
])
def test_decode_thin_slices(T, d, r, E, k, act, L):
    desc = B.make_desc(T, d, r, E, k, L, B.BF16)
    units = 16 if E <= 128 and L * r <= 4096 else 32
    assert B.predict_workspace_bytes(desc) == 4 * L * (r // units) * T * E             # thin slices are chosen
    x, W1, W2, b1, b2 = _rand_layers(400 + T + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, path="decode", what=f"decode thin T={T} d={d} r={r} E={E}")
    assert out.path == "decode"


# The other two kernels, in calls with more hidden units than those: r in slices of 128 and r in slices of 64.
@pytest.mark.parametrize("T,d,r,E,k,L", [
    (1, 128, 128, 64, 6, 65), (33, 256, 256, 130, 5, 33), (64, 128, 128, 16, 2, 66),
    (1, 128, 192, 64, 6, 43), (16, 256, 64, 17, 3, 129), (33, 128, 320, 40, 4, 26), (64, 384, 192, 64, 6, 43),
])
def test_decode_many_layers(T, d, r, E, k, L):
    x, W1, W2, b1, b2 = _rand_layers(500 + T + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", path="decode", what=f"decode T={T} d={d} r={r} E={E} L={L}")
    assert out.path == "decode"


@pytest.mark.parametrize("L,r,E", [(1, 2048, 64), (2, 2048, 128), (4, 2048, 64), (2, 4096, 256), (1, 192, 130)])
@pytest.mark.parametrize("d", [2048, 4096])
def test_decode_workspace_for_more_tokens_serves_fewer(L, r, E, d):
    sizes = [B.predict_workspace_bytes(B.make_desc(T, d, r, E, 1, L, B.BF16)) for T in range(1, 65)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("L,T,d,r,E,act", [(2, 64, 1536, 2048, 64, "none"), (1, 1, 2048, 1024, 128, "silu"),
                                           (4, 16, 2048, 2048, 200, "gelu"), (1, 33, 1664, 128, 60, "none")])
def test_decode_runs_in_the_scores_of_64_wide_slices(L, T, d, r, E, act):
    """The workspace that every decode call can do with: L * (r / 64) * T * E floats, never more for fewer layers.  Thin
    slices want more and are left out then: the same hidden vector to the bit, the scores in wider slices (2e-6 of the
    row's scale: r products of 2^-24 each, as a random walk, four times over).  One byte less is refused."""
    x, W1, W2, b1, b2 = _rand_layers(450 + T, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    args = _dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), 5
    opts = dict(b1=_dev(b1, "bf16"), b2=_dev(b2, "bf16"), act=act, want_logits=True, path="decode")
    need = 4 * L * (r // 64) * T * E
    assert B.predict_workspace_bytes(B.make_desc(T, d, r, E, 5, L, B.BF16)) > need
    best = B.predict(*args, **opts)
    least = B.predict(*args, workspace=torch.empty(need, dtype=torch.uint8, device="cuda"), **opts)
    torch.cuda.synchronize()
    scale = best.logits.abs().amax(dim=2, keepdim=True)
    assert ((best.logits - least.logits).abs() <= 2e-6 * scale).all()
    assert torch.equal(least.idx.long(), torch.sort(least.logits, dim=2, descending=True, stable=True).indices[:, :, :5])
    with pytest.raises(B.PaepError, match="WORKSPACE"):
        B.predict(*args, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"), **opts)


def test_decode_row_split_many_experts_and_wide_k():
    # 512 experts (eight per lane in the finalize kernel, four expert blocks per wave in the slices kernel) and k = 32
    x, W1, W2, b1, b2 = _rand_layers(57, L=2, T=40, d=256, r=256, E=512, dtype="bf16", bias=True)
    _run_and_check(x, W1, W2, b1, b2, 32, "bf16", act="silu", path="decode", what="decode rows E=512 k=32")
    x, W1, W2, b1, b2 = _rand_layers(58, L=2, T=9, d=128, r=128, E=130, dtype="bf16", bias=True)
    _run_and_check(x, W1, W2, b1, b2, 16, "bf16", path="decode", what="decode rows E=130 k=16")


# ------------------------------------------------------------------ prefill path
def test_prefill_shared_tokens_across_layers():
    x, W1, W2, _, _ = _rand_layers(51, L=5, T=333, d=256, r=256, E=48, dtype="bf16")
    _run_and_check(x[:1], W1, W2, None, None, 6, "bf16", path="prefill", what="prefill shared x")


@pytest.mark.parametrize("T", [1, 127, 128, 300])
def test_prefill_path_small(T):
    x, W1, W2, b1, b2 = _rand_layers(60 + T, L=2, T=T, d=256, r=256, E=64, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, 6, "bf16", path="prefill", what=f"prefill T={T}")
    assert out.path == "prefill"


@pytest.mark.parametrize("E,k,act", [(16, 2, "none"), (40, 8, "silu"), (128, 8, "none"), (256, 12, "gelu"), (200, 16, "none")])
def test_prefill_path_expert_counts(E, k, act):
    x, W1, W2, b1, b2 = _rand_layers(80 + E, L=2, T=150, d=128, r=384, E=E, dtype="bf16", bias=(act != "none"))
    _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, path="prefill", what=f"prefill E={E} k={k} {act}")


def test_duplicate_w2_rows_tie_to_lower_id_on_every_path():
    for path, T in (("simple", 40), ("decode", 40), ("prefill", 200)):
        x, W1, W2, _, _ = _rand_layers(90, L=1, T=T, d=256, r=128, E=32, dtype="bf16")
        W2[0, 20] = W2[0, 3]
        out, tot, tot_m = _run_and_check(x, W1, W2, None, None, 6, "bf16", path=path, what=f"ties {path}")
        idx = out.idx.cpu().numpy()[0]
        z = out.logits.cpu().numpy()[0]
        assert np.array_equal(z[:, 3], z[:, 20])
        both = 0
        for row in idx.tolist():
            assert not (20 in row and 3 not in row)
            if 3 in row and 20 in row:
                both += 1
                assert row.index(20) == row.index(3) + 1
        assert both > 0


def test_results_are_reproducible_bit_for_bit():
    for path, T in (("decode", 33), ("prefill", 260), ("simple", 20)):
        x, W1, W2, _, _ = _rand_layers(95, L=2, T=T, d=256, r=128, E=64, dtype="bf16")
        xs, a, b = _dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16")
        outs = []
        for _ in range(3):
            o = B.predict(xs, a, b, 6, path=path, want_logits=True)
            torch.cuda.synchronize()
            outs.append((o.idx.cpu().numpy().tobytes(), o.probs.cpu().numpy().tobytes(), o.logits.cpu().numpy().tobytes()))
        assert outs[0] == outs[1] == outs[2], path


def test_empty_call():
    x, W1, W2, _, _ = _rand_layers(96, L=2, T=0, d=256, r=128, E=64, dtype="bf16")
    o = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), 6)
    assert o.idx.shape == (2, 0, 6)


@pytest.mark.parametrize("E,k,r,d,L,T", [
    (64, 6, 256, 64, 4, 8229), (128, 8, 128, 64, 4, 8229), (256, 8, 384, 64, 4, 8229), (24, 2, 512, 64, 4, 8229),
    # d = 4096: the token tile is large enough that r is split over two workgroups per tile
    # (score tiles through the workspace, added by the finalize kernels); so it is, further, in
    # every case here with fewer than 256 tiles
    (64, 6, 512, 4096, 4, 8300), (200, 8, 256, 4096, 4, 8300),
    # several chunks of r per tile, many layers, a single layer with many tiles
    (64, 6, 768, 64, 4, 8229), (64, 6, 1024, 64, 16, 8229), (128, 8, 640, 64, 9, 8229), (16, 2, 1280, 32, 1, 33000),
    # 64 < E <= 128 with r a multiple of 256: the 256 x 256 tile with the waves side by side
    (128, 8, 512, 64, 4, 8229), (100, 8, 256, 128, 4, 8229),
    # more than 64 experts with d = 96 and d = 32: three tiles and one tile per chunk of r, so the W2 slice in
    # LDS has to be waited for explicitly before each second product
    (128, 8, 256, 96, 4, 8229), (200, 8, 256, 32, 4, 8229),
])
def test_prefill_large_tile_configs_with_ragged_tail(E, k, r, d, L, T):
    """Enough tokens that the large-tile kernels are chosen, a token count that
    is not a multiple of any tile, every row checked; with the least workspace, so that
    the fused kernel runs where two passes would."""
    x, W1, W2, b1, b2 = _rand_layers(70 + E, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    least = B.predict_workspace_min_bytes(B.make_desc(T, d, r, E, k, L, B.BF16, path="prefill"))
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", path="prefill", what=f"prefill large tiles E={E} r={r} d={d}",
                             workspace=torch.empty(max(least, 16), dtype=torch.uint8, device="cuda"))
    assert out.path == "prefill"


@pytest.mark.parametrize("E,k,r,d,L,T,tile,groups,cpg", [
    # at least 256 token tiles: every workgroup walks all of r by itself, several chunks of it --
    # the configuration a whole model's worth of layers runs in
    (64, 6, 1024, 64, 8, 8229, "256x256", 1, 4),
    (128, 8, 1024, 64, 8, 8229, "256x256 wide", 1, 4),
    (256, 8, 512, 64, 8, 8229, "256x128", 1, 4),
    (200, 12, 640, 128, 8, 8229, "256x128", 1, 5),
    # 9 layers x 33 tiles = 256 + 41: the 41 tiles beyond the full round are cut along r into four pieces each
    # that meet in the workspace, the other 256 are not (same kernel, two parts of one grid)
    (64, 6, 1024, 64, 9, 8229, "256x256", 1, 4),
    (128, 8, 1024, 64, 9, 8229, "256x256 wide", 1, 4),
    (256, 8, 512, 64, 9, 8229, "256x128", 1, 4),
    # ... and with long rows (d = 4096) r split over two workgroups per tile, again at >= 256 tiles:
    # score tiles through the workspace, added by the finalize kernels
    (64, 6, 512, 4096, 8, 8300, "256x256", 2, 1),
])
def test_prefill_many_tiles_every_row(E, k, r, d, L, T, tile, groups, cpg):
    plan = _plan(T, d, r, E, k, L)
    assert (plan.path, plan.tile, plan.groups, plan.chunks_per_group) == ("prefill", tile, groups, cpg), plan
    x, W1, W2, b1, b2 = _rand_layers(170 + E + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", what=f"prefill many tiles E={E} r={r} d={d} {plan}")
    assert out.path == "prefill"


# ------------------------------------------------------------------ paper-shaped, full size, sampled rows
def _paper_shaped(name, T, layers, n_rows, path):
    w = configs.get(name)
    L = len(layers)
    lays = [datagen.make_layer(w, l, T) for l in layers]
    x = np.stack([a.x for a in lays]); W1 = np.stack([a.W1 for a in lays]); W2 = np.stack([a.W2 for a in lays])
    b2 = np.stack([a.b2 for a in lays]) if lays[0].b2 is not None else None
    rows = None
    if n_rows < T:
        g = np.random.default_rng(1234 + T)
        rows = np.sort(np.concatenate([g.choice(T, n_rows - 2, replace=False), [0, T - 1]]))
        for a in lays:
            if a.tie_rows.size:
                rows = np.union1d(rows, a.tie_rows[:32])
    out, tot, tot_m = _run_and_check(x, W1, W2, None, b2, w.k, w.dtype, rows=rows, what=f"{name} T={T} L={L}")
    assert out.path == path
    return out, tot, tot_m, lays


@pytest.mark.parametrize("T", [1, 8, 64])
def test_deepseek_shaped_decode_all_layers(T):
    _paper_shaped("deepseek_v2_lite", T, range(26), T, "decode")


def test_deepseek_shaped_prefill_all_layers_every_row():
    w = configs.get("deepseek_v2_lite")
    plan = _plan(4096, w.d, w.r, w.E, w.k, w.L)
    assert (plan.tile, plan.groups, plan.chunks_per_group) == ("256x256", 1, 8), plan
    out, tot, tot_m, _ = _paper_shaped("deepseek_v2_lite", 4096, range(26), 4096, "prefill")
    assert tot.rows == 26 * 4096


@pytest.mark.parametrize("T", [1, 16, 64])
def test_qwen3_shaped_decode(T):
    _paper_shaped("qwen3_30b_a3b", T, range(0, 48, 6), T, "decode")


def test_qwen3_shaped_prefill_sampled():
    """Eight layers: 256 token tiles, which makes the launcher choose what it chooses for all 48."""
    w = configs.get("qwen3_30b_a3b")
    layers = [0, 6, 13, 17, 24, 30, 41, 47]
    full, part = _plan(8192, w.d, w.r, w.E, w.k, w.L), _plan(8192, w.d, w.r, w.E, w.k, len(layers))
    assert full == part and (part.tile, part.groups, part.chunks_per_group) == ("256x256 wide", 1, 8), (full, part)
    _paper_shaped("qwen3_30b_a3b", 8192, layers, 48, "prefill")


@pytest.mark.parametrize("T", [1, 32])
def test_phi_shaped_decode(T):
    _paper_shaped("phi_mini_moe", T, range(0, 32, 4), T, "decode")


def test_phi_shaped_prefill_sampled():
    w = configs.get("phi_mini_moe")
    layers = [0, 4, 9, 13, 20, 24, 27, 31]
    full, part = _plan(8192, w.d, w.r, w.E, w.k, w.L), _plan(8192, w.d, w.r, w.E, w.k, len(layers))
    assert full == part and part.groups == 2, (full, part)
    _paper_shaped("phi_mini_moe", 8192, layers, 32, "prefill")


def test_stress_shaped_prefill_sampled_with_near_ties():
    """Two layers of 32768 tokens: 256 token tiles, the launcher's choice for all 48 layers."""
    w = configs.get("stress")
    full, part = _plan(32768, w.d, w.r, w.E, w.k, w.L), _plan(32768, w.d, w.r, w.E, w.k, 2)
    assert full == part and (part.tile, part.groups, part.chunks_per_group) == ("two-pass 256x256", 4, 4), (full, part)
    out, tot, tot_m, lays = _paper_shaped("stress", 32768, [0, 47], 64, "prefill")
    assert lays[0].tie_rows.size == 328
    # the planted rows sit inside the tolerance band; they must still be valid selections
    assert tot.exempt > 0


# ------------------------------------------------------------------ properties of the whole output at full size
def _check_output_properties(out, E, k):
    """What must hold for every row at any size: ids in range and distinct, probabilities positive,
    descending, and no more than the whole softmax mass."""
    idx, probs = out.idx, out.probs
    assert bool(((idx >= 0) & (idx < E)).all())
    srt = torch.sort(idx, dim=-1).values
    assert bool((srt[..., 1:] != srt[..., :-1]).all()), "an expert selected twice in one row"
    assert bool((probs > 0).all()) and bool(torch.isfinite(probs).all())
    assert bool((probs[..., :-1] >= probs[..., 1:]).all()), "probabilities not in descending order"
    assert float(probs.sum(dim=-1).max()) <= 1.0 + 1e-5


@pytest.mark.parametrize("name,T", [("deepseek_v2_lite", 4096), ("deepseek_v2_lite", 64), ("qwen3_30b_a3b", 8192),
                                    ("phi_mini_moe", 8192), ("stress", 32768)])
def test_full_size_outputs_have_the_required_properties_and_feed_grouping(name, T):
    """All layers, the benchmark's launch configuration, random weights generated on the device; every row of the
    output is checked for the properties above, and grouping/scoring of it for their conservation laws."""
    w = configs.get(name)
    g = torch.Generator(device="cuda"); g.manual_seed(7)
    x = torch.randn((w.L, T, w.d), device="cuda", generator=g).to(torch.bfloat16)
    W1 = (torch.randn((w.L, w.r, w.d), device="cuda", generator=g) / w.d ** 0.5).to(torch.bfloat16)
    W2 = (torch.randn((w.L, w.E, w.r), device="cuda", generator=g) / w.r ** 0.5).to(torch.bfloat16)
    out = B.predict(x, W1, W2, w.k)
    torch.cuda.synchronize()
    _check_output_properties(out, w.E, w.k)
    grp = B.group_by_expert(out.idx, w.E)
    sc = B.score(out.idx, out.idx, w.E)
    torch.cuda.synchronize()
    assert bool((grp.counts.sum(dim=1) == T * w.k).all()) and bool((grp.offsets[:, -1] == T * w.k).all())
    assert bool((grp.n_invalid == 0).all())
    # every position appears exactly once in a layer's token lists
    pos = torch.sort(grp.token_pos, dim=1).values
    assert bool((pos == torch.arange(T * w.k, device="cuda", dtype=torch.int32)[None, :]).all())
    # a prediction scored against itself: every row exact, every expert a hit
    assert sc.cpu().tolist() == [[T, T * w.k, T, T]] * w.L


# ------------------------------------------------------------------ the smallest shapes each kernel family accepts
@pytest.mark.parametrize("path,T,d,r,E,k,L", [
    ("prefill", 1, 32, 128, 1, 1, 1), ("prefill", 3, 32, 128, 2, 2, 3), ("prefill", 129, 64, 256, 5, 5, 1),
    ("prefill", 257, 32, 128, 33, 16, 2), ("decode", 1, 128, 64, 1, 1, 1), ("decode", 64, 128, 64, 3, 2, 2),
    ("decode", 2, 128, 128, 512, 32, 1), ("simple", 1, 8, 8, 1, 1, 1), ("simple", 2, 16, 8, 3, 3, 2),
])
def test_smallest_shapes(path, T, d, r, E, k, L):
    x, W1, W2, b1, b2 = _rand_layers(500 + T + E, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True, outliers=False)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", path=path, what=f"smallest {path} T={T} d={d} r={r} E={E}")
    assert out.path == path


# ------------------------------------------------------------------ activation counts from the predictor's epilogue
@pytest.mark.parametrize("path,T,d,r,E,k,L,dtype", [
    ("simple", 37, 72, 40, 13, 5, 2, "f32"), ("decode", 7, 256, 128, 40, 8, 3, "bf16"),
    ("decode", 64, 256, 128, 250, 12, 2, "bf16"), ("prefill", 300, 128, 384, 64, 6, 2, "bf16"),
    ("prefill", 700, 128, 256, 200, 16, 3, "bf16"), ("prefill", 8300, 64, 512, 64, 6, 4, "bf16"),
])
def test_counted_predict_adds_the_histogram_of_its_selections(path, T, d, r, E, k, L, dtype):
    x, W1, W2, _, _ = _rand_layers(900 + T, L=L, T=T, d=d, r=r, E=E, dtype=dtype)
    xs, a, b = _dev(x, dtype), _dev(W1, dtype), _dev(W2, dtype)
    plain = B.predict(xs, a, b, k, path=path)
    counts = torch.full((L, E), 3, dtype=torch.int32, device="cuda")          # not zero: the call adds
    out = B.predict(xs, a, b, k, path=path, counts=counts)
    out2 = B.predict(xs, a, b, k, path=path, counts=counts)                   # accumulates over calls
    torch.cuda.synchronize()
    assert out.path == path
    assert torch.equal(out.idx, plain.idx) and torch.equal(out.probs, plain.probs) and torch.equal(out2.idx, plain.idx)
    for l in range(L):
        hist = torch.bincount(out.idx[l].flatten().to(torch.int64), minlength=E).to(torch.int32)
        assert torch.equal(counts[l], 3 + 2 * hist), f"layer {l}"
    # against the oracle: its own selection on the rows where the selection is unambiguous (strict rows:
    # every gap among its top k+1 scores above the tolerance; in fp32 that is every row), the kernel's
    # selection on the others (those rows are checked for validity by the parity tests)
    tol = parity.TOL_MODEL if dtype == "bf16" else parity.TOL["f32"]
    n_strict = 0
    for l in range(L):
        idx_o, _, z_o = oracle.predict(x[l], W1[l], W2[l], k, round_h=(dtype == "bf16"))
        zs = -np.sort(-z_o, axis=1)
        s_t = np.abs(z_o).max(axis=1)
        strict = (zs[:, :min(k, E - 1)] - zs[:, 1:min(k, E - 1) + 1] >= tol * s_t[:, None]).all(axis=1)
        n_strict += int(strict.sum())
        mixed = np.where(strict[:, None], idx_o, out.idx[l].cpu().numpy())
        want = oracle.group_by_expert(mixed, E)[0]
        assert np.array_equal((counts[l].cpu().numpy() - 3) // 2, want), f"layer {l}"
    assert n_strict > 0.1 * L * T                 # the oracle's own selection decides a good share of the rows


# ------------------------------------------------------------------ confidence outputs (sections 6 and 4.4)
@pytest.mark.parametrize("path,T,d,r,E,k,L,dtype", [
    ("simple", 37, 72, 40, 13, 5, 2, "f32"), ("simple", 9, 64, 128, 40, 32, 1, "f32"),
    ("decode", 7, 256, 128, 40, 8, 3, "bf16"), ("decode", 64, 256, 128, 250, 12, 2, "bf16"),
    ("prefill", 300, 128, 384, 64, 6, 2, "bf16"), ("prefill", 700, 128, 256, 200, 15, 3, "bf16"),
    ("prefill", 8300, 64, 512, 128, 8, 4, "bf16"), ("prefill", 150, 128, 128, 8, 8, 1, "bf16"),
])
def test_confidence_outputs_match_the_oracle(path, T, d, r, E, k, L, dtype):
    x, W1, W2, _, _ = _rand_layers(1300 + T + k, L=L, T=T, d=d, r=r, E=E, dtype=dtype)
    xs, a, b = _dev(x, dtype), _dev(W1, dtype), _dev(W2, dtype)
    base = B.predict(xs, a, b, k, path=path, want_logits=True)
    outs = {m: B.predict(xs, a, b, k, path=path, prob=m, want_margin=True) for m in ("softmax", "softmax_topk", "sigmoid")}
    torch.cuda.synchronize()
    tol = parity.TOL["bf16" if dtype == "bf16" else "f32"]
    for m, o in outs.items():
        assert o.path == path, (m, o.path)
        assert torch.equal(o.idx, base.idx), m                    # all three scores are monotone: same selection
        assert torch.equal(o.margin, outs["softmax"].margin)
    assert torch.equal(outs["softmax"].probs, base.probs)
    zg = base.logits.cpu().numpy()
    idx = base.idx.cpu().numpy()
    for l in range(L):
        # (a) sharp, against the kernel's own scores: definitions evaluated in float64 on what it selected from
        soft_o, sig_o, margin_o = oracle.confidence_outputs(zg[l].astype(np.float64), idx[l])
        for name, want in (("softmax_topk", soft_o), ("sigmoid", sig_o)):
            got = outs[name].probs[l].cpu().numpy().astype(np.float64)
            assert np.abs(got - want).max() <= parity.PROB_TOL_OWN * np.abs(want).max() + 1e-30, (name, l)
            assert (np.abs(got - want) <= parity.PROB_TOL_OWN * want + 1e-12).all(), (name, l)
        mg = outs["softmax"].margin[l].cpu().numpy()
        if k < E:
            own = -np.sort(-zg[l], axis=1)
            assert np.array_equal(mg, own[:, k - 1] - own[:, k]), f"margin layer {l}"      # one fp32 subtraction
        else:
            assert np.isinf(mg).all() and (mg > 0).all()
        # (b) against the oracle's own scores, within what the score tolerance allows
        idx_r, _, z_r = oracle.predict(x[l], W1[l], W2[l], k)
        _, _, margin_r = oracle.confidence_outputs(z_r, idx_r)
        delta = tol * np.abs(z_r).max(axis=1)
        if k < E:
            assert (np.abs(mg - margin_r) <= 2 * delta + 1e-6).all(), f"margin vs oracle, layer {l}"
        soft_r, sig_r, _ = oracle.confidence_outputs(z_r, idx[l])          # the oracle's scores at the kernel's selection
        got = outs["softmax_topk"].probs[l].cpu().numpy()
        assert (np.abs(got - soft_r) <= (np.expm1(2 * delta)[:, None] + 2e-5) * soft_r + 1e-30).all()
        got = outs["sigmoid"].probs[l].cpu().numpy()
        assert (np.abs(got - sig_r) <= (np.expm1(delta)[:, None] + 2e-5) * sig_r + 1e-30).all()
    assert np.allclose(outs["softmax_topk"].probs.sum(dim=-1).cpu().numpy(), 1.0, atol=1e-5)


def test_margin_on_the_prefill_path_needs_room_for_one_more_candidate():
    x, W1, W2, _, _ = _rand_layers(1400, L=1, T=200, d=128, r=128, E=64, dtype="bf16")
    xs, a, b = _dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16")
    with pytest.raises(B.PaepError) as e:
        B.predict(xs, a, b, 16, path="prefill", want_margin=True)
    assert e.value.status == 8                                          # PAEP_ERR_UNSUPPORTED
    o = B.predict(xs, a, b, 16, want_margin=True, want_logits=True)      # AUTO falls back to a family that can
    torch.cuda.synchronize()
    assert o.path == "simple"
    own = -np.sort(-o.logits[0].cpu().numpy(), axis=1)
    assert np.array_equal(o.margin[0].cpu().numpy(), own[:, 15] - own[:, 16])


# ------------------------------------------------------------------ BatchNorm folded into the first layer (section 4.3)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_fold_batchnorm_matches_the_oracle_and_feeds_predict(dtype):
    g = np.random.default_rng(77)
    L, T, d, r, E, k = 2, 50, 72, 40, 13, 5
    x, W1, W2, b1, _ = _rand_layers(78, L=L, T=T, d=d, r=r, E=E, dtype=dtype, bias=True)
    gamma = (1 + 0.3 * g.standard_normal((L, r))).astype(np.float32)
    beta = (0.2 * g.standard_normal((L, r))).astype(np.float32)
    mean = (0.5 * g.standard_normal((L, r))).astype(np.float32)
    var = (0.5 + g.random((L, r))).astype(np.float32)
    f32 = lambda v: torch.from_numpy(v).cuda()
    W1f, b1f = B.fold_batchnorm(_dev(W1, dtype), _dev(b1, dtype), f32(gamma), f32(beta), f32(mean), f32(var), 1e-5)
    W1n, _ = B.fold_batchnorm(_dev(W1, dtype), None, f32(gamma), f32(beta), f32(mean), f32(var), 1e-5)
    torch.cuda.synchronize()
    assert torch.equal(W1n, W1f)
    ulp = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -22                   # one rounding to storage + fp32 arithmetic
    for l in range(L):
        Wo, bo = oracle.fold_batchnorm(W1[l], b1[l], gamma[l], beta[l], mean[l], var[l], 1e-5)
        assert (np.abs(W1f[l].float().cpu().numpy() - Wo) <= ulp * np.abs(Wo) + 1e-30).all()
        assert (np.abs(b1f[l].float().cpu().numpy() - bo) <= ulp * np.abs(bo) + 1e-6).all()
    # Architecture 1 end to end: folded weights + exact GELU through the predictor, against the oracle on the same weights
    Wh, bh = W1f.float().cpu().numpy(), b1f.float().cpu().numpy()
    _run_and_check(x, Wh, W2, bh, None, k, dtype, act="gelu", path="simple", what=f"arch-1 folded {dtype}")


@pytest.mark.parametrize("E,k,margin", [(4, 4, True), (12, 2, False), (16, 7, True), (20, 16, False), (64, 8, False),
                                        (64, 15, True), (100, 8, True), (128, 1, True), (132, 12, False), (256, 8, True),
                                        (130, 6, True), (64, 20, False), (13, 8, True),
                                        (15, 15, False), (62, 6, False), (63, 12, True), (250, 2, False), (255, 15, True)])
def test_finalize_many_rows(E, k, margin):
    """6400 rows whose slices of r (two or four) meet in the workspace: several lanes per row with 4, 16, 8 x 16 and
    16 x 16 scores between them and lists of 2, 8 and 16, E a multiple of 4 and not; k above 16 takes a wave per row.
    Every row against the oracle; the margin equals the difference of the two exported scores."""
    T = 400 if k <= 16 else 64
    x, W1, W2, b1, b2 = _rand_layers(700 + E + k, L=16, T=T, d=128, r=256, E=E, dtype="bf16", bias=True)
    path = "auto" if k <= 16 else "decode"
    _run_and_check(x, W1, W2, b1, b2, k, "bf16", path=path, what=f"finalize E={E} k={k}")
    if margin:
        o = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k, b1=_dev(b1, "bf16"), b2=_dev(b2, "bf16"),
                      path=path, want_logits=True, want_margin=True)
        z = o.logits.sort(dim=2, descending=True).values
        want = z[:, :, k - 1] - z[:, :, k] if k < E else torch.full_like(o.margin, float("inf"))
        assert torch.equal(o.margin, want)


@pytest.mark.parametrize("E,k", [(1, 1), (2, 2), (3, 1), (5, 5), (7, 3)])
def test_finalize_many_rows_of_few_experts(E, k):
    """The same with so few experts that a row's largest score can be close to 0, which the oracle check's scale (that
    score) does not fit: scores within 0.02 of the scores' norm over the batch (bf16 rounding of h, the bound of the
    oracle check), selection, probabilities and margin from the exported scores."""
    x, W1, W2, _, b2 = _rand_layers(750 + E, L=16, T=400, d=128, r=256, E=E, dtype="bf16", bias=True)
    xs, a, b, c = (_dev(v, "bf16") for v in (x, W1, W2, b2))
    o = B.predict(xs, a, b, k, b2=c, want_logits=True, want_margin=True)
    z = torch.matmul(torch.matmul(xs.double(), a.double().transpose(1, 2)), b.double().transpose(1, 2)) + c.double()[:, None]
    assert float((o.logits - z).abs().max()) <= 0.02 * float(z.square().mean().sqrt()) * 5     # 5: the largest of 6400 E
    srt, order = torch.sort(o.logits, dim=2, descending=True, stable=True)
    assert torch.equal(o.idx.long(), order[:, :, :k])
    want = torch.softmax(o.logits.double(), dim=2).gather(2, order[:, :, :k])
    assert float(((o.probs - want) / want).abs().max()) <= parity.PROB_TOL_OWN
    assert torch.equal(o.margin, srt[:, :, k - 1] - srt[:, :, k] if k < E else torch.full_like(o.margin, float("inf")))


# ------------------------------------------------------------------ activations on the bf16 grid
@pytest.mark.parametrize("act", ["silu", "gelu"])
@pytest.mark.parametrize("path,T,d,r", [("prefill", 4096, 32, 128), ("decode", 64, 128, 64), ("decode", 64, 128, 128)])
def test_activation_over_the_bf16_grid(path, T, d, r, act):
    """One hidden unit per token holds a bf16 value v (x[t, 0] = v, W1 = 1), the score of expert 0 is act(v): it must be
    act(v) in float64 rounded to bf16, to the bit, for every v of magnitude 2^-60 .. 64 whose result is a normal number.
    A value within 1e-6 of a rounding boundary may go either way (the float32 arithmetic's own bound)."""
    from scipy.special import log_ndtr
    bits = np.arange(65536, dtype=np.uint32) << 16
    v = bits.view(np.float32)
    v = v[np.isfinite(v) & (np.abs(v) >= 2.0 ** -60) & (np.abs(v) <= 64)].astype(np.float64)
    exact = v * np.exp(log_ndtr(v)) if act == "gelu" else v * np.exp(-np.logaddexp(0.0, -v))
    keep = np.abs(exact) >= 2.0 ** -125
    v, exact = v[keep], exact[keep]
    L = -(-v.size // T)
    x = torch.zeros((L, T, d), dtype=torch.bfloat16, device="cuda")
    flat = torch.zeros(L * T, dtype=torch.float64)
    flat[:v.size] = torch.from_numpy(v)
    x[:, :, 0] = flat.view(L, T).to(torch.bfloat16).cuda()
    W1 = torch.zeros((L, r, d), dtype=torch.bfloat16, device="cuda")
    W1[:, :, 0] = 1.0
    W2 = torch.zeros((L, 2, r), dtype=torch.bfloat16, device="cuda")
    W2[:, 0, r - 3] = 1.0
    out = B.predict(x, W1, W2, 1, act=act, path=path, want_logits=True)
    torch.cuda.synchronize()
    got = out.logits[:, :, 0].reshape(-1)[:v.size].double().cpu().numpy()

    def to_bf16(a):
        m, e = np.frexp(a)
        return np.ldexp(np.rint(m * 256) / 256, e)
    lo, hi = to_bf16(exact * (1 - 1e-6)), to_bf16(exact * (1 + 1e-6))
    bad = (got != lo) & (got != hi)
    assert not bad.any(), (v[bad][:5], got[bad][:5], exact[bad][:5])
    print(f"{path} {act}: {v.size} values, {(got != to_bf16(exact)).sum()} not correctly rounded", flush=True)


# ------------------------------------------------------------------ biases that start anywhere
@pytest.mark.parametrize("T,d,r,E,L,act", [(300, 64, 256, 40, 2, "none"), (8200, 64, 512, 64, 8, "gelu"),
                                           (1000, 64, 1024, 200, 33, "silu"), (5, 128, 128, 20, 3, "none"),
                                           (40, 128, 192, 20, 3, "silu")])
def test_biases_that_start_in_the_middle_of_a_word(T, d, r, E, L, act):
    """b1 and b2 need no alignment beyond their own: shifted by one element they give the same bits."""
    x, W1, W2, b1, b2 = _rand_layers(60 + T, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    args = _dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), 4
    a1, a2 = _dev(b1, "bf16"), _dev(b2, "bf16")
    shift = lambda t: torch.cat([t.new_full((1,), 99.0), t.flatten()])[1:].view(t.shape)
    s1, s2 = shift(a1), shift(a2)
    assert s1.data_ptr() % 4 == 2 and s2.data_ptr() % 4 == 2
    a = B.predict(*args, b1=a1, b2=a2, act=act, want_logits=True)
    b = B.predict(*args, b1=s1, b2=s2, act=act, want_logits=True)
    assert torch.equal(a.logits, b.logits) and torch.equal(a.idx, b.idx) and torch.equal(a.probs, b.probs)


def _same_with_counts_and_margin(x, W1, W2, b1, b2, k, act, out, workspace=None):
    """The call again with counts and margin: the same outputs, counts added to what is there, the margin of the scores."""
    L, E = W2.shape[:2]
    dev = lambda v: None if v is None else _dev(v, "bf16")
    counts = torch.full((L, E), 3, dtype=torch.int32, device="cuda")
    o = B.predict(dev(x), dev(W1), dev(W2), k, b1=dev(b1), b2=dev(b2), act=act, counts=counts, want_margin=k < 16,
                  workspace=workspace)
    torch.cuda.synchronize()
    assert torch.equal(o.idx, out.idx) and torch.equal(o.probs, out.probs)
    ref = torch.stack([torch.bincount(o.idx[l].flatten().long(), minlength=E) for l in range(L)])
    assert torch.equal(counts.long() - 3, ref)
    if k < 16:
        srt = torch.sort(out.logits, dim=2, descending=True).values
        assert torch.equal(o.margin, srt[:, :, k - 1] - srt[:, :, k] if k < E else torch.full_like(o.margin, float("inf")))


@pytest.mark.parametrize("E,k,r,d,L,T,act,bias,kernel", [
    # 256 tiles of 256 tokens: whole rounds, no tiles of 224, r not split; one to three chunks of r; d of an odd multiple of
    # 32: half a stage at the end; the last tile of 1 to 255 rows; up to 32 and up to 64 experts
    (16, 2, 256, 160, 16, 3841, "none", True, "256x256"), (8, 3, 512, 448, 16, 4090, "none", False, "256x256"),
    (32, 8, 512, 288, 16, 4000, "silu", True, "256x256"), (20, 5, 256, 224, 16, 4095, "gelu", True, "256x256"),
    (64, 12, 512, 1056, 16, 3900, "none", True, "256x256"), (48, 5, 256, 384, 16, 4096, "none", False, "256x256"),
    (64, 16, 256, 320, 16, 4095, "silu", True, "256x256"), (33, 6, 768, 192, 16, 4095, "gelu", True, "256x256"),
    # r split over two and three workgroups; 256 + 41 tiles, of which the 41 are
    (64, 12, 512, 1056, 8, 4099, "none", True, "256x256"), (24, 6, 768, 160, 5, 8229, "silu", True, "256x256"),
    (64, 6, 1024, 192, 9, 8229, "none", True, "256x256"), (30, 6, 1024, 160, 9, 8229, "gelu", True, "256x256"),
    # more experts
    (65, 8, 512, 160, 16, 4097, "silu", True, "256x256 wide"), (128, 16, 256, 32, 16, 4351, "gelu", True, "256x256 wide"),
    (100, 15, 512, 192, 16, 4095, "silu", True, "256x256 wide"), (128, 7, 768, 96, 16, 4000, "none", False, "256x256 wide"),
    (128, 8, 512, 288, 8, 4100, "none", True, "256x256 wide"),
    (70, 8, 384, 224, 16, 4100, "none", True, "256x128"), (90, 7, 384, 160, 16, 4000, "gelu", True, "256x128"),
    (129, 3, 640, 288, 16, 4100, "gelu", True, "256x128"), (256, 16, 512, 32, 16, 4100, "silu", True, "256x128"),
    (255, 8, 128, 160, 16, 4099, "none", True, "256x128"), (256, 15, 384, 96, 16, 4095, "none", False, "256x128"),
])
def test_prefill_tiles_of_256_tokens(E, k, r, d, L, T, act, bias, kernel):
    """One- and two-half stages, ragged tiles, experts on either side of a block of 16 and of a shape's limit; with the
    least workspace, so that the fused kernel runs.  Every seventh row and the last tile's; counts and margin."""
    x, W1, W2, b1, b2 = _rand_layers(270 + E + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    desc = B.make_desc(T, d, r, E, k, L, B.BF16, act=act)
    ws = torch.empty(max(B.predict_workspace_min_bytes(desc), 16), dtype=torch.uint8, device="cuda")
    assert B.predict_kernel(desc, workspace_bytes=ws.numel(), with_b1=bias) == "prefill256_kernel " + kernel
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"256 tokens E={E} r={r} d={d} {act}",
                             rows=np.unique(np.concatenate([np.arange(0, T, 7), np.arange(T - 260, T)])), workspace=ws)
    assert out.path == "prefill"
    _same_with_counts_and_margin(x, W1, W2, b1, b2, k, act, out, ws)


@pytest.mark.parametrize("E,k,r,d,L,T,act,bias", [
    # one, two and four chunks of r; d of an odd multiple of 32; 14 blocks of 16 tokens, the last tile of 1, 64 and 223 rows;
    # experts on either side of a block of 16 and of 32
    (64, 6, 512, 640, 26, 4096, "none", False), (33, 16, 512, 160, 26, 4033, "gelu", True),
    (16, 2, 256, 1056, 26, 4033, "none", True), (32, 8, 1024, 224, 25, 4255, "silu", True),
    (5, 5, 512, 672, 25, 4096, "none", False), (64, 15, 1024, 160, 25, 4255, "none", True),
])
def test_prefill_tiles_of_224_tokens(E, k, r, d, L, T, act, bias):
    """Calls of 400 to 442 tiles of 256 tokens, 475 to 494 of 224, take the latter.  Every ninth row and the last tile's; counts
    and margin."""
    assert B.predict_kernel(B.make_desc(T, d, r, E, k, L, B.BF16, act=act), with_b1=bias) == "prefill256_kernel 224x256"
    x, W1, W2, b1, b2 = _rand_layers(370 + E + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"224 tokens E={E} r={r} d={d} {act}",
                             rows=np.unique(np.concatenate([np.arange(0, T, 9), np.arange(T - 224, T)])))
    assert out.path == "prefill"
    _same_with_counts_and_margin(x, W1, W2, b1, b2, k, act, out)


@pytest.mark.parametrize("E,k,r,d,L,T,act,bias", [
    # 256 x 256 tiles in eight waves: short rows, d = 32 to 608; r split into four and whole, the last 41 of 297 tiles cut
    (64, 6, 512, 64, 8, 8229, "gelu", True), (20, 15, 256, 128, 16, 4095, "silu", True), (33, 8, 512, 160, 16, 4095, "none", False),
    (16, 2, 1024, 608, 9, 8229, "none", False), (64, 12, 1024, 96, 4, 8229, "none", True), (64, 8, 2048, 224, 16, 3000, "none", False),
])
def test_prefill_short_rows_of_few_experts(E, k, r, d, L, T, act, bias):
    """Every seventh row and the last tile's; counts and margin."""
    assert B.predict_kernel(B.make_desc(T, d, r, E, k, L, B.BF16, act=act), with_b1=bias).startswith("prefill_kernel 256x256")
    x, W1, W2, b1, b2 = _rand_layers(420 + E + d, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"short rows E={E} r={r} d={d} {act}",
                             rows=np.unique(np.concatenate([np.arange(0, T, 7), np.arange(T - 260, T)])))
    assert out.path == "prefill"
    _same_with_counts_and_margin(x, W1, W2, b1, b2, k, act, out)


@pytest.mark.parametrize("T,r,E,L,d", [(300, 1024, 20, 3, 192), (300, 1024, 200, 3, 192), (130, 384, 100, 5, 192), (65, 512, 64, 1, 192),
                                       (513, 1024, 16, 2, 192),
                                       (65, 1024, 16, 3, 2048), (130, 1024, 16, 5, 2048), (300, 640, 200, 3, 4096),
                                       (257, 1024, 20, 5, 2048), (1000, 1024, 20, 3, 2048)])
def test_prefill_few_tiles_of_several_layers(T, r, E, L, d):
    """Shares of the chip's eight parts that end within a layer, groups of hidden units fastest in them or, with long rows,
    token tiles, in tiles of 64 x 64, 128 x 128 and those of many experts; every row (of more than 600, every fourth)."""
    name = B.predict_kernel(B.make_desc(T, d, r, E, 6, L, B.BF16), with_b1=True)
    assert name.startswith("prefill_kernel ") and name.endswith("tiles first") == (d >= 2048), name
    x, W1, W2, b1, b2 = _rand_layers(470 + E, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, 6, "bf16", what=f"few tiles T={T} r={r} E={E} L={L} d={d} {name}",
                             rows=np.unique(np.concatenate([np.arange(0, T, 4), np.arange(max(0, T - 70), T)])) if T > 600 else None)
    assert out.path == "prefill"


@pytest.mark.parametrize("L,T,d,r,E,k", [(1, 3, 128, 128, 60, 16), (1, 3, 128, 128, 200, 16), (1, 100, 64, 128, 60, 7),
                                         (16, 4097, 160, 256, 60, 16), (16, 4097, 160, 256, 100, 2),
                                         (16, 4097, 160, 256, 200, 7), (64, 64, 128, 128, 60, 8)])
def test_selection_of_infinities_zeros_and_nan(L, T, d, r, E, k):
    """Tokens of zeros leave the scores to b2: infinities, both zeros (a tie), NaN (below everything), the largest and the
    smallest values, each of them several times.  Selection and order are the rule's on every row."""
    vals = np.array([np.inf, -np.inf, 0.0, -0.0, np.nan, 3.0e38, -3.0e38, 1e-38, -1e-38, 1.0, -1.0], dtype=np.float32)
    g = np.random.default_rng(E + k)
    b2 = vals[g.integers(0, len(vals), (L, E))]
    x = torch.zeros((L, T, d), dtype=torch.bfloat16, device="cuda")
    w = lambda *s: torch.full(s, 0.5, dtype=torch.bfloat16, device="cuda")
    out = B.predict(x, w(L, r, d), w(L, E, r), k, b2=_dev(b2, "bf16"))
    torch.cuda.synchronize()
    key = np.where(np.isnan(b2), -np.inf, b2 + 0.0)
    want = np.stack([np.lexsort((np.arange(E), -key[l], np.isnan(b2[l])))[:k] for l in range(L)])
    assert (out.idx.cpu().numpy() == want[:, None, :]).all()


# ------------------------------------------------------------------ two passes for many experts
@pytest.mark.parametrize("T,d,r,E,k,L,act,bias", [
    (4097, 64, 256, 129, 8, 8, "none", False),             # 17 tiles a layer, one row in the last; one chunk of r
    (8191, 96, 768, 256, 15, 4, "silu", True),             # three chunks: one workgroup per tile takes them all
    (1000, 64, 1024, 200, 3, 33, "gelu", True),            # four chunks, four workgroups per tile; 132 tiles
    (4100, 768, 512, 250, 8, 16, "none", True),            # scores that are no multiple of 4 apart
    (6000, 1024, 256, 140, 8, 11, "none", True),           # 264 tiles: from 256 on not with narrower tokens
    (12300, 1536, 256, 100, 6, 8, "gelu", True),           # up to 128 experts: from 384 tiles on
])
def test_two_passes_and_one(T, d, r, E, k, L, act, bias):
    """First layer and scores as two kernels, against the oracle, and the fused kernel that runs with a smaller
    workspace: the hidden vector is the same to the bit, the scores add the same products in another order (2e-6 of the
    row's scale: r products of 2^-24 each, as a random walk, four times over)."""
    x, W1, W2, b1, b2 = _rand_layers(700 + E, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"two passes T={T} d={d} r={r} E={E}",
                             rows=np.unique(np.concatenate([np.arange(0, T, 9), np.arange(T - 300, T)])))
    need = B.predict_workspace_bytes(B.make_desc(T, d, r, E, k, L, B.BF16, act=act))
    assert need >= 2 * T * r                               # h of a layer at least
    counts = torch.zeros((L, E), dtype=torch.int32, device="cuda")
    args = _dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k
    opts = dict(b1=None if b1 is None else _dev(b1, "bf16"), b2=None if b2 is None else _dev(b2, "bf16"), act=act,
                want_logits=True)
    two = B.predict(*args, counts=counts, **opts)
    one = B.predict(*args, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"), **opts)
    torch.cuda.synchronize()
    assert torch.equal(two.idx, out.idx) and torch.equal(two.probs, out.probs)
    scale = one.logits.abs().amax(dim=2, keepdim=True)
    assert ((two.logits - one.logits).abs() <= 2e-6 * scale).all()
    ref = torch.stack([torch.bincount(two.idx[l].flatten().long(), minlength=E) for l in range(L)])
    assert torch.equal(counts.long(), ref)


@pytest.mark.parametrize("E,k,margin", [(129, 1, True), (144, 2, False), (200, 2, True), (130, 7, True), (255, 8, False),
                                        (256, 15, True), (256, 16, False)])
@pytest.mark.parametrize("prob", ["softmax", "softmax_topk", "sigmoid"])
def test_two_passes_finish_their_rows(E, k, margin, prob):
    """Whole r in one slice: the scores kernel selects by itself, with lists of 2, 8 and 16 keys.  Against the definition in
    float64 on its own scores; probabilities to 2e-5 of their value, the bound of tests/parity.py for the same comparison."""
    T, d, r, L = 4097, 64, 256, 12
    assert _plan(T, d, r, E, k, L).tile == "two-pass 256x256"
    x, W1, W2, _, b2 = _rand_layers(E + k, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=True)
    o = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k, b2=_dev(b2, "bf16"), prob=prob, want_logits=True,
                  want_margin=margin)
    srt, order = torch.sort(o.logits, dim=2, descending=True, stable=True)
    assert torch.equal(o.idx.long(), order[:, :, :k])
    if margin:
        assert torch.equal(o.margin, srt[:, :, k - 1] - srt[:, :, k])
    z = srt.double()
    want = torch.sigmoid(z) if prob == "sigmoid" else torch.softmax(z[:, :, :k] if prob == "softmax_topk" else z, dim=2)
    want = want[:, :, :k]
    assert ((o.probs.double() - want).abs() <= 2e-5 * want).all()


@pytest.mark.parametrize("E", [200, 256])
def test_two_pass_probabilities_are_sums_of_short_chains(E):
    """The first probability, 1 / sum exp(z - max), against float64 on the row's own scores, over 50000 rows.  With u = 2.5e-8, the
    rms of one float32 rounding relative to a value of any mantissa: chains of 16 terms in 16 accumulators that are then
    added in pairs give 1.5 u, the reciprocal and the product 1 u together, the exponentials' mean error 2.1e-8: 5.0e-8 (5.3 to 5.4
    seen).  Chains of 64 in 4 accumulators give 2.6 u, in all 7.3e-8 (7.2 to 7.7 seen).  The bar stands between."""
    L, T, d, r = 50, 1000, 64, 256
    assert _plan(T, d, r, E, 8, L).tile == "two-pass 256x256"
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, W1, W2 = rnd(L, T, d), rnd(L, r, d) / d ** 0.5, rnd(L, E, r) / r ** 0.5
    o = B.predict(x.to(torch.bfloat16), W1.to(torch.bfloat16), W2.to(torch.bfloat16), 8, want_logits=True)
    z = o.logits.double()
    want = 1 / torch.exp(z - z.amax(dim=2, keepdim=True)).sum(dim=2)
    assert float(((o.probs[..., 0].double() - want) / want).square().mean().sqrt()) <= 6.2e-8


@pytest.mark.parametrize("T,d,r,E,k,L,act,shared,batches", [
    (5000, 768, 4096, 200, 8, 32, "none", False, (11, 11, 10)),
    (5000, 768, 4096, 256, 15, 32, "silu", True, (11, 11, 10)),
    (8100, 2048, 2048, 128, 8, 21, "gelu", False, (11, 10)),
])
def test_two_passes_in_batches_of_layers(T, d, r, E, k, L, act, shared, batches):
    """More layers than 600 MB of hidden vectors hold: batches of them, the last one shorter, each with its own part of
    every operand and output; a ragged last tile.  Both biases, scores, margin and counts; layers that share their
    tokens.  Rows of every layer against the oracle, every row against the fused kernel (2e-6 of the row's scale, as
    above)."""
    desc = B.make_desc(T, d, r, E, k, L, B.BF16, act=act)
    assert B.predict_plan(desc, want_margin=True).tile == "two-pass 256x256"
    need, tiles = B.predict_workspace_bytes(desc), -(-T // 256)
    assert sum(batches) == L and batches[0] * tiles * 256 * (r * 2 + E * 4) == need
    g = torch.Generator(device="cuda").manual_seed(T + E)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)
    x = torch.stack([rnd(T, d).to(torch.bfloat16) for _ in range(1 if shared else L)])
    W1 = torch.stack([(rnd(r, d) / d ** 0.5).to(torch.bfloat16) for _ in range(L)])
    W2 = (rnd(L, E, r) / r ** 0.5).to(torch.bfloat16)
    b1, b2 = (0.3 * rnd(L, r)).to(torch.bfloat16), (0.5 * rnd(L, E)).to(torch.bfloat16)
    opts = dict(b1=b1, b2=b2, act=act, want_logits=True, want_margin=True)
    counts = torch.full((L, E), 5, dtype=torch.int32, device="cuda")
    out = B.predict(x, W1, W2, k, counts=counts, **opts)
    one = B.predict(x, W1, W2, k, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"), **opts)
    torch.cuda.synchronize()
    scale = one.logits.abs().amax(dim=2, keepdim=True)
    assert ((out.logits - one.logits).abs() <= 2e-6 * scale).all()
    srt, order = torch.sort(out.logits, dim=2, descending=True, stable=True)
    assert torch.equal(out.idx.long(), order[:, :, :k])
    assert torch.equal(out.margin, srt[:, :, k - 1] - srt[:, :, k])
    ref = torch.stack([torch.bincount(out.idx[l].flatten().long(), minlength=E) for l in range(L)])
    assert torch.equal(counts.long() - 5, ref)
    rows = np.unique(np.concatenate([np.arange(7, T, T // 6), [0, T - 1]]))
    cpu = lambda t: t.float().cpu().numpy()
    for l in range(L):
        parity.check_layer(cpu(x[0 if shared else l][rows]), cpu(W1[l]), cpu(W2[l]), cpu(b1[l]), cpu(b2[l]), ACT_ID[act], k,
                           "bf16", out.idx[l].cpu().numpy()[rows], out.probs[l].cpu().numpy()[rows],
                           out.logits[l].cpu().numpy()[rows], what=f"batches layer {l}")


def test_predict_runs_where_its_best_workspace_does_not_fit(monkeypatch):
    """The allocation of h for two passes fails: the call goes on in the least workspace instead of raising."""
    T, d, r, E, k, L = 1000, 64, 1024, 200, 3, 33
    desc = B.make_desc(T, d, r, E, k, L, B.BF16)
    least, best = B.predict_workspace_min_bytes(desc), B.predict_workspace_bytes(desc)
    assert B.predict_plan(desc).tile == "two-pass 256x256" and least < best
    x, W1, W2, _, _ = _rand_layers(3, L=L, T=T, d=d, r=r, E=E, dtype="bf16")
    args = _dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k
    one = B.predict(*args, want_logits=True, workspace=torch.empty(max(least, 16), dtype=torch.uint8, device="cuda"))
    empty, sizes = torch.empty, []

    def full_device(*size, **kw):
        if kw.get("dtype") == torch.uint8:
            sizes.append(size[0])
            if size[0] > least:
                raise torch.OutOfMemoryError("planted")
        return empty(*size, **kw)
    monkeypatch.setattr(torch, "empty", full_device)
    out = B.predict(*args, want_logits=True)
    monkeypatch.undo()
    assert sizes[0] == best
    assert torch.equal(out.logits, one.logits) and torch.equal(out.idx, one.idx) and torch.equal(out.probs, one.probs)


@pytest.mark.parametrize("T,E,k", [(64, 64, 6), (63, 16, 2), (64, 16, 12), (33, 16, 12)])
def test_counts_of_a_decode_batch(T, E, k):
    """33 layers, 1089 to 2112 rows: counted by a wave per row, by several lanes per row, from the selections of those."""
    x, W1, W2, _, _ = _rand_layers(T + k, L=33, T=T, d=128, r=256, E=E, dtype="bf16")
    counts = torch.full((33, E), 7, dtype=torch.int32, device="cuda")
    out = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k, counts=counts)
    torch.cuda.synchronize()
    assert out.path == "decode"
    ref = torch.stack([torch.bincount(out.idx[l].flatten().long(), minlength=E) for l in range(33)])
    assert torch.equal(counts.long() - 7, ref)


def test_counts_of_rows_finished_outside_the_prefill_kernel():
    """More than 1024 rows whose r is split: the counts come from the selections, whole layers and the last tiles of a call
    (33 x 9 tiles: the 41 beyond the full round of 256 are cut along r)."""
    for T, d, r, E, L in ((500, 64, 512, 64, 3), (8229, 64, 1024, 64, 9)):
        x, W1, W2, _, _ = _rand_layers(T, L=L, T=T, d=d, r=r, E=E, dtype="bf16")
        counts = torch.full((L, E), 7, dtype=torch.int32, device="cuda")
        out = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), 6, counts=counts)
        torch.cuda.synchronize()
        ref = torch.stack([torch.bincount(out.idx[l].flatten().long(), minlength=E) for l in range(L)])
        assert torch.equal(counts.long() - 7, ref)


# ------------------------------------------------------------------ 64 x 64 tiles
@pytest.mark.parametrize("T,d,r,E,k,L,act,bias", [
    (65, 64, 128, 16, 2, 1, "none", False),                # one stage per chunk, one row in the second tile
    (127, 192, 256, 33, 6, 3, "silu", True),               # three stages: fewer than the ring
    (200, 640, 384, 64, 6, 2, "gelu", True),               # two blocks of experts, a ragged tile
    (512, 448, 512, 128, 8, 1, "none", True),              # four blocks
    (1000, 320, 512, 65, 12, 2, "silu", False),            # several rows' finalize form, 256 workgroups
])
def test_prefill_64x64_tiles(T, d, r, E, k, L, act, bias):
    """Against the oracle, every row, and the 128 x 128 tiles that run with a smaller workspace: the same hidden vector,
    the scores' slices of r half as wide (2e-6 of the row's scale, as for the two passes)."""
    assert _plan(T, d, r, E, k, L).tile == "64x64"
    x, W1, W2, b1, b2 = _rand_layers(800 + T, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"64x64 T={T} d={d} r={r} E={E}")
    need = B.predict_workspace_bytes(B.make_desc(T, d, r, E, k, L, B.BF16))
    one = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k, act=act, want_logits=True,
                    b1=None if b1 is None else _dev(b1, "bf16"), b2=None if b2 is None else _dev(b2, "bf16"),
                    workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    scale = one.logits.abs().amax(dim=2, keepdim=True)
    assert ((out.logits - one.logits).abs() <= 2e-6 * scale).all()


# ------------------------------------------------------------------ few tokens: 128 to 256 tokens x 256 hidden units
@pytest.mark.parametrize("L,T,d,r,E,k,act,bias,kernel,groups", [
    (60, 130, 96, 256, 33, 6, "none", False, "128x256", 1),            # two rows in the second tile; a stage and a half
    (26, 130, 64, 768, 64, 12, "none", True, "128x256", 3),            # r in three, one stage per chunk
    (40, 223, 320, 768, 16, 2, "none", True, "128x256", 3),
    (13, 900, 64, 512, 100, 12, "silu", True, "128x256", 2),           # up to 128 experts; a ragged last tile
    (60, 200, 32, 256, 128, 15, "none", True, "128x256", 1),           # ... one stage in all
    (127, 130, 32, 256, 16, 2, "silu", True, "160x256", 1),            # half a stage
    (40, 159, 448, 768, 64, 6, "gelu", False, "160x256", 3),           # seven stages
    (40, 161, 192, 768, 64, 8, "gelu", True, "192x256", 3),
    (40, 161, 32, 768, 20, 3, "none", False, "192x256", 3),            # ... few experts
    (30, 210, 32, 1024, 33, 6, "none", True, "224x256", 4),            # ragged, r split
    (33, 208, 32, 1024, 16, 2, "gelu", False, "224x256", 4),           # ... few experts
    (40, 480, 256, 768, 33, 6, "silu", False, "256x256", 3),
    (43, 225, 32, 768, 20, 12, "silu", True, "256x256", 3),            # ... few experts
    # token tiles fastest in an XCD's share of the grid, which ends within a layer (of 7 layers one share is 17 or 18 of 20
    # workgroups a layer); r whole and in five, last tiles of 3 to 222 rows
    (5, 3003, 736, 256, 16, 2, "none", True, "128x256 tiles first", 1),
    (7, 387, 960, 1280, 33, 6, "silu", True, "128x256 tiles first", 5),
    (6, 387, 992, 1280, 128, 7, "gelu", True, "128x256 tiles first", 5),
    (6, 2387, 768, 256, 100, 6, "none", False, "128x256 tiles first", 1),
    (6, 1076, 896, 1280, 33, 6, "none", True, "160x256 tiles first", 5),
    (6, 1323, 736, 1280, 20, 3, "silu", False, "192x256 tiles first", 5),
    (6, 1566, 1248, 1280, 40, 9, "none", True, "224x256 tiles first", 5),
])
def test_prefill_few_tokens(L, T, d, r, E, k, act, bias, kernel, groups):
    """Against the oracle; and, every row of three layers, against calls of those layers alone, which run another kernel's tiles of
    64 x 64 or 128 x 128: the same hidden vector, scores of other slices of r (2e-6 of the row's scale, as for the two passes);
    with counts and margin."""
    desc = B.make_desc(T, d, r, E, k, L, B.BF16, act=act)
    assert B.predict_kernel(desc, with_b1=bias) == "prefill256_kernel " + kernel
    assert B.predict_plan(desc) == B.Plan("prefill", "128-256x256", groups, r // 256 // groups)
    assert B.predict_kernel(B.make_desc(T, d, r, E, k, 1, B.BF16, act=act), with_b1=bias).startswith("prefill_kernel ")
    x, W1, W2, b1, b2 = _rand_layers(1000 + T + E, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    rows = np.unique(np.concatenate([np.arange(0, T, 7 if T < 1000 else 41), np.arange(T - 40, T)]))
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"few tokens {L} x {T} d={d} r={r} E={E}", rows=rows)
    _same_with_counts_and_margin(x, W1, W2, b1, b2, k, act, out)
    for l in (0, L // 2, L - 1):
        one = B.predict(_dev(x[l], "bf16"), _dev(W1[l], "bf16"), _dev(W2[l], "bf16"), k, act=act, want_logits=True,
                        b1=None if b1 is None else _dev(b1[l], "bf16"), b2=None if b2 is None else _dev(b2[l], "bf16"))
        scale = one.logits.abs().amax(dim=2, keepdim=True)
        assert ((out.logits[l] - one.logits).abs() <= 2e-6 * scale).all()


@pytest.mark.parametrize("L,T,d,r,E", [(60, 130, 64, 256, 64), (60, 200, 32, 256, 128), (12, 4096, 512, 512, 64),
                                       (12, 4096, 512, 256, 128)])
def test_probabilities_are_sums_of_short_chains(L, T, d, r, E):
    """The first probability of calls that finish their rows in prefill256_kernel, as in the test of two passes: one or two lanes
    a row with 8 chains each, of up to 16 terms, 5.0e-8 (5.1 to 5.5 seen); one chain a lane, of 32 to 128 terms, gives 7.5e-8 to
    1.7e-7 (both seen)."""
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, W1, W2 = rnd(L, T, d), rnd(L, r, d) / d ** 0.5, rnd(L, E, r) / r ** 0.5
    assert _plan(T, d, r, E, 8, L).groups == 1
    o = B.predict(x.to(torch.bfloat16), W1.to(torch.bfloat16), W2.to(torch.bfloat16), 8, want_logits=True)
    z = o.logits.double()
    want = 1 / torch.exp(z - z.amax(dim=2, keepdim=True)).sum(dim=2)
    assert float(((o.probs[..., 0].double() - want) / want).square().mean().sqrt()) <= 6.2e-8


# ------------------------------------------------------------------ 128 to 511 tiles: r split evenly
@pytest.mark.parametrize("L,T,d,r,E,k,act,bias,kernel,groups", [
    (64, 300, 192, 256, 40, 6, "silu", True, "160x256", 1), (64, 300, 192, 512, 16, 3, "silu", True, "160x256", 2),
    (64, 265, 160, 512, 33, 6, "none", False, "160x256", 2), (33, 1000, 416, 768, 60, 6, "gelu", True, "160x256", 1),
    (40, 1000, 192, 256, 16, 2, "silu", True, "192x256", 1), (64, 357, 288, 512, 40, 6, "none", False, "192x256", 2),
    (40, 1000, 192, 1024, 16, 3, "none", True, "192x256", 2),          # an even split for b1's sake
    (30, 1569, 160, 512, 33, 8, "silu", True, "224x256", 1),
    (43, 589, 384, 768, 16, 4, "none", False, "224x256", 3), (64, 422, 320, 512, 33, 6, "gelu", True, "224x256", 2),
    (16, 1929, 192, 1024, 33, 12, "gelu", True, "256x256", 2),
    (64, 339, 256, 1024, 100, 6, "silu", True, "256x256 wide", 2), (16, 1800, 640, 768, 128, 12, "none", False, "256x256 wide", 1),
])
def test_prefill_even_splits(L, T, d, r, E, k, act, bias, kernel, groups):
    """Against the oracle; and against the layout that runs with the least workspace, which splits r otherwise or has other
    tiles: the same hidden vector, scores of other slices of r (2e-6 of the row's scale, as for the two passes); with counts
    and margin."""
    desc = B.make_desc(T, d, r, E, k, L, B.BF16, act=act)
    least, asked = B.predict_workspace_min_bytes(desc), B.predict_workspace_bytes(desc)
    assert B.predict_kernel(desc, with_b1=bias) == "prefill256_kernel " + kernel and asked > least
    if not bias or act != "none":                          # else the plan, which knows of no b1, is another
        assert B.predict_plan(desc).groups == groups
    x, W1, W2, b1, b2 = _rand_layers(1100 + T + E, L=L, T=T, d=d, r=r, E=E, dtype="bf16", bias=bias)
    rows = np.unique(np.concatenate([np.arange(0, T, 29), np.arange(T - 20, T)]))
    out, *_ = _run_and_check(x, W1, W2, b1, b2, k, "bf16", act=act, what=f"even splits {L} x {T} d={d} r={r} E={E}", rows=rows)
    _same_with_counts_and_margin(x, W1, W2, b1, b2, k, act, out)
    one = B.predict(_dev(x, "bf16"), _dev(W1, "bf16"), _dev(W2, "bf16"), k, act=act, want_logits=True,
                    b1=None if b1 is None else _dev(b1, "bf16"), b2=None if b2 is None else _dev(b2, "bf16"),
                    workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    other = B.predict_kernel(desc, workspace_bytes=least, with_b1=bias)
    # tiles of another size are seen in the name; workgroups of another number by the order of the scores' sums
    assert other != "prefill256_kernel " + kernel or not torch.equal(out.logits, one.logits)
    scale = one.logits.abs().amax(dim=2, keepdim=True)
    assert ((out.logits - one.logits).abs() <= 2e-6 * scale).all()
    if groups > 1:                                         # score tiles of all of them, tokens of the tile x experts
        tokens = int(kernel.split("x")[0])
        assert asked >= -(-T // tokens) * L * groups * tokens * E * 4


@pytest.mark.parametrize("d,r,E,act,groups", [(3072, 512, 16, "none", 2), (3616, 768, 64, "silu", 1), (4064, 1024, 40, "gelu", 2),
                                              (5120, 1024, 64, "none", 4)])
def test_prefill_long_rows_of_many_tiles(d, r, E, act, groups):
    """512 tiles and more: two workgroups to a tile from d = 3072 (where the chunks of r divide), four from 5120; layers that
    share their tokens.  Every row against the layout of the least workspace (2e-6 of the row's scale, as above; the same one
    where the chunks do not divide), some against the oracle."""
    T, L, k = 2041, 64, 6
    desc = B.make_desc(T, d, r, E, k, L, B.BF16, act=act)
    assert _plan(T, d, r, E, k, L).groups == groups
    g = torch.Generator(device="cuda").manual_seed(d)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=g)
    x = rnd(1, T, d).to(torch.bfloat16)
    W1 = torch.stack([(rnd(r, d) / d ** 0.5).to(torch.bfloat16) for _ in range(L)])
    W2 = (rnd(L, E, r) / r ** 0.5).to(torch.bfloat16)
    b1, b2 = (0.3 * rnd(L, r)).to(torch.bfloat16), (0.5 * rnd(L, E)).to(torch.bfloat16)
    opts = dict(b1=b1, b2=b2, act=act, want_logits=True)
    out = B.predict(x, W1, W2, k, **opts)
    least = B.predict_workspace_min_bytes(desc)
    one = B.predict(x, W1, W2, k, workspace=torch.empty(max(least, 16), dtype=torch.uint8, device="cuda"), **opts)
    torch.cuda.synchronize()
    scale = one.logits.abs().amax(dim=2, keepdim=True)
    assert ((out.logits - one.logits).abs() <= 2e-6 * scale).all()
    assert torch.equal(out.logits, one.logits) == (groups == 1)        # another order of the scores' sums: not the same call twice
    assert torch.equal(out.idx.long(), torch.sort(out.logits, dim=2, descending=True, stable=True).indices[:, :, :k])
    rows = np.array([0, 255, 256, 1791, T - 1])
    cpu = lambda t: t.float().cpu().numpy()
    for l in (0, 31, L - 1):
        parity.check_layer(cpu(x[0][rows]), cpu(W1[l]), cpu(W2[l]), cpu(b1[l]), cpu(b2[l]), ACT_ID[act], k, "bf16",
                           out.idx[l].cpu().numpy()[rows], out.probs[l].cpu().numpy()[rows], out.logits[l].cpu().numpy()[rows],
                           what=f"long rows layer {l}")
