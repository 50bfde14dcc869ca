"""Training calls on small blocks (scores in the workspace) against the oracle at the sizes where their tiles, splits and paddings
end; and the block kernels, which larger blocks use, on the cases of test_gpu_loss_bwd.py that are too small to reach them."""
import numpy as np
import pytest
import torch

import test_gpu_loss_bwd as base
from helpers import RTOL_BF16, RTOL_F32, dev_idx, gpu_model, make_case, norm_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scorer,dim,bf16,B,N", [
    ("transe", 256, True, 33, 65), ("rotate", 256, False, 31, 2049),   # one row over a tile; two splits of the queries' pass
    ("complex", 400, True, 2100, 40), ("distmult", 64, False, 2049, 33),   # ... of the pass over the negatives
    ("transe", 72, False, 16, 16), ("complex", 16, True, 15, 17),      # one matrix step and its neighbours; narrow rows
    ("rotate", 144, True, 64, 4200), ("distmult", 248, False, 260, 255),
    ("transe", 512, True, 7, 1)])
@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
def test_small_blocks_match_oracle(orc, scorer, dim, bf16, B, N, loss):
    amp = 0.3 if scorer in ("distmult", "complex") else 0.1
    G = make_case(scorer, 3000, 9, dim, B, N, bf16, amp=amp, zipf=True)
    kw = dict(n_ent_for_c=3000) if loss == "sampled_softmax" else dict(gamma=1.0, adv_temp=0.7)
    base._compare(orc, scorer, loss, G, bf16, 3000, kw=dict(kw, reg_l3=1e-3 if B % 2 else 0.0))


# the largest padded blocks on the small side of every line of the rule (limits of 2, 4 and 7 million pairs by row width and shape)
LARGEST_SMALL = [
    ("transe", 256, True, "logsigmoid", 1024, 4096), ("complex", 256, True, "sampled_softmax", 900, 4000),     # many negatives: 4M pairs
    ("transe", 240, True, "sampled_softmax", 2040, 1020), ("distmult", 256, True, "logsigmoid", 1500, 1200),   # otherwise 2M
    ("rotate", 256, False, "logsigmoid", 2560, 2816), ("distmult", 128, False, "sampled_softmax", 3000, 2300), # other rows: 7M
    ("complex", 400, True, "sampled_softmax", 700, 9000), ("transe", 512, True, "logsigmoid", 1400, 4600),
    ("complex", 400, True, "logsigmoid", 256, 12000), ("transe", 64, False, "logsigmoid", 200, 16000)]         # very many negatives: 4M


@pytest.mark.parametrize("scorer,dim,bf16,loss,B,N", LARGEST_SMALL)
def test_both_sides_of_the_rule_agree(scorer, dim, bf16, loss, B, N):
    """Each route against the other (block_passes takes the block kernels for all); that the two are different kernels shows in the bits."""
    import torch
    import paper_2211_12281_amd as kge
    G = make_case(scorer, 9000, 9, dim, B, N, bf16, amp=0.3 if scorer in ("distmult", "complex") else 0.1, zipf=True)
    model = gpu_model(scorer, G, bf16)
    args = (dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]))
    kw = dict(n_ent_for_c=9000) if loss == "sampled_softmax" else dict(gamma=2.0, adv_temp=0.8)
    got = {k: v.clone() for k, v in kge.loss_bwd(model, loss, *args, **kw).items() if v is not None}
    kge.debug_select("block_passes", True)
    try:
        want = kge.loss_bwd(model, loss, *args, **kw)
    finally:
        kge.debug_select("block_passes", False)
    assert not torch.equal(got["g_ent"][2 * B:], want["g_ent"][2 * B:]) and not torch.equal(got["g_ent"][:B], want["g_ent"][:B])
    tol = RTOL_BF16 if bf16 else RTOL_F32
    assert abs(got["loss"].item() - want["loss"].item()) <= 1e-4 * abs(want["loss"].item())
    for sl in (slice(0, B), slice(B, 2 * B), slice(2 * B, 2 * B + N)):
        assert norm_err(got["g_ent"][sl].cpu().numpy(), want["g_ent"][sl].cpu().numpy()) <= tol
    assert norm_err(got["g_rel"].cpu().numpy(), want["g_rel"].cpu().numpy()) <= tol


@pytest.mark.parametrize("scorer,dim,bf16,loss,B,N", [("complex", 256, True, "sampled_softmax", 900, 4600), ("rotate", 128, False, "logsigmoid", 2600, 2700),
                                                      ("complex", 400, True, "sampled_softmax", 300, 12000)])
def test_blocks_over_the_line_match_oracle(orc, scorer, dim, bf16, loss, B, N):
    """The smallest blocks that the library's own dispatch gives to the block kernels."""
    G = make_case(scorer, 9000, 9, dim, B, N, bf16, amp=0.3 if scorer == "complex" else 0.1, zipf=True)
    base._compare(orc, scorer, loss, G, bf16, 9000, kw=dict(n_ent_for_c=9000) if loss == "sampled_softmax" else dict(gamma=2.0, adv_temp=0.8))


@pytest.mark.parametrize("scorer,dim,B,N,amp", [("distmult", 256, 300, 900, 0.5), ("distmult", 400, 130, 2500, 0.9), ("transe", 256, 200, 1024, 0.1)])
def test_query_gradients_hold_more_than_one_bf16_of_a_coefficient(orc, scorer, dim, B, N, amp):
    """bf16 tables, with relations that leave the heads as they are (no rounding of the query): the heads' gradient rows are then
    sum_n c_n t_n (distances: c_n / distance (t_n - q)) with exact operands, and c_n in two bf16 pieces is within 2^-17 of itself -
    peaked scores, whose dominating coefficient one bf16 would move by up to 2^-8."""
    import paper_2211_12281_amd as kge
    G = make_case(scorer, 3000, 5, dim, B, N, True, amp=amp)
    G["rel"][:] = 1.0 if scorer == "distmult" else 0.0
    loss, kw = ("sampled_softmax", dict(n_ent_for_c=3000)) if scorer == "distmult" else ("logsigmoid", dict(gamma=1.0, adv_temp=4.0))
    out = kge.loss_bwd(gpu_model(scorer, G, True), loss, *(dev_idx(G[k]) for k in ("h", "r", "t", "neg")), loss_scale=1.0, **kw)
    ref = orc.loss_bwd(scorer, loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], loss_scale=1.0, **kw)
    pos, S = orc.score_batch(scorer, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"])
    T, q = G["ent"][G["neg"]].astype(np.float64), G["ent"][G["h"]].astype(np.float64)
    if loss == "sampled_softmax":
        z = np.concatenate([pos[:, None], S + np.log(2999 / N)], axis=1)
        z = np.exp(z - z.max(axis=1, keepdims=True))
        c, spread = z[:, 1:] / z.sum(axis=1, keepdims=True), np.abs(T)
        terms = c @ spread
    else:
        w = np.exp(4.0 * (S - S.max(axis=1, keepdims=True)))
        c = w / w.sum(axis=1, keepdims=True) / (1.0 + np.exp(-(1.0 + S))) / np.maximum(-S, 1e-30)
        terms = np.stack([c[b] @ np.abs(T - q[b]) for b in range(B)])
    want = ref["g_ent"][:B]
    excess = np.abs(out["g_ent"][:B].cpu().numpy().astype(np.float64) - want) - (2.0 ** -17 * terms + RTOL_F32 * np.abs(want).max())
    assert excess.max() <= 0, float(excess.max() / np.abs(want).max())


@pytest.mark.parametrize("dim,B,N", [(256, 5, 300), (400, 3, 1100)])
@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
def test_negative_gradients_of_distances_take_unrounded_sums(orc, dim, B, N, loss):
    """bf16 TransE, negatives far larger than the queries: a negative's gradient sum_b c_b q_b - (sum_b c_b) t has the rounding of its
    coefficients (one bf16, eight significand bits: up to 2^-8) on the queries alone; rounded coefficients in the sum would put it on
    the larger t."""
    import paper_2211_12281_amd as kge
    G = make_case("transe", 3000, 5, dim, B, N, True, amp=1.0)
    heads = np.unique(np.concatenate([G["h"], G["t"]]))
    G["ent"][heads] *= np.float32(2.0 ** -6)
    G["neg"] = np.where(np.isin(G["neg"], heads), (heads.max() + 1) % 3000, G["neg"]).astype(np.int32)
    G["neg"] = G["neg"][~np.isin(G["neg"], heads)]
    G["rel"][:] = 0.0
    kw = dict(n_ent_for_c=3000) if loss == "sampled_softmax" else dict(gamma=12.0, adv_temp=0.3)
    out = kge.loss_bwd(gpu_model("transe", G, True), loss, *(dev_idx(G[k]) for k in ("h", "r", "t", "neg")), loss_scale=1.0, **kw)
    ref = orc.loss_bwd("transe", loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], loss_scale=1.0, **kw)
    pos, S = orc.score_batch("transe", G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"])
    if loss == "sampled_softmax":
        z = np.concatenate([pos[:, None], S + np.log(2999 / len(G["neg"]))], axis=1)
        z = np.exp(z - z.max(axis=1, keepdims=True))
        c = z[:, 1:] / z.sum(axis=1, keepdims=True)
    else:
        w = np.exp(0.3 * (S - S.max(axis=1, keepdims=True)))
        c = w / w.sum(axis=1, keepdims=True) / (1.0 + np.exp(-(12.0 + S)))
    c = c / -S
    q, T = np.abs(G["ent"][G["h"]].astype(np.float64)), np.abs(G["ent"][G["neg"]].astype(np.float64))
    want = ref["g_ent"][2 * B:]
    bound = 2.0 ** -8 * (c.T @ q) + (2.0 ** -17 * c.sum(axis=0)[:, None]) * T + RTOL_F32 * np.abs(want)
    excess = np.abs(out["g_ent"][2 * B:].cpu().numpy().astype(np.float64) - want) / bound
    assert excess.max() <= 1.0, float(excess.max())


@pytest.mark.parametrize("scorer,dim,bf16", [("distmult", 64, False), ("complex", 256, True), ("distmult", 256, False), ("transe", 96, False)])
@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
def test_scores_too_large_for_an_exact_exponent(orc, scorer, dim, bf16, loss):
    """Scores of 1e10 to 1e15, where one rounding of the row's maximum is worth hundreds of units of the exponent: losses and gradients
    stay finite, and the loss is the oracle's."""
    import torch
    import paper_2211_12281_amd as kge
    G = make_case(scorer, 500, 5, dim, 70, 130, bf16, amp=0.5)
    G["ent"] *= np.float32(2.0 ** (40 if scorer == "transe" else 22))
    kw = dict(n_ent_for_c=500) if loss == "sampled_softmax" else dict(gamma=1.0, adv_temp=1.0)
    out = kge.loss_bwd(gpu_model(scorer, G, bf16), loss, *(dev_idx(G[k]) for k in ("h", "r", "t", "neg")), **kw)
    ref = orc.loss_bwd(scorer, loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], **kw)
    assert all(bool(torch.isfinite(v).all()) for v in out.values() if v is not None and v.is_floating_point())
    assert abs(out["loss"].item() - ref["loss"]) <= (RTOL_BF16 if bf16 else RTOL_F32) * abs(ref["loss"])


@pytest.fixture
def block_passes():
    import paper_2211_12281_amd as kge
    kge.debug_select("block_passes", True)
    try:
        yield
    finally:
        kge.debug_select("block_passes", False)


@pytest.mark.parametrize("scorer", base.SCORERS)
@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
@pytest.mark.parametrize("bf16", [False, True])
def test_block_kernels_match_oracle(orc, block_passes, scorer, loss, bf16):
    base.test_loss_and_gradients_match_oracle(orc, scorer, loss, bf16)


@pytest.mark.parametrize("scorer,dim,bf16", [("complex", 256, True), ("transe", 256, False), ("distmult", 128, False), ("rotate", 256, True),
                                             ("distmult", 32, False), ("complex", 512, True)])
def test_block_kernels_other_row_sizes(orc, block_passes, scorer, dim, bf16):
    base.test_other_row_sizes(orc, scorer, dim, bf16)


@pytest.mark.parametrize("scorer", base.SCORERS)
@pytest.mark.parametrize("bf16", [False, True])
def test_block_kernels_regulariser(orc, block_passes, scorer, bf16):
    base.test_l3_regulariser_matches_oracle(orc, scorer, bf16)


@pytest.mark.parametrize("scorer", ["transe", "complex"])
def test_block_kernels_edge_shapes(orc, block_passes, scorer):
    base.test_edge_shapes(orc, scorer)


@pytest.mark.parametrize("scorer,loss", base.WIDE_CASES)
def test_block_kernels_wide_score_range(orc, block_passes, scorer, loss):
    base.test_wide_score_range_raises_the_reference_repeatedly(orc, scorer, loss)


@pytest.mark.parametrize("scorer,loss", base.WIDE_BF16_CASES)
def test_block_kernels_wide_score_range_bf16(orc, block_passes, scorer, loss):
    base.test_wide_score_range_bf16_tables(orc, scorer, loss)


def test_block_kernels_repeated_calls(orc, block_passes):
    base.test_repeated_calls_are_bitwise_identical(orc)


@pytest.mark.parametrize("scorer,B,N", base.STORED_CASES)
def test_block_kernels_stored_weights(orc, block_passes, scorer, B, N):
    base.test_stored_weights_of_the_forward_pass_serve_the_pass_over_the_negatives(orc, scorer, B, N)


@pytest.mark.parametrize("scorer,dim,bf16,loss,B,N", base.DRAWN_CASES)
def test_block_kernels_drawn_negatives(block_passes, scorer, dim, bf16, loss, B, N):
    base.test_negatives_drawn_inside_the_call_equal_the_two_calls(scorer, dim, bf16, loss, B, N)


@pytest.mark.parametrize("scorer,dim,bf16,loss,B,N", base.PLANNED_CASES)
def test_block_kernels_planned_call(block_passes, scorer, dim, bf16, loss, B, N):
    base.test_planned_call_equals_the_sampled_call_followed_by_the_plans(scorer, dim, bf16, loss, B, N)


@pytest.mark.parametrize("scorer,dim,B,N", [("transh", 128, 129, 257), ("transh", 8, 31, 33), ("transe", 40, 1, 4000), ("rotate", 128, 300, 1),
                                            ("complex", 64, 130, 95), ("distmult", 120, 127, 161),
                                            ("transe", 256, 129, 257), ("rotate", 136, 31, 33), ("complex", 200, 1, 4000)])
@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
def test_block_kernels_on_planes(orc, block_passes, scorer, dim, B, N, loss):
    """fp32 rows, which the block kernels read as fp16 pieces: padding columns, a row more or less than a tile; the
    heads among the negatives and short relations, so that distances of the norm expansion cancel and are taken again from the rows."""
    G = make_case(scorer, 3000, 9, dim, B, N, False, amp=0.3 if scorer in ("distmult", "complex") else 0.1, zipf=True)
    if scorer in ("transe", "transh"):
        G["rel"] *= 0.03
        n = min(B, N // 2)
        G["neg"][:n] = G["h"][:n]
    kw = dict(n_ent_for_c=3000) if loss == "sampled_softmax" else dict(gamma=1.0, adv_temp=0.7)
    base._compare(orc, scorer, loss, G, False, 3000, kw=kw)


@pytest.mark.parametrize("scorer,dim,loss,B,N", [
    ("transh", 128, "logsigmoid", 1800, 1001), ("transh", 96, "sampled_softmax", 2040, 1300),          # splits of two tiles; three, the last with fewer
    ("transe", 256, "sampled_softmax", 1025, 2300), ("rotate", 200, "logsigmoid", 1281, 1537),         # three and two tiles
    ("complex", 136, "sampled_softmax", 600, 1500), ("distmult", 256, "logsigmoid", 2300, 1250)])      # two tiles and one; five and three
def test_block_kernels_on_planes_few_tiles(orc, block_passes, scorer, dim, loss, B, N):
    """Rows of 1,024 bytes and TransH, whose rounds work on two tiles at a time: splits that end after the first rounds, with rows that
    grow by a factor of 64 along the stream, so that the scales of a split's first tiles are lowered by those behind them."""
    G = make_case(scorer, 3000, 9, dim, B, N, False, amp=0.2 if scorer in ("distmult", "complex") else 0.1)
    G["neg"] = np.sort(G["neg"])
    G["ent"] *= (2.0 ** (np.arange(3000) / 500.0 - 5.0)).astype(np.float32)[:, None]
    kw = dict(n_ent_for_c=3000) if loss == "sampled_softmax" else dict(gamma=1.0, adv_temp=0.7)
    base._compare(orc, scorer, loss, G, False, 3000, kw=kw)


@pytest.mark.parametrize("scorer,bf16", [("transh", False), ("rotate", True), ("complex", False), ("transe", True), ("distmult", False)])
@pytest.mark.parametrize("dim", [64, 128, 144, 256, 272])
@pytest.mark.parametrize("N", [50, 2100])
def test_columns_per_lane_of_the_row_kernels(orc, scorer, bf16, dim, N):
    """Widths on both sides of the lines between the row kernels for 128, 256 and 512 columns, with few and with many splits."""
    dim = dim if bf16 or dim <= 256 else 240               # (fp32 rows end at 256 columns)
    G = make_case(scorer, 3000, 9, dim, 37, N, bf16, amp=0.3 if scorer in ("distmult", "complex") else 0.1, zipf=True)
    base._compare(orc, scorer, "logsigmoid", G, bf16, 3000, kw=dict(gamma=1.0, adv_temp=0.7, reg_l3=1e-3))


@pytest.mark.parametrize("scorer,dim,bf16,p_norm,B,N,n_ent", [
    ("transe", 64, True, 2, 1, 1, 50), ("distmult", 64, False, 2, 257, 2051, 4000),        # rows beyond the last group of four, beyond the eight scores a thread keeps
    ("rotate", 128, True, 1, 130, 300, 900), ("transh", 64, False, 1, 67, 95, 300),        # 1-norm; without coefficients
    ("transe", 32, True, 1, 70, 33_000, 60_000)])                                          # entity ids for the radix passes: the rows have their own launch
def test_row_pass_beside_the_sorts(scorer, dim, bf16, p_norm, B, N, n_ent):
    """kge_loss_bwd_sampled_planned on score blocks in memory against the call and its plans: bit for bit, plans as updates."""
    import kge_synth as ks
    import paper_2211_12281_amd as kge
    g = torch.Generator(device="cuda").manual_seed(B + N)
    dt = torch.bfloat16 if bf16 else torch.float32
    rows = lambda n, d: (torch.randn((n, d), generator=g, device="cuda") * 0.3).to(dt)
    k_rel = dim // 2 if scorer == "rotate" else dim
    model = kge.Model(scorer, rows(n_ent, dim), rows(9, k_rel), rows(9, dim) if scorer == "transh" else None, p_norm=p_norm)
    draw_ids = lambda n, size: torch.randint(0, n, (size,), generator=g, device="cuda", dtype=torch.int32)
    h, r, t = draw_ids(n_ent, B), draw_ids(9, B), draw_ids(n_ent, B)
    res = []
    for planned in (False, True):
        ids = torch.cat([h, t, torch.full((N,), -1, dtype=torch.int32, device="cuda")])
        ws = (kge.Workspace(), kge.Workspace())
        plans = [(n_ent, dim, ids, ws[0]), (9, k_rel, r, ws[1])]
        kw = dict(gamma=6.0, adv_temp=1.0, n_ent_for_c=n_ent, draw=(ks.BASE_SEED, 3, ks.TAG_NEG, 0, n_ent))
        out = kge.loss_bwd(model, "logsigmoid", h, r, t, ids[2 * B:], plans=plans if planned else None, **kw)
        if not planned:
            kge.sparse_adam_plan_tables(plans)
        st = [torch.zeros((n, d), device="cuda") for n, d in ((n_ent, dim), (9, k_rel)) for _ in range(3)]
        kge.sparse_adam_apply_tables([(st[0], None, st[1], st[2], out["g_ent"], ws[0]), (st[3], None, st[4], st[5], out["g_rel"], ws[1])],
                                     1e-2, step=2)
        torch.cuda.synchronize()
        res.append([x for x in out.values() if x is not None] + [ids] + st)
    for a, b in zip(*res):
        assert torch.equal(a, b)
    assert bool((res[0][-1] != 0).any())


@pytest.mark.parametrize("scorer,dim,loss,order", [
    ("transe", 128, "logsigmoid", -1), ("transe", 256, "sampled_softmax", -1), ("rotate", 256, "logsigmoid", 1), ("rotate", 64, "sampled_softmax", -1),
    ("transh", 128, "logsigmoid", -1), ("transh", 64, "sampled_softmax", 1), ("distmult", 256, "logsigmoid", 1), ("complex", 128, "sampled_softmax", -1),
    ("distmult", 200, "sampled_softmax", 1)])
def test_block_kernels_on_planes_with_rows_of_all_sizes(orc, block_passes, scorer, dim, loss, order):
    """Every row of the planes has a scale of its own, and so have the coefficients of an own row: negatives between 2^-40 and 4 times
    the usual size, the largest first (the coefficients of a distance scorer, weight over distance times row scale, then grow 2^42-fold along
    the pass: what is accumulated is rescaled again and again) or last (the first tile sets a scale that later ones don't reach); heads
    and tails likewise, so that the pass over the negatives meets the same."""
    G = make_case(scorer, 6000, 9, dim, 300, 700, False, amp=0.3 if scorer in ("distmult", "complex") else 0.1)
    used = np.unique(np.concatenate([G["h"], G["t"], G["neg"]]))
    size = np.float32(2.0) ** np.linspace(-40, 2, len(used)).round().astype(np.float32)
    G["ent"][used] *= size[:, None]
    of = dict(zip(used.tolist(), size.tolist()))
    G["neg"] = np.array(sorted(G["neg"].tolist(), key=lambda i: order * of[i]), dtype=np.int32)
    at = np.array(sorted(range(len(G["h"])), key=lambda b: order * of[int(G["h"][b])]))
    for k in ("h", "r", "t"):
        G[k] = np.ascontiguousarray(G[k][at])
    base._compare(orc, scorer, loss, G, False, 6000)


@pytest.mark.parametrize("scorer,dim", [("transe", 128), ("rotate", 64), ("rotate", 256)])
def test_block_kernels_on_planes_of_tiny_rows(orc, block_passes, scorer, dim):
    """Rows whose largest element lies below 2^-64: the product of two rows' scales is no fp32 number, their dot product and their
    squared norms (2^-124) are."""
    G = make_case(scorer, 3000, 9, dim, 130, 300, False, amp=0.5)
    G["neg"] = np.setdiff1d(np.arange(3000, dtype=np.int32), np.concatenate([G["h"], G["t"]]))[:300].copy()    # (squares of r alone are 0)
    G["ent"] *= np.float32(2.0 ** -64.6 / np.abs(G["ent"]).max())
    if scorer == "transe":
        G["rel"] *= np.float32(2.0 ** -76)
    base._compare(orc, scorer, "logsigmoid", G, False, 3000, kw=dict(gamma=1.0, adv_temp=1.0))


@pytest.mark.parametrize("scorer", ["distmult", "complex"])
@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
@pytest.mark.parametrize("dim", [128, 256])
def test_block_kernels_on_planes_keep_a_loss_beside_a_score_of_minus_infinity(orc, block_passes, scorer, loss, dim):
    """A negative with an infinite element, whose score is -inf for every query, weighs nothing: the loss and all gradients are those
    of a negative with -1e30 in its place."""
    import paper_2211_12281_amd as kge
    G = make_case(scorer, 3000, 9, dim, 140, 300, False, amp=0.3)
    G["neg"] = np.setdiff1d(np.arange(3000, dtype=np.int32), np.concatenate([G["h"], G["t"]]))[:300].copy()
    G["ent"][G["h"], 3] = 0.25                              # (q_3 > 0 for both scorers)
    G["rel"][:, 3] = 0.25
    if scorer == "complex":
        G["ent"][G["h"], dim // 2 + 3] = 0.0
    G["ent"][G["neg"][77], 3] = -1e30
    kw = dict(n_ent_for_c=3000) if loss == "sampled_softmax" else dict(gamma=0.0, adv_temp=1.0)
    ref = orc.loss_bwd(scorer, loss, G["ent"], G["rel"], G["relw"], G["h"], G["r"], G["t"], G["neg"], **kw)
    G["ent"][G["neg"][77], 3] = -np.inf
    out = kge.loss_bwd(gpu_model(scorer, G, False), loss, dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]), **kw)
    assert abs(out["loss"].item() - ref["loss"]) <= RTOL_F32 * abs(ref["loss"])
    for k in ("g_ent", "g_rel"):
        assert norm_err(out[k].cpu().numpy(), ref[k]) <= RTOL_F32


@pytest.mark.parametrize("scorer,dim,loss", [("distmult", 128, "logsigmoid"), ("distmult", 256, "sampled_softmax"), ("complex", 64, "sampled_softmax"),
                                             ("complex", 256, "logsigmoid"), ("transe", 128, "logsigmoid")])
def test_block_kernels_on_planes_with_columns_of_all_sizes(orc, block_passes, scorer, dim, loss):
    """Columns between 2^0 and 2^-20 of the rows' largest elements, each compared by itself.  An element keeps 2^-24 of itself or 2^-40 of
    the largest: 2^-20 = 1e-6 for the smallest column.  A column's sum over 300 or 700 pairs of either sign is down to a fortieth of its
    terms' size (the same calls leave up to 4.1e-5 where every element keeps 24 bits): 1e-4."""
    import paper_2211_12281_amd as kge
    G = make_case(scorer, 6000, 9, dim, 300, 700, False, amp=0.3 if scorer in ("distmult", "complex") else 0.1)
    half = dim // 2 if scorer == "complex" else dim
    size = np.float32(2.0) ** -np.round(np.arange(half) * 20 / (half - 1)).astype(np.float32)
    G["ent"] *= np.concatenate([size] * (dim // half))
    kw = base._kw(scorer, loss, 6000)
    ref = orc.loss_bwd(scorer, loss, G["ent"], G["rel"], G["relw"], G["h"], G["r"], G["t"], G["neg"], **kw)
    out = kge.loss_bwd(gpu_model(scorer, G, False), loss, dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]), **kw)
    got, want = out["g_ent"].cpu().numpy().astype(np.float64), ref["g_ent"]
    for sl in (slice(0, 300), slice(600, 1300)):
        err = np.linalg.norm(got[sl] - want[sl], axis=0) / np.linalg.norm(want[sl], axis=0)
        assert err.max() <= 1e-4, (sl, int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("top", [30.0, 39.0, 45.0, 120.0])
@pytest.mark.parametrize("loss,dim", [("sampled_softmax", 64), ("logsigmoid", 128), ("sampled_softmax", 256)])
def test_block_kernels_on_planes_when_later_small_rows_outweigh_large_ones(orc, block_passes, loss, dim, top):
    """Of every four tiles of negatives the first holds rows of 2^30 with scores of about -top, the others rows of 1 with scores of about
    top: the reference rises by 2^90 (top 30) after the first tile, and the scale of the coefficients, set for 2^30 times theirs, with
    it, or ends where it would pass 2^126 (some rows at 39, all above).  The large elements lie where the queries are zero; the other columns are compared."""
    import paper_2211_12281_amd as kge
    B, N, half = 4096, 1600, dim // 2
    g = np.random.default_rng(dim)
    ent = np.zeros((B + N + 10, dim), dtype=np.float32)
    ent[:B, :half] = g.uniform(0.5, 1.5, (B, half))
    sign = np.where(np.arange(N) % 128 < 32, -1.0, 1.0)[:, None]
    ent[B:B + N, :half] = sign * top / half * g.uniform(0.9, 1.1, (N, half))
    ent[B:B + N, half:] = np.where(sign < 0, 2.0 ** 30, 1.0) * g.uniform(-1, 1, (N, half))
    G = dict(ent=ent, rel=np.ones((3, dim), dtype=np.float32), relw=None, h=np.arange(B, dtype=np.int32), r=(np.arange(B) % 3).astype(np.int32),
             t=np.full(B, B + N, dtype=np.int32), neg=np.arange(B, B + N, dtype=np.int32))
    kw = dict(n_ent_for_c=len(ent)) if loss == "sampled_softmax" else dict(gamma=1.0, adv_temp=1.0)
    ref = orc.loss_bwd("distmult", loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], **kw)
    out = kge.loss_bwd(gpu_model("distmult", G, False), loss, dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]), **kw)
    assert abs(out["loss"].item() - ref["loss"]) <= RTOL_F32 * abs(ref["loss"])
    got, want = out["g_ent"].cpu().numpy()[:B, :half], ref["g_ent"][:B, :half]
    assert norm_err(got, want) <= 2 * RTOL_F32


@pytest.mark.parametrize("scorer,dim,B,N,size", [("complex", 8, 2600, 2700, 42469632), ("transh", 48, 1500, 2700, 59421952),
                                                 ("distmult", 128, 2600, 2700, 42469632), ("transe", 64, 4096, 4096, 45869312)])
def test_block_kernels_on_planes_in_a_smaller_workspace(orc, scorer, dim, B, N, size):
    """Two workgroups share a compute unit, so these calls would like up to twice the split partials that one needs; in a workspace sized for
    those they run with fewer splits, in one of a third with fewer still, and one without room for a split each is refused."""
    import paper_2211_12281_amd as kge
    class Fixed:
        def __init__(self, n): self.buf = torch.empty(n, dtype=torch.uint8, device="cuda")
        def get(self, n): return self.buf
    G = make_case(scorer, 9000, 9, dim, B, N, False, amp=0.3 if scorer in ("distmult", "complex") else 0.1, zipf=True)
    model, kw = gpu_model(scorer, G, False), dict(gamma=1.0, adv_temp=0.8)
    args = (dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]))
    run = lambda ws: {k: v.clone() for k, v in kge.loss_bwd(model, "logsigmoid", *args, ws=ws, **kw).items() if v is not None}
    want = run(kge.Workspace())
    for n in (size, size // 3):
        buf = Fixed(n + (1 << 20))
        buf.buf[n:] = 77
        buf.buf, guard = buf.buf[:n], buf.buf[n:]
        got = run(buf)
        assert bool((guard == 77).all())
        assert abs(got["loss"].item() - want["loss"].item()) <= 1e-6 * abs(want["loss"].item())
        for k in ("g_ent", "g_rel"):
            assert norm_err(got[k].cpu().numpy(), want[k].cpu().numpy()) <= RTOL_F32
    with pytest.raises(RuntimeError):
        run(Fixed(1 << 20))
