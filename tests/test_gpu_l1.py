"""The 1-norm variants of TransE, RotatE and TransH on the GPU (kge_score, kge_loss_bwd with p_norm = 1) against the
oracle.  The gradient of a 1-norm is discontinuous where a coordinate of h + r - t crosses zero, so the TransE
cases put the tables on a binary grid on which every sum and difference is exact in fp32 and in bf16 (no sign can
differ between the two implementations; with the relations on the same grid the micro-batch is full of exact ties,
which must give the sub-gradient 0).  RotatE goes through sin / cos and TransH through projections, where a sign may
flip for a coordinate within fp32 rounding of zero: there every outlying gradient element must be explained from the
oracle's side by such a coordinate (helpers.l1_sign_flips_justified)."""
import numpy as np
import pytest

import kge_synth as ks
from helpers import RTOL_BF16, RTOL_F32, dev_idx, l1_sign_flips_justified, norm_err, small_graph, to_dev

pytestmark = pytest.mark.gpu


def _grid_case(scorer, n_ent, n_rel, dim, B, N, ties, seed=ks.BASE_SEED):
    G = small_graph(scorer, n_ent, n_rel, dim, B, N, seed=seed, amp=0.5)
    G["ent"] = (np.round(G["ent"] * 64) / 64).astype(np.float32)
    if scorer == "transe":
        # off the entities' grid by half a step: no coordinate of h + r - t can be zero
        G["rel"] = (np.round(G["rel"] * 64) / 64 + (0.0 if ties else 1.0 / 128)).astype(np.float32)
    z = ks.ZipfIds(n_ent, 1.1)
    g = ks.rng(seed, ks.TAG_BATCH, 1)
    G["h"], G["t"] = z.draw(g, B), z.draw(g, B)
    return G


def _model(scorer, G, bf16):
    import paper_2211_12281_amd as kge
    return kge.Model(scorer, to_dev(G["ent"], bf16), to_dev(G["rel"], bf16), None, p_norm=1)


def _outliers(x, ref, tol):
    e = np.abs(np.asarray(x, np.float64) - ref) / max(float(np.max(np.abs(ref))), 1e-300)
    return int(np.sum(e > tol)), float(e.max()) if e.size else 0.0


def _compare(orc, scorer, loss, G, bf16, n_ent, kw):
    import paper_2211_12281_amd as kge
    out = kge.loss_bwd(_model(scorer, G, bf16), loss, dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]), **kw)
    ref = orc.loss_bwd(scorer + "_l1", loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], **kw)
    tol = RTOL_BF16 if bf16 else RTOL_F32
    assert abs(out["loss"].item() - ref["loss"]) <= tol * abs(ref["loss"])
    B, N = len(G["h"]), len(G["neg"])
    ge = out["g_ent"].cpu().numpy()
    total = 0
    for name, x, r in (("g_head", ge[:B], ref["g_ent"][:B]), ("g_tail", ge[B:2 * B], ref["g_ent"][B:2 * B]),
                       ("g_neg", ge[2 * B:], ref["g_ent"][2 * B:]), ("g_rel", out["g_rel"].cpu().numpy(), ref["g_rel"])):
        if r.size == 0:
            continue
        bad, worst = _outliers(x, r, tol)
        total += bad
        assert bad == 0, (name, bad, worst)               # exact grids: no sign can differ
    assert np.array_equal(out["g_ent_idx"].cpu().numpy(), ref["g_ent_idx"])
    assert np.array_equal(out["g_rel_idx"].cpu().numpy(), ref["g_rel_idx"])
    return total


@pytest.mark.parametrize("scorer", ["transe", "rotate"])
@pytest.mark.parametrize("bf16", [False, True])
def test_scores_match_oracle(orc, scorer, bf16):
    import paper_2211_12281_amd as kge
    for (B, N, dim) in [(70, 300, 32), (257, 1000, 208)]:
        G = small_graph(scorer, 3000, 9, dim, B, N, amp=0.3)
        if bf16:
            G["ent"], G["rel"] = ks.round_to_bf16(G["ent"]), ks.round_to_bf16(G["rel"])
        pos, neg = kge.score(_model(scorer, G, bf16), dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]))
        rp, rn = orc.score_batch(scorer + "_l1", G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"])
        # the arithmetic is fp32 also for bf16 tables (the query is not rounded to the table type)
        assert norm_err(pos.cpu().numpy(), rp) <= RTOL_F32
        assert norm_err(neg.cpu().numpy(), rn) <= RTOL_F32


@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("ties", [False, True])
def test_transe_loss_and_gradients(orc, loss, bf16, ties):
    G = _grid_case("transe", 4000, 12, 64, 200, 333, ties)
    kw = dict(n_ent_for_c=4000) if loss == "sampled_softmax" else dict(gamma=6.0, adv_temp=0.5)
    _compare(orc, "transe", loss, G, bf16, 4000, kw)
    if ties:
        # the case is only worth its name if exact ties are frequent
        q = G["ent"][G["h"]] + G["rel"][G["r"]]
        assert np.mean(q[:, None, :] == G["ent"][G["neg"]][None, :, :]) > 0.005


@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
@pytest.mark.parametrize("bf16", [False, True])
def test_rotate_loss_and_gradients(orc, loss, bf16):
    G = small_graph("rotate", 4000, 12, 64, 200, 333, amp=0.3)
    if bf16:
        G["ent"], G["rel"] = ks.round_to_bf16(G["ent"]), ks.round_to_bf16(G["rel"])
    kw = dict(n_ent_for_c=4000) if loss == "sampled_softmax" else dict(gamma=8.0, adv_temp=0.3)
    # the arithmetic is fp32 for both table types: fp32 tolerance; a sign may differ only where the oracle finds a
    # coordinate within rounding of zero
    import paper_2211_12281_amd as kge
    out = kge.loss_bwd(_model("rotate", G, bf16), loss, dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]), **kw)
    ref = orc.loss_bwd("rotate_l1", loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], **kw)
    assert abs(out["loss"].item() - ref["loss"]) <= RTOL_F32 * abs(ref["loss"])
    got = {k2: out[k2].cpu().numpy() for k2 in ("g_ent", "g_rel")}
    flips = l1_sign_flips_justified(orc, "rotate", loss, G["ent"], G["rel"], None, G["h"], G["r"], G["t"], G["neg"], kw, got, ref, 2e-5)
    assert flips <= 1e-4 * (got["g_ent"].size + got["g_rel"].size)


@pytest.mark.parametrize("dim,bf16", [(128, False), (256, True), (512, True), (32, False)])
def test_other_row_sizes_and_shapes(orc, dim, bf16):
    for (B, N) in [(150, 260), (1, 1), (3, 0), (130, 1), (1, 130)]:
        G = _grid_case("transe", 3000, 9, dim, B, N, False)
        _compare(orc, "transe", "sampled_softmax", G, bf16, 3000, dict(n_ent_for_c=3000))
        # the margin follows the typical distance (about 0.35 per coordinate on this grid), else sigma(gamma + s)
        # underflows in fp32 for the long rows
        _compare(orc, "transe", "logsigmoid", G, bf16, 3000, dict(gamma=0.35 * dim, adv_temp=0.2, loss_scale=0.37))


@pytest.mark.parametrize("dim,bf16,B,N", [
    (72, False, 1440, 1473), (64, True, 1408, 1472),     # score tiles of 64 queries (the sizes above take tiles of 32) and the last of the others
    (136, False, 257, 1300),                             # columns past the row in its last tile; rows past the block in its last tiles
    (48, True, 33, 256), (64, False, 97, 511),           # tiles of 48 negatives whose last reaches past the padded rows
    (64, False, 480, 1024),                              # 330 workgroups of 48 negatives against 240 of 64: the tile of 64 has less to do
    (32, True, 1024, 40), (32, True, 1025, 40)])         # four waves per row in the chain rule, and one
def test_tiles_and_their_edges(orc, dim, bf16, B, N):
    G = _grid_case("transe", 3000, 9, dim, B, N, False)
    _compare(orc, "transe", "sampled_softmax", G, bf16, 3000, dict(n_ent_for_c=3000))
    _compare(orc, "transe", "logsigmoid", G, bf16, 3000, dict(gamma=0.35 * dim, adv_temp=0.2, loss_scale=0.37))


@pytest.mark.parametrize("dim,bf16,B,N", [
    (32, False, 31, 63), (72, False, 33, 65), (144, True, 64, 16), (64, True, 1, 17),      # edges of a chunk of queries and of a wave's negatives
    (256, False, 321, 1025),                             # the last wave, the last block and the last chunk with one row each
    (136, False, 2050, 700),                             # several chunks to a split, a last split with fewer
    (336, True, 1024, 2048), (272, True, 1100, 2048),    # two blocks of negatives to a group, four chunks to each; the two passes
    (272, True, 1024, 2048),                             # too few workgroups for eight rounds
    (192, False, 311, 5439), (64, True, 383, 5285)])     # four rounds with enough of them, and without
def test_both_gradients_from_one_sign(orc, dim, bf16, B, N):
    G = _grid_case("transe", 3000, 9, dim, B, N, True)   # (with ties: sign(0) = 0 on either side)
    _compare(orc, "transe", "sampled_softmax", G, bf16, 3000, dict(n_ent_for_c=3000))


def test_half_the_columns_take_less_time():
    """2,048 x 2,048 at 64 columns is a quarter of the workgroups of 256: a walk of eight rounds in each would take nearly the time of 128."""
    import torch
    import paper_2211_12281_amd as kge
    ms = []
    for dim in (64, 128):
        G = _grid_case("transe", 3000, 9, dim, 2048, 2048, False)
        model = _model("transe", G, True)
        args = [model, "logsigmoid", dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"])]
        ws, best = kge.Workspace(), 1e9
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(10):
                kge.loss_bwd(*args, gamma=0.35 * dim, adv_temp=0.5, ws=ws)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) / 10)
        ms.append(best)
    assert ms[0] < 0.8 * ms[1], ms


def test_regulariser_and_repeatability(orc):
    import paper_2211_12281_amd as kge
    G = _grid_case("transe", 2000, 5, 64, 96, 200, True)
    kw = dict(n_ent_for_c=2000, reg_l3=1e-2)
    _compare(orc, "transe", "sampled_softmax", G, False, 2000, kw)
    m = _model("transe", G, False)
    args = (dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]))
    a = {k: v.clone() for k, v in kge.loss_bwd(m, "sampled_softmax", *args, **kw).items() if v is not None}
    b = kge.loss_bwd(m, "sampled_softmax", *args, **kw)
    for k in a:
        assert bool((a[k] == b[k]).all()), k


def _transh_model(G, bf16):
    import paper_2211_12281_amd as kge
    return kge.Model("transh", to_dev(G["ent"], bf16), to_dev(G["rel"], bf16), to_dev(G["relw"], bf16), p_norm=1)


def _transh_case(n_ent, n_rel, dim, B, N, bf16):
    G = small_graph("transh", n_ent, n_rel, dim, B, N, amp=0.3)
    if bf16:
        for k in ("ent", "rel", "relw"):
            G[k] = ks.round_to_bf16(G[k])
    return G


@pytest.mark.parametrize("bf16", [False, True])
def test_transh_scores_match_oracle(orc, bf16):
    import paper_2211_12281_amd as kge
    for (B, N, dim) in [(70, 300, 32), (257, 1000, 208), (5, 1, 512 if bf16 else 256)]:
        G = _transh_case(3000, 9, dim, B, N, bf16)
        pos, neg = kge.score(_transh_model(G, bf16), dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]))
        rp, rn = orc.score_batch("transh_l1", G["ent"], G["rel"], G["relw"], G["h"], G["r"], G["t"], G["neg"])
        assert norm_err(pos.cpu().numpy(), rp) <= RTOL_F32          # fp32 arithmetic on unrounded q' and w^
        assert norm_err(neg.cpu().numpy(), rn) <= RTOL_F32


@pytest.mark.parametrize("loss", ["logsigmoid", "sampled_softmax"])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("shape", [(200, 333, 64), (130, 70, 208), (1, 1, 32), (3, 0, 32), (65, 129, 128)])
def test_transh_loss_and_gradients(orc, loss, bf16, shape):
    """TransH with the 1-norm: the normalisation of w and the projections make exact grids impossible, so a sign may
    flip for a coordinate within rounding of zero: every outlying gradient element must be explained by such a coordinate."""
    import paper_2211_12281_amd as kge
    B, N, dim = shape
    G = _transh_case(4000, 12, dim, B, N, bf16)
    kw = dict(n_ent_for_c=4000) if loss == "sampled_softmax" else dict(gamma=0.12 * dim, adv_temp=0.3)
    out = kge.loss_bwd(_transh_model(G, bf16), loss, dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]), **kw)
    ref = orc.loss_bwd("transh_l1", loss, G["ent"], G["rel"], G["relw"], G["h"], G["r"], G["t"], G["neg"], **kw)
    assert abs(out["loss"].item() - ref["loss"]) <= RTOL_F32 * abs(ref["loss"])
    got = {k2: out[k2].cpu().numpy() for k2 in ("g_ent", "g_rel", "g_relw")}
    flips = l1_sign_flips_justified(orc, "transh", loss, G["ent"], G["rel"], G["relw"], G["h"], G["r"], G["t"], G["neg"], kw, got, ref, 2e-5)
    assert flips <= 1e-3 * sum(v.size for v in got.values()) + 8
    assert np.array_equal(out["g_ent_idx"].cpu().numpy(), ref["g_ent_idx"])
    assert np.array_equal(out["g_rel_idx"].cpu().numpy(), ref["g_rel_idx"])


def test_transh_one_norm_repeatable_with_regulariser(orc):
    import paper_2211_12281_amd as kge
    G = _transh_case(2000, 5, 64, 96, 200, False)
    kw = dict(n_ent_for_c=2000, reg_l3=1e-2)
    m = _transh_model(G, False)
    args = (dev_idx(G["h"]), dev_idx(G["r"]), dev_idx(G["t"]), dev_idx(G["neg"]))
    a = {k: v.clone() for k, v in kge.loss_bwd(m, "sampled_softmax", *args, **kw).items() if v is not None}
    b = kge.loss_bwd(m, "sampled_softmax", *args, **kw)
    for k in a:
        assert bool((a[k] == b[k]).all()), k
    ref = orc.loss_bwd("transh_l1", "sampled_softmax", G["ent"], G["rel"], G["relw"], G["h"], G["r"], G["t"], G["neg"], **kw)
    assert abs(a["loss"].item() - ref["loss"]) <= RTOL_F32 * abs(ref["loss"])
