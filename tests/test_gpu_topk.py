"""kge_topk and kge_partition_triples against the oracle: indices bit-exact, scores within tolerance."""
import numpy as np
import pytest
import torch

import kge_synth as ks
from helpers import RTOL_BF16, RTOL_F32, dev_idx, gpu_model, make_case, norm_err, rank_band_eps, small_graph, to_dev

pytestmark = pytest.mark.gpu


def _check(orc, scorer, G, bf16, lo, hi, K, true_t=None):
    import paper_2211_12281_amd as kge
    model = gpu_model(scorer, G, bf16)
    tt = None if true_t is None else dev_idx(true_t)
    idx, sc, rank = kge.topk(model, dev_idx(G["h"]), dev_idx(G["r"]), lo, hi, K, tt)
    relw = G.get("relw")
    ridx, rsc, rrank = orc.topk(scorer, G["ent"], G["rel"], relw, G["h"], G["r"], lo, hi, K, true_t)
    idx, sc = idx.cpu().numpy(), sc.cpu().numpy()
    if scorer in ("rotate", "transh") and not np.array_equal(idx, ridx):
        # the key passes through cos / sin in fp64, whose last bit belongs to the math library (TransH: through the
        # normalisation of w and two fp64 dot products whose summation order is the implementation's): two candidates
        # whose keys agree to 1e-12 may legitimately swap places; anything else must be identical
        for (q, i) in np.argwhere(idx != ridx):
            one = slice(q, q + 1)
            _, s = orc.score_batch(scorer, G["ent"], G["rel"], relw, G["h"][one], G["r"][one], G["h"][one], idx[q, i:i + 1])
            assert abs(s[0, 0] - rsc[q, i]) <= 1e-12 * max(abs(rsc[q, i]), 1e-30), (q, i)
    else:
        assert np.array_equal(idx, ridx), np.argwhere(idx != ridx)[:5]
    fin = np.isfinite(rsc)
    assert np.array_equal(np.isfinite(sc), fin)
    if fin.any():
        assert np.max(np.abs(sc[fin] - rsc[fin])) <= RTOL_F32 * np.max(np.abs(rsc[fin]))   # fp64 key, rounded to fp32 once
    if true_t is not None:
        rank = rank.cpu().numpy()
        n = min(K, hi - lo)
        inside = rrank <= n
        assert np.array_equal(rank[inside], rrank[inside])          # exact whenever the tail is in the list
        assert np.all(rank[~inside] > n)
        # beyond the list the rank is counted with matrix-core values: it may differ from the exact rank by at most the
        # number of candidates whose exact key lies inside the error band of those values around the true tail's key,
        # which the oracle counts in the same pass
        if (~inside).any() and hi > lo:
            t_max = float(np.max(np.linalg.norm(G["ent"][lo:hi].astype(np.float64), axis=1)))
            eps = rank_band_eps(scorer, G["ent"][G["h"]], G["rel"][G["r"]], None if relw is None else relw[G["r"]], bf16, t_max)
            _, _, rrank2, band = orc.topk_band(scorer, G["ent"], G["rel"], relw, G["h"], G["r"], lo, hi, K, true_t, eps)
            assert np.array_equal(rrank2, rrank)
            assert np.all(np.abs(rank[~inside] - rrank[~inside]) <= band[~inside])


@pytest.mark.parametrize("scorer", ["distmult", "transe", "complex", "rotate", "transh"])
@pytest.mark.parametrize("bf16", [False, True])
def test_full_ranking_small_graph(orc, scorer, bf16):
    """64 queries over all 1,000 entities, K = 100 (the tiny configuration's brute-force ranking)."""
    G = small_graph(scorer, 1000, 10, 32, 64, 0, normal=True)
    if bf16:
        G["ent"], G["rel"] = ks.round_to_bf16(G["ent"]), ks.round_to_bf16(G["rel"])
        if G["relw"] is not None:
            G["relw"] = ks.round_to_bf16(G["relw"])
    _check(orc, scorer, G, bf16, 0, 1000, 100, G["t"])


@pytest.mark.parametrize("scorer,bf16,dim", [("distmult", True, 256), ("transe", True, 256), ("distmult", False, 64),
                                             ("transe", False, 128), ("distmult", True, 512), ("transe", False, 256),
                                             ("complex", True, 256), ("rotate", True, 256), ("complex", False, 72),
                                             ("rotate", False, 128), ("complex", True, 512), ("rotate", True, 48),
                                             ("transh", True, 256), ("transh", False, 128), ("transh", True, 80),
                                             ("transh", False, 24)])
def test_many_candidates_several_chunks(orc, scorer, bf16, dim):
    G = make_case(scorer, 60000, 20, dim, 300, 0, bf16)
    true_t = ks.uniform_ids(ks.rng(3, ks.TAG_HELDOUT), 0, 60000, 300)
    _check(orc, scorer, G, bf16, 0, 60000, 100, true_t)


@pytest.mark.parametrize("scorer,bf16,dim,Q", [
    ("transe", True, 256, 128), ("transe", True, 208, 129), ("rotate", False, 128, 512), ("transe", True, 256, 513),
    ("distmult", True, 256, 512), ("complex", False, 64, 513),        # one / two blocks of queries per wave
    ("transe", True, 512, 512), ("rotate", False, 256, 513),          # rows over 512 bytes: norms inside / outside the scan
    ("distmult", True, 400, 130),
    ("transh", True, 64, 3072), ("transh", False, 32, 3073)])         # ... TransH
def test_query_counts_around_the_scan_variants(orc, scorer, bf16, dim, Q):
    n = 2000 if Q > 1000 else 5003                                     # (two chunks and a ragged last tile)
    G = make_case(scorer, n, 7, dim, Q, 0, bf16)
    _check(orc, scorer, G, bf16, 1, n, 20, ks.uniform_ids(ks.rng(4, ks.TAG_HELDOUT), 0, n, Q))


# few queries: all candidates appended in one chunk and a sampled threshold (4,096 rows and one more), and larger tables
@pytest.mark.parametrize("n", [4096, 4097, 40960, 40961, 409601])
@pytest.mark.parametrize("K", [5, 100])
def test_few_queries_with_fast_growing_chunks(orc, n, K):
    G = make_case("transe", n, 5, 16, 3, 0, False)
    _check(orc, "transe", G, False, 0, n, K, ks.uniform_ids(ks.rng(6, ks.TAG_HELDOUT), 0, n, 3))


@pytest.mark.parametrize("Q,dim,bf16,K,n", [
    (3, 16, False, 5, 16416), (3, 16, False, 5, 16417),                # one tile behind a maximum of the sample, and two
    (3, 16, False, 5, 20000), (3, 16, False, 5, 20001),                # four maxima per lane and group, and one
    (3, 16, False, 5, 65568), (3, 16, False, 5, 65569), (3, 16, False, 5, 131393),       # ... behind one, two and three tiles
    (3, 16, False, 100, 1_053_900), (3, 16, False, 100, 1_054_500),    # one chunk behind the sample, and two
    (8200, 16, True, 5, 148_500), (8200, 16, True, 5, 148_800),        # the same with 32 splits
    (8200, 16, True, 5, 436_000), (8200, 16, True, 5, 436_800),        # two and three
    (8200, 16, True, 5, 463_200), (8200, 16, True, 5, 463_800),        # three in order of the ids, and in strides
    (8200, 16, True, 256, 277_300), (8200, 16, True, 256, 277_900)])   # two, the same
def test_edges_of_the_stages(orc, Q, dim, bf16, K, n):
    """Sizes on both sides of the lines between the forms of a call; 24 of the queries against the oracle."""
    import paper_2211_12281_amd as kge
    G = make_case("distmult", n, 5, dim, Q, 0, bf16)
    true_t = ks.uniform_ids(ks.rng(6, ks.TAG_HELDOUT), 0, n, Q)
    idx, sc, rank = (v.cpu().numpy() for v in kge.topk(gpu_model("distmult", G, bf16), dev_idx(G["h"]), dev_idx(G["r"]), 0, n, K, dev_idx(true_t)))
    some = np.unique(np.linspace(0, Q - 1, 24).astype(int))
    ridx, rsc, rrank = orc.topk("distmult", G["ent"], G["rel"], None, G["h"][some], G["r"][some], 0, n, K, true_t[some])
    assert np.array_equal(idx[some], ridx)
    assert np.max(np.abs(sc[some] - rsc)) <= RTOL_F32 * np.max(np.abs(rsc))
    inside = rrank <= K
    assert np.array_equal(rank[some][inside], rrank[inside]) and np.all(rank[some][~inside] > K)


def test_clusters_of_neighbouring_rows_overflow_no_append_area():
    """A table whose rows come in clusters of 50 that are alike, as one sorted by community has them: the winners of a query are neighbours
    and land in few append areas.  A query whose area overflows is ranked exhaustively, which takes a hundred times as long as the scan, so
    the call's time beside that of the same rows in any order shows whether one did."""
    import paper_2211_12281_amd as kge
    n, d, Q, K = 1_000_000, 256, 512, 100
    g = torch.Generator(device="cuda").manual_seed(5)
    cen = torch.randn((n // 50, d), generator=g, device="cuda") * 0.06
    ent = torch.empty((n, d), dtype=torch.bfloat16, device="cuda")
    for i in range(0, n, 1 << 18):
        j = min(n, i + (1 << 18))
        ent[i:j] = (cen[torch.arange(i, j, device="cuda") // 50] + torch.randn((j - i, d), generator=g, device="cuda") * 0.02).bfloat16()
    rel = (torch.randn((9, d), generator=g, device="cuda") * 0.01).bfloat16()
    h = torch.randint(0, n, (Q,), generator=g, device="cuda", dtype=torch.int32)
    r = torch.randint(0, 9, (Q,), generator=g, device="cuda", dtype=torch.int32)
    order = torch.randperm(n, generator=g, device="cuda")
    at = torch.empty_like(order)
    at[order] = torch.arange(n, device="cuda")
    ms = []
    for model, heads in ((kge.Model("transe", ent, rel), h), (kge.Model("transe", ent[order].contiguous(), rel), at[h.long()].int())):
        for _ in range(2):
            kge.topk(model, heads, r, 0, n, K)
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(3):
            kge.topk(model, heads, r, 0, n, K)
        e[1].record()
        torch.cuda.synchronize()
        ms.append(e[0].elapsed_time(e[1]) / 3)
    assert ms[0] <= 10 * ms[1], ms


def test_long_lists_of_appends(orc):
    """Scores that rise with the id, K = 256 and repeated rows, whose values tie at the cut; and a million scores that rise and that fall:
    all that beat the first threshold, some 5,000 of a query, are in one chunk - more than the compaction holds in registers, while no
    append area overflows."""
    G = make_case("distmult", 16384, 3, 32, 5, 0, False)
    G["rel"][:] = np.abs(G["rel"]) + 0.01
    G["ent"] = np.abs(G["ent"]) * np.linspace(0.1, 3.0, 16384).astype(np.float32)[:, None]
    G["ent"] = G["ent"][np.argsort(G["ent"].astype(np.float64).sum(1))].astype(np.float32)
    G["ent"][9000:9400] = G["ent"][9000]
    G["ent"][15000:16384] = G["ent"][15000]
    _check(orc, "distmult", G, False, 0, 16384, 256, np.array([15500, 3, 9100, 16383, 0], dtype=np.int32))
    _check(orc, "distmult", G, False, 0, 9300, 200, None)
    n = 1_000_000
    G = make_case("distmult", n, 3, 16, 5, 0, True)
    G["rel"] = ks.round_to_bf16(np.abs(G["rel"]) + 0.01)
    rising = (1 + 0.1 * np.random.default_rng(1).normal(size=(n, 16))) * np.linspace(0.1, 1.0, n)[:, None]
    for ent in (rising, rising[::-1]):
        G["ent"] = ks.round_to_bf16(np.ascontiguousarray(ent, dtype=np.float32))
        _check(orc, "distmult", G, True, 0, n, 256, np.array([0, n - 1, n // 2, 77, n - 300], dtype=np.int32))


@pytest.mark.parametrize("scorer,dim,bf16,Q", [("distmult", 64, True, 200), ("transh", 64, True, 100), ("complex", 400, True, 60),
                                               ("transe", 128, False, 128)])
def test_neighbouring_winners_fit_an_append_area(scorer, dim, bf16, Q):
    """Tables whose ids are sorted by type: 100 neighbouring rows beat every query's threshold.  They fit the append areas of their
    split (50 per lane half of 64 entries), so the call takes the time of the same rows in another order and not that of the exhaustive
    scan, which is some tens of times longer; and the same list either way."""
    import torch
    import paper_2211_12281_amd as kge
    n, hot = 400_000, 100
    g = torch.Generator(device="cuda").manual_seed(3)
    table = torch.rand((n, dim), generator=g, device="cuda") * 0.1 + 0.01
    at = 300_013
    table[at:at + hot] = 0.25 + 0.01 * torch.rand((hot, dim), generator=g, device="cuda")
    r = torch.zeros((3, dim), device="cuda")
    if scorer in ("distmult", "complex"):
        r[:, :dim // 2 if scorer == "complex" else dim] = 1.0
    else:
        r += 0.2                                           # the queries lie near the hot rows
    relw = torch.randn((3, dim), generator=g, device="cuda") if scorer == "transh" else None
    dt = torch.bfloat16 if bf16 else torch.float32
    h = torch.randint(0, at, (Q,), generator=g, device="cuda", dtype=torch.int32)
    rr = torch.randint(0, 3, (Q,), generator=g, device="cuda", dtype=torch.int32)
    perm = torch.randperm(n, generator=g, device="cuda")
    back = torch.empty_like(perm)
    back[perm] = torch.arange(n, device="cuda")            # row i of the table is row back[i] of the shuffled one
    res, times = [], []
    for t, heads in ((table, h), (table[perm], back[h.long()].to(torch.int32))):
        model = kge.Model(scorer, t.to(dt).contiguous(), r.to(dt), relw.to(dt) if relw is not None else None)
        best = 1e9
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            idx, sc, _ = kge.topk(model, heads, rr, 0, n, 100)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
        res.append(((idx if t is table else perm[idx.long()].to(torch.int32)).cpu().numpy(), sc.cpu().numpy()))
    assert np.array_equal(res[0][1], res[1][1])            # (ties are ordered by the table's own ids: compared as sets)
    assert np.mean([set(a) == set(b) for a, b in zip(res[0][0], res[1][0])]) > 0.9
    assert times[0] < 3 * times[1], times


@pytest.mark.parametrize("order,scorer,dim,bf16,Q,n,K", [
    (order, *case) for case in [("distmult", 32, True, 8192, 1_000_000, 100), ("complex", 64, False, 4000, 300_000, 30)]      # 32 splits, several chunks
    for order in ("falling", "rising", "rank", "hot head", "hot tail", "groups")] + [
    (order, "distmult", 32, True, 1000, 1 << 20, 100) for order in ("runs", "falling", "hot head")] + [                       # 128 splits
    (order, "distmult", 32, True, 8192, 1 << 20, 256) for order in ("every other", "every 1,024th", "parts", "sorted")])               # ... and the sample
def test_order_of_the_rows_costs_nothing(scorer, dim, bf16, Q, n, K, order):
    """Tables whose rows are sorted by length, popularity or group, or that repeat every 2^k tiles: no append area of the scan
    overflows (where one does, the query is ranked exhaustively, some tens of times longer) and the call takes the time of
    the same rows in another order; and the same lists either way.  Tables that repeat with a period and tables in the order of the
    scores: every maximum of the sample that the first threshold comes from stands for rows of all phases and of the whole table."""
    import torch
    import paper_2211_12281_amd as kge
    g = torch.Generator(device="cuda").manual_seed(5)
    i = torch.arange(n, device="cuda")
    length = {"falling": lambda: torch.linspace(1.5, 0.3, n, device="cuda"), "rising": lambda: torch.linspace(0.3, 1.5, n, device="cuda"),
              "rank": lambda: (i + 1.0) ** -0.2, "hot head": lambda: torch.where(i < n // 100, 5.0, 1.0),
              "hot tail": lambda: torch.where(i >= n - n // 100, 5.0, 1.0),
              "every other": lambda: torch.where(i % 2 == 1, 1.0, 0.2), "every 1,024th": lambda: torch.where(i % 1024 == 1023, 5.0, 1.0),
              "parts": lambda: torch.where(i % (n // 32) >= n // 32 - 200, 5.0, 1.0),
              "sorted": lambda: torch.linspace(0.01, 1.0, n, device="cuda"),
              "runs": lambda: torch.where(i % 16384 < 32, 5.0, 1.0),
              "groups": lambda: torch.exp2(torch.randint(-3, 3, (n // 5000 + 1,), generator=g, device="cuda").float())[i // 5000]}[order]()
    dt = torch.bfloat16 if bf16 else torch.float32
    table = torch.randn((n, dim), generator=g, device="cuda")
    r = torch.randn((3, dim), generator=g, device="cuda")
    if order == "sorted":                                  # (all scores positive and nearly proportional to the row's length)
        table, r = 1.0 + 0.1 * table, r.abs()
    table, r = (table * length[:, None]).to(dt), r.to(dt)
    h = torch.randint(0, n, (Q,), generator=g, device="cuda", dtype=torch.int32)
    rr = torch.randint(0, 3, (Q,), generator=g, device="cuda", dtype=torch.int32)
    perm = torch.randperm(n, generator=g, device="cuda")
    back = torch.empty_like(perm)
    back[perm] = i                                         # row i of the table is row back[i] of the shuffled one
    res, times = [], []
    for t, heads in ((table, h), (table[perm], back[h.long()].to(torch.int32))):
        model = kge.Model(scorer, t, r)
        best = 1e9
        for _ in range(3):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            idx, sc, _ = kge.topk(model, heads, rr, 0, n, K)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
        res.append((idx if t is table else perm[idx.long()].to(torch.int32), sc))
    assert torch.equal(res[0][1], res[1][1])               # (equal scores are ordered by the table's own ids)
    assert (res[0][0] == res[1][0]).float().mean() > 0.99
    assert times[0] < 2.5 * times[1], times


def test_ties_sub_ranges_and_padding(orc):
    G = make_case("distmult", 3000, 5, 32, 10, 0, False)
    for dst, src in [(1500, 3), (77, 3), (2999, 120), (10, 120), (5, 6)]:
        G["ent"][dst] = G["ent"][src]                      # exact ties: lower index first
    true_t = np.array([1500, 77, 3, 2999, 10, 6, 0, 1, 2, 2999], dtype=np.int32)
    for (lo, hi, K) in [(0, 3000, 50), (2, 2900, 256), (100, 101, 3), (40, 70, 64), (7, 7, 5)]:
        _check(orc, "distmult", G, False, lo, hi, K, true_t)
    _check(orc, "distmult", G, False, 0, 3000, 10, None)


def test_adversarial_candidate_order_still_exact(orc):
    """Candidates sorted by increasing score for every query: each new row beats the threshold, buffers
    overflow, and the exhaustive fp64 path must take over."""
    G = make_case("distmult", 30000, 3, 32, 4, 0, False)
    G["rel"][:] = np.abs(G["rel"]) + 0.01
    G["ent"] = np.abs(G["ent"])
    order = np.argsort(G["ent"].astype(np.float64).sum(1))
    scale = np.linspace(0.1, 3.0, 30000).astype(np.float32)[:, None]
    G["ent"] = (G["ent"][order] * scale).astype(np.float32)
    G["h"] = np.array([5, 17, 100, 29999], dtype=np.int32)
    _check(orc, "distmult", G, False, 0, 30000, 20, np.array([29990, 3, 15000, 29999], dtype=np.int32))


@pytest.mark.parametrize("order", ["rising", "falling", "clusters", "equal"])
@pytest.mark.parametrize("scorer,dim,bf16,Q,n,K", [
    ("distmult", 32, True, 5, 4129, 256), ("transe", 24, False, 129, 8191, 100),      # a tile more than one chunk; the smallest sample
    ("complex", 272, True, 130, 5001, 10), ("transh", 48, True, 300, 9999, 50),       # rows over 512 bytes; two contractions
    ("rotate", 64, False, 520, 6000, 256), ("distmult", 16, True, 8200, 2100, 3)])    # two blocks of queries; 32 splits
def test_sampled_threshold_on_sorted_tables(orc, scorer, dim, bf16, Q, n, K, order):
    """The threshold that the scan starts with comes from a sample of rows at even distances: tables sorted by length, tables whose
    neighbours are alike, and tables that are one row over and over (more equal values than a list holds, lowest index first)."""
    G = make_case(scorer, n, 7, dim, Q, 0, bf16)
    if order == "clusters":
        G["ent"] = G["ent"][np.arange(n) // 300 * 300] + (0.05 * G["ent"]).astype(np.float32)
    elif order == "equal":
        G["ent"][100:] = G["ent"][100]
    else:
        s = np.linspace(0.3, 1.5, n).astype(np.float32)[:, None]
        G["ent"] = G["ent"] * (s if order == "rising" else s[::-1])
    if bf16:
        G["ent"] = ks.round_to_bf16(np.ascontiguousarray(G["ent"]))
    G["ent"] = np.ascontiguousarray(G["ent"], dtype=np.float32)
    _check(orc, scorer, G, bf16, 0, n, K, ks.uniform_ids(ks.rng(9, ks.TAG_HELDOUT), 0, n, Q))


@pytest.mark.parametrize("scorer", ["distmult", "transe", "transh"])
@pytest.mark.parametrize("dim,bf16,Q", [(16, True, 70), (144, True, 130), (248, False, 600), (8, False, 520), (240, True, 1030), (304, True, 130)])
def test_columns_behind_a_row_are_not_read(scorer, dim, bf16, Q):
    """Tables that are the left columns of wider ones, whose other columns hold NaN: rows that do not fill 512 or 1,024 bytes, whose
    padding must come from neither the row's neighbour nor the memory behind the table.  The same lists as from tables of their own;
    clusters of equal rows give lanes of the scan several hits in one tile, and the last tile is ragged."""
    import paper_2211_12281_amd as kge
    if scorer == "transh" and dim * (2 if bf16 else 4) > 512:
        pytest.skip("TransH ranks rows of up to 512 bytes")
    n, dt = 9_001, torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(dim)
    wide = torch.full((n, dim + 64), float("nan"), dtype=dt, device="cuda")
    ent = torch.randn((n, dim), generator=g, device="cuda")
    ent[5000:5040] = ent[5000]
    ent[8990:] = ent[8990]
    wide[:, :dim] = ent.to(dt)
    rel = torch.randn((4, dim), generator=g, device="cuda").to(dt)
    relw = torch.randn((4, dim), generator=g, device="cuda").to(dt) if scorer == "transh" else None
    h, t = (torch.randint(0, n, (Q,), generator=g, device="cuda", dtype=torch.int32) for _ in range(2))
    h[:20] = torch.tensor([5000, 8990] * 10, dtype=torch.int32)
    r = torch.randint(0, 4, (Q,), generator=g, device="cuda", dtype=torch.int32)
    one = kge.topk(kge.Model(scorer, wide[:, :dim], rel, relw), h, r, 0, n, 30, t)
    two = kge.topk(kge.Model(scorer, wide[:, :dim].contiguous(), rel, relw), h, r, 0, n, 30, t)
    for a, b in zip(one, two):
        assert torch.equal(a, b)
    assert bool(torch.isfinite(two[1]).all())


@pytest.mark.parametrize("scorer,dim,Q,n", [
    ("distmult", 256, 130, 9001), ("transe", 136, 40, 4127), ("complex", 128, 513, 8200), ("transh", 120, 100, 6000),
    ("rotate", 8, 20, 4200), ("transe", 64, 600, 5000), ("distmult", 32, 7, 33)])
def test_fp32_rows_of_all_sizes(orc, scorer, dim, Q, n):
    """fp32 rows, which the scan takes as two fp16 pieces scaled by row: rows over a factor of 2^40 and elements over 2^12, rows of zeros, of
    subnormal numbers and of one element alone."""
    g = np.random.default_rng(dim + Q)
    G = make_case(scorer, n, 20, dim, Q, 0, False)
    e = G["ent"]
    e *= (2.0 ** g.integers(-36, 5, n)).astype(np.float32)[:, None] * (2.0 ** g.integers(-12, 1, e.shape)).astype(np.float32)
    at = g.permutation(n)
    e[at[0]] = 0
    e[at[1]] = (g.normal(size=dim) * 1e-40).astype(np.float32)
    e[at[2]] = 0
    e[at[2], dim // 2] = 3.0
    G["h"][:3] = at[:3]
    true_t = g.integers(0, n, Q).astype(np.int32)
    true_t[:3] = at[2::-1]
    _check(orc, scorer, G, False, 0, n, min(50, n), true_t)


@pytest.mark.parametrize("scorer", ["distmult", "transe", "transh"])
def test_fp32_rows_with_nan_and_infinity(scorer):
    """A row with a NaN is nobody's candidate and changes no other's place; rows and queries with an infinity are ranked by the exact scores:
    plus infinity first, no place for a NaN, equal scores in order of the ids."""
    import paper_2211_12281_amd as kge
    dim, Q, n, K = 128, 70, 5000, 20
    g = np.random.default_rng(3)
    G = make_case(scorer, n, 20, dim, Q, 0, False)
    bad = np.setdiff1d(g.permutation(n)[:300], G["h"])[:40]
    args = [dev_idx(G["h"]), dev_idx(G["r"]), 0, n, K]
    G["ent"][bad] = -G["ent"][G["h"][0]] if scorer == "distmult" else 100.0      # far from every query
    want = [x.cpu().numpy() for x in kge.topk(gpu_model(scorer, G, False), *args)[:2]]
    G["ent"][bad, g.integers(0, dim, len(bad))] = np.nan
    got = [x.cpu().numpy() for x in kge.topk(gpu_model(scorer, G, False), *args)[:2]]
    clean = ~np.isin(want[0], bad).any(axis=1)
    assert clean.sum() > Q // 2 and np.array_equal(got[0][clean], want[0][clean]) and np.array_equal(got[1][clean], want[1][clean])
    G["ent"][bad] = 0.0
    G["ent"][bad[0], 5] = np.inf
    G["ent"][bad[1], 7] = -np.inf
    G["h"][3] = bad[0]                                                           # a query with an infinity
    got = [x.cpu().numpy() for x in kge.topk(gpu_model(scorer, G, False), dev_idx(G["h"]), *args[1:])[:2]]
    e, q = G["ent"].astype(np.float64), G["ent"][G["h"]].astype(np.float64) * G["rel"][G["r"]]
    finite = np.isfinite(e).all(axis=1)
    if scorer == "distmult":
        with np.errstate(invalid="ignore"):
            s = q @ np.where(finite[:, None], e, 0.0).T
            s[:, bad[0]], s[:, bad[1]] = (q * e[bad[0]]).sum(axis=1), (q * e[bad[1]]).sum(axis=1)
            s[3] = (q[3] * e).sum(axis=1)
        assert np.isposinf(s[:, bad[:2]]).any() and np.isneginf(s[:, bad[:2]]).any() and np.isnan(s[3]).any()
        for k in range(Q):
            order = np.lexsort((np.arange(n), -s[k]))
            order = order[~np.isnan(s[k][order])][:K]
            assert np.array_equal(got[0][k], order), k
            assert np.array_equal(np.isinf(got[1][k]), np.isinf(s[k][order]))
    else:                                                                        # (infinitely far: from an infinite query everything is)
        G["ent"] = np.where(finite[:, None], G["ent"], np.float32(1e6))
        want = kge.topk(gpu_model(scorer, G, False), dev_idx(G["h"]), *args[1:])[0].cpu().numpy()
        rest = np.arange(Q) != 3
        assert np.array_equal(got[0][rest], want[rest])
        if scorer == "transe":
            assert np.array_equal(got[0][3], np.flatnonzero(finite)[:K]) and np.isneginf(got[1][3]).all()


def test_partition_bucketing(orc):
    import paper_2211_12281_amd as kge
    g = ks.rng(1, ks.TAG_TRIPLE_H)
    for (n_ent, D, n) in [(1003, 4, 5000), (90000, 16, 200000), (50, 64, 3000), (10, 1, 7)]:
        part = -(-n_ent // D)
        h, t = ks.uniform_ids(g, 0, n_ent, n), ks.uniform_ids(g, 0, n_ent, n)
        off, order = kge.partition_triples(dev_idx(h), dev_idx(t), part, D)
        rc, ro, rord = orc.bucket_triples(h, t, part, D)
        assert np.array_equal(off.cpu().numpy(), ro) and np.array_equal(order.cpu().numpy(), rord)
