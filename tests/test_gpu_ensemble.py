"""kge_ensemble against the oracle: indices bit-exact, scores to fp32 rounding."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _lists(g, M, Q, K, n_ent, pool):
    out = np.empty((M, Q, K), dtype=np.int32)
    for q in range(Q):
        cand = g.choice(n_ent, size=pool, replace=False)
        for m in range(M):
            out[m, q] = g.permutation(cand)[:K]
    return out


def _check(orc, lists, p, K_out):
    import paper_2211_12281_amd as kge
    idx, sc = kge.ensemble(torch.from_numpy(lists).cuda(), p, K_out)
    ridx, rsc = orc.ensemble(lists, p, K_out)
    assert np.array_equal(idx.cpu().numpy(), ridx)
    sc = sc.cpu().numpy()
    fin = np.isfinite(rsc)
    assert np.array_equal(np.isfinite(sc), fin)
    assert np.array_equal(sc[fin], rsc[fin].astype(np.float32))       # the fp64 sum, rounded once


@pytest.mark.parametrize("p", [1.0, -1.0, 2.0, -0.5, 0.3])
def test_matches_oracle(orc, p):
    g = np.random.default_rng(31)
    lists = _lists(g, 7, 40, 100, 100000, 260)
    lists[2, 3, 60:] = -1
    lists[4, 7, 9] = lists[4, 7, 2]
    _check(orc, lists, p, 10)


def test_shapes_and_ties(orc):
    g = np.random.default_rng(32)
    _check(orc, _lists(g, 1, 5, 10, 1000, 10), -1.0, 10)              # one model: the list itself
    _check(orc, _lists(g, 3, 9, 1, 50, 2), 1.0, 4)                    # K = 1, fewer candidates than K_out: padding
    _check(orc, _lists(g, 32, 6, 256, 5000, 300), -1.0, 16)           # 8192 entries: the largest supported query
    _check(orc, _lists(g, 85, 4, 96, 100000, 400), -1.0, 10)          # many models
    # identical lists in a different model order, integer power: exact ties between entities, broken by the id
    base = _lists(g, 2, 8, 12, 40, 12)
    sym = np.stack([base[0], base[0][:, ::-1]])                       # ranks k and K + 1 - k: every sum equals K + 1
    _check(orc, sym, 1.0, 12)
    all_pad = np.full((3, 2, 8), -1, dtype=np.int32)
    _check(orc, all_pad, -1.0, 5)


def test_limits_are_refused():
    import paper_2211_12281_amd as kge
    big = torch.zeros((40, 1, 256), dtype=torch.int32, device="cuda")  # 10,240 entries
    with pytest.raises(kge.KgeError):
        kge.ensemble(big, -1.0)
    ok = torch.zeros((2, 1, 4), dtype=torch.int32, device="cuda")
    with pytest.raises(kge.KgeError):
        kge.ensemble(ok, 0.0)


@pytest.mark.parametrize("M,K,K_out,pool,p", [
    (32, 256, 256, 8192, -1.0),      # 8,192 entries, most of them distinct: the table fills up; more than 256 candidates
    (32, 256, 32, 8192, 1.0),        # ... the last K_out of the 64-bin bound
    (33, 65, 33, 140, 1.0),          # lists of one piece and one rank, the first K_out of the 256-bin bound
    (5, 256, 100, 256, -0.5),        # every model lists the same entities
    (1, 1, 2, 1, -1.0)])
def test_table_and_selection_edges(orc, M, K, K_out, pool, p):
    g = np.random.default_rng(M * 1000 + K)
    lists = np.stack([[g.permutation(pool)[:K] + 1_000_000 * q for q in range(3)] for _ in range(M)]).astype(np.int32)
    if pool >= 8192:                                                   # lists that share next to nothing
        lists = g.permutation(3 * M * K).reshape(M, 3, K).astype(np.int32)
    if K > 64:                                                         # repeats inside a list: in one piece of 64 ranks, across pieces, many
        lists[0, 0, 40] = lists[0, 0, 3]
        lists[M // 2, 1, K - 1] = lists[M // 2, 1, 0]
        lists[M - 1, 2, 5:] = lists[M - 1, 2, 4]
        lists[M - 1, 0, 7:60:3] = -1
    _check(orc, lists, p, K_out)


def _agreeing(g, M, Q, K, spread):
    """Lists of models that rank one pool alike up to noise, as trained models do."""
    out = np.empty((M, Q, K), dtype=np.int32)
    for q in range(Q):
        ids = g.choice(5_000_000, size=4 * K, replace=False)
        base = -np.log(np.arange(1, 4 * K + 1))
        for m in range(M):
            out[m, q] = ids[np.argsort(-(base + spread * g.standard_normal(4 * K)))[:K]]
    return out


@pytest.mark.parametrize("M,K,K_out,spread,p,Q", [
    (16, 100, 10, 0.7, -1.0, 1281),      # one wave per query from 1,281 queries on; every query is proved
    (16, 100, 10, 0.7, 1.0, 1281),
    (16, 100, 10, 30.0, 1.0, 1281),      # lists that share little: the bound holds for none, all queries go to the other kernel
    (16, 100, 10, 3.0, -0.5, 1283),      # ... for some
    (64, 100, 20, 3.0, -1.0, 257),       # more than the small table's 128 entities in the first ranks: the walk ends early
    (5, 100, 26, 0.7, 0.3, 2049),        # the middle table, a model count that fills no word of ranks
    (128, 64, 36, 0.7, -1.0, 258),       # the most models
    (9, 100, 80, 0.7, -1.0, 1793),       # the widest table
    (63, 128, 200, 0.7, -1.0, 257),      # the longest whole lists of the widest table, two waves per workgroup and one
    (64, 128, 200, 0.7, 1.0, 257),
    (20, 129, 200, 0.7, 1.0, 769),       # the first without a table
    (2, 255, 200, 0.7, 1.0, 2049),       # the longest list whose ranks fit a byte: two models of it fit the widest table
    (1, 256, 200, 0.7, 1.0, 2049),
    (12, 10, 100, 0.7, -1.0, 13),        # short lists taken whole; fewer entities than winners
    (4, 64, 50, 30.0, 1.0, 13),          # 256 entries: every entity fits, nothing to prove
    (43, 3, 40, 0.7, -64.0, 13),         # sums that a float can't tell apart
    (1, 200, 10, 0.7, 16.0, 2050)])
def test_wave_kernel_and_the_queries_it_leaves(orc, M, K, K_out, spread, p, Q):
    g = np.random.default_rng(M * 1000 + K + K_out)
    lists = _agreeing(g, M, 13, K, spread)
    if K >= 64:                                                        # repeats: neighbours, in one piece of 64 entries, far apart; short lists
        lists[0, 0, 1] = lists[0, 0, 0]
        lists[M - 1, 1, 5:30] = lists[M - 1, 1, 4]
        lists[M // 2, 2, K - 1] = lists[M // 2, 2, 0]
        lists[0, 3, 2:] = -1
        lists[:, 4, 3:] = -7
        lists[:, 5] = lists[0, 5]
        lists[:, 6, 20:40] = lists[:, 6, :20]
    lists[:, 7] = -1
    _check(orc, np.ascontiguousarray(lists[:, np.arange(Q) % 13]), p, K_out)


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5, 6, 7, 16])
@pytest.mark.parametrize("K", [100, 129, 150, 192, 193, 255])
def test_wave_kernel_counts_an_entity_at_its_first_position(orc, M, K):
    """A list that repeats one of its first entities in its 2nd, 3rd or 4th 64 ranks, in queries that repeat nothing else: list 0, which
    is walked last, and list M - 1; lists of two, three and four pieces of 64 ranks, whose number leaves every remainder modulo 4."""
    g = np.random.default_rng(100 * M + K)
    lists = _agreeing(g, M, 13, K, 0.7)
    at = [64, 65, 99, K - 1, K - 2, min(130, K - 1), min(191, K - 1), K // 2]
    for q, k in enumerate(at):
        lists[0, q, k] = lists[0, q, q % 3]
    for q, k in enumerate(at[2:6]):
        lists[M - 1, 8 + q, k] = lists[M - 1, 8 + q, 0]
    _check(orc, np.ascontiguousarray(lists[:, np.arange(2060) % 13]), -1.0, 10)     # (one wave per query from 2,049 queries on, or fewer)
