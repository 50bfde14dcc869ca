"""Workspace sizes never fall as a call grows: one workspace sized for the largest batch serves every smaller one (host only)."""
import ctypes as C
import random

import pytest

import paper_2211_12281_amd.binding as b


def _model(rng, scorer):
    m = b.KgeModelT()
    m.scorer, m.p_norm, m.dtype = scorer, rng.choice([1, 2, 2]), rng.randrange(2)
    unit, most = (16, 512) if m.dtype == 1 else (8, 256)
    m.dim = unit * rng.choice([rng.randint(1, most // unit), most // unit, most // unit // 2])
    m.rel_dim = m.dim // 2 if scorer == b.SCORERS["rotate"] else m.dim
    m.n_ent = m.n_rel = 10 ** 7
    m.ent = m.rel = m.relw = 4096
    m.ent_ld = m.rel_ld = m.relw_ld = m.dim
    return m


def _pair(rng, bits):
    """A size and one that is no larger: near it, or anything below."""
    big = int(2 ** rng.uniform(0, bits)) - (rng.random() < 0.1)
    return big, rng.choice([big, rng.randint(0, big), max(0, big - rng.randint(0, 600))])


def _check(pairs):
    worse = [(c, small, large) for c, small, large in pairs if not 0 < small <= large]
    assert not worse, (len(worse), worse[:3])


@pytest.mark.parametrize("scorer", sorted(b.SCORERS))
def test_topk(scorer):
    lib, rng = b.load(), random.Random(scorer)
    def run():
        for _ in range(4000):
            m = _model(rng, b.SCORERS[scorer])
            (Q, q), (n, m_) = _pair(rng, 14), _pair(rng, 24)
            K = rng.randint(1, 256)
            k = rng.choice([K, rng.randint(1, K)])
            yield (m.dtype, m.dim, (q, m_, k), (Q, n, K)), lib.kge_workspace_bytes(3, C.byref(m), q, m_, k), lib.kge_workspace_bytes(3, C.byref(m), Q, n, K)
    _check(run())


@pytest.mark.parametrize("op", [0, 1])                     # kge_score, kge_loss_bwd
@pytest.mark.parametrize("scorer", sorted(b.SCORERS))
def test_score_and_loss(scorer, op):
    """Among the pairs: sizes around the lines between the routes of kge_loss_bwd, whose workspaces differ most."""
    lib, rng = b.load(), random.Random(scorer + str(op))
    def run():
        for _ in range(12000):
            m = _model(rng, b.SCORERS[scorer])
            (B, B_), (N, N_) = _pair(rng, 14), _pair(rng, 15)
            if rng.random() < 0.3:                          # (a million to eight million pairs)
                B = int(2 ** rng.uniform(7, 13)); N = int(2 ** rng.uniform(20, 23) / B)
                B_, N_ = max(0, B - rng.randint(0, B // 2)), max(0, N - rng.choice([0, rng.randint(0, N // 2)]))
            yield ((scorer, m.dtype, m.dim, m.p_norm, B_, N_, B, N), lib.kge_workspace_bytes(op, C.byref(m), B_, N_, 0),
                   lib.kge_workspace_bytes(op, C.byref(m), B, N, 0))
    _check(run())


@pytest.mark.parametrize("op", [6, 7])                     # kge_encode, kge_encode_bwd
def test_encoder(op):
    lib, rng = b.load(), random.Random(op)
    def run():
        for _ in range(20000):
            e = b.KgeEncoderT()
            e.dtype = rng.randrange(2)
            unit = 16 if e.dtype == 1 else 8
            e.dim, e.feat_dim = unit * rng.randint(1, 512 // unit), unit * rng.choice([rng.randint(1, 1024 // unit), 768 // unit])
            e.n_ent, e.ent_ld, e.feat_ld, e.m_ld = 10 ** 6, e.dim, e.feat_dim, e.feat_dim
            e.ent_s = e.feat = e.m_h = e.m_t = 4096
            (B, B_), (N, N_) = _pair(rng, 14), _pair(rng, 15)
            yield ((e.dtype, e.dim, e.feat_dim, B_, N_, B, N), lib.kge_encode_workspace_bytes(op, C.byref(e), B_, N_),
                   lib.kge_encode_workspace_bytes(op, C.byref(e), B, N))
    _check(run())
