"""GPU tests of the matrix-core gradient (k_grad) against the FP64 oracle at
the sizes where its layout can go wrong: pattern counts around an item, a
wave's 16 to 64 patterns and a tile, every padded category count, two taxa
up, ambiguous tip codes, both precisions, with and without second derivatives,
and partials scaled in either sweep.

Tolerances are the library's bars: FP64 1e-7 and FP32 partials 1e-3, relative
to max(1, |d|); lnL 1e-9 relative."""
import numpy as np
import pytest

import paper_1811_11007_amd as pt
import synth
from oracle import core as oc

pytestmark = pytest.mark.gpu

RATES, FREQS = np.array([0.7, 2.1, 0.4, 1.3, 3.0, 1.0]), np.array([0.31, 0.18, 0.23, 0.28])


@pytest.fixture(scope="module")
def ctx():
    c = pt.Context(0)
    yield c
    c.close()


def check(ctx, e, b, tips, w, K, what, alpha=0.6):
    A = pt.Alignment(ctx, tips, w, RATES, FREQS, alpha, K)
    T = pt.Trees([e])
    want_l, want_g, want_h = oc.gradient(oc.Data(tips, w, RATES, FREQS, alpha, K), e, b)
    for prec, tol in ((pt.PT_FP64, 1e-7), (pt.PT_FP32, 1e-3)):
        for hess in (False, True):
            lnl, g, h = pt.pt_batch_branch_grad(ctx, [A], T, b, prec, hess=hess)
            eg = np.max(np.abs(g - want_g) / np.maximum(1.0, np.abs(want_g)))
            eh = np.max(np.abs(h - want_h) / np.maximum(1.0, np.abs(want_h))) if hess else 0.0
            el = abs(lnl[0] - want_l) / abs(want_l)
            print(what, "prec", prec, "hess", hess, "lnL %.2g d1 %.2g d2 %.2g" % (el, eg, eh), flush=True)
            assert el <= 1e-9 and eg <= tol and eh <= tol


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8])
def test_edges_of_tiles(ctx, K):
    rng = np.random.default_rng(800 + K)
    for n in (2, 3, 4, 9):
        for P in (1, 2, 3, 4, 5, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 257):
            e, b = synth.yule_tree(n, rng, mean=0.1)
            b = b + 0.01
            tips = (1 << rng.integers(0, 4, size=(n, P))).astype(np.uint8)
            some = rng.random((n, P)) < 0.2
            tips[some] = rng.integers(1, 16, size=int(some.sum())).astype(np.uint8)
            w = rng.integers(1, 5, size=P).astype(np.float64)
            check(ctx, e, b, tips, w, K, "K %d n %d P %d" % (K, n, P))


@pytest.mark.parametrize("K,n", [(1, 300), (4, 150)])
def test_scaled_partials(ctx, K, n):
    """Random tips: every pattern is scaled, in the post-order sweep and in
    the outer partials of the pre-order one."""
    rng = np.random.default_rng(850 + K)
    e, b = synth.yule_tree(n, rng, mean=0.2)
    b = b + 0.01
    tips = (1 << rng.integers(0, 4, size=(n, 50))).astype(np.uint8)
    check(ctx, e, b, tips, np.ones(50), K, "scaled K %d n %d" % (K, n))


def test_batch_over_alignments(ctx):
    """Trees of several alignments, category counts and shapes in one plan."""
    rng = np.random.default_rng(870)
    alns, data, tops, lens, idx = [], [], [], [], []
    for i, (n, P, K) in enumerate(((12, 333, 4), (7, 70, 2), (33, 129, 3))):
        tips = (1 << rng.integers(0, 4, size=(n, P))).astype(np.uint8)
        w = rng.integers(1, 5, size=P).astype(np.float64)
        alns.append(pt.Alignment(ctx, tips, w, RATES, FREQS, 0.6, K))
        data.append(oc.Data(tips, w, RATES, FREQS, 0.6, K))
        for _ in range(5):
            e, b = synth.yule_tree(n, rng, mean=0.1)
            tops.append(e)
            lens.append(b + 0.01)
            idx.append(i)
    T = pt.Trees(tops, idx)
    for prec, tol in ((pt.PT_FP64, 1e-7), (pt.PT_FP32, 1e-3)):
        lnl, g, h = pt.pt_batch_branch_grad(ctx, alns, T, np.concatenate(lens), prec, hess=True)
        for t in range(len(tops)):
            wl, wg, wh = oc.gradient(data[idx[t]], tops[t], lens[t])
            s = slice(T.edge_offset[t], T.edge_offset[t + 1])
            assert abs(lnl[t] - wl) <= 1e-9 * abs(wl)
            assert np.all(np.abs(g[s] - wg) <= tol * np.maximum(1.0, np.abs(wg)))
            assert np.all(np.abs(h[s] - wh) <= tol * np.maximum(1.0, np.abs(wh)))


@pytest.mark.parametrize("prec", [pt.PT_FP64, pt.PT_FP32])
def test_small_trees_under_an_arena_cap(ctx, monkeypatch, prec):
    """Batches are split so that every part keeps within the cap, also where a
    plan is mostly its tiles' rows of sums: trees of two taxa, and of three
    beside one of forty."""
    rng = np.random.default_rng(880)
    alns, tops, lens, idx = [], [], [], []
    for i, (n, P, count) in enumerate(((2, 16000, 30), (3, 4000, 30), (40, 64, 1))):
        tips = (1 << rng.integers(0, 4, size=(n, P))).astype(np.uint8)
        alns.append(pt.Alignment(ctx, tips, np.ones(P), RATES, FREQS, 0.6, 4))
        for _ in range(count):
            e, b = synth.yule_tree(n, rng, mean=0.1)
            tops.append(e)
            lens.append(b + 0.01)
            idx.append(i)
    order = rng.permutation(len(tops))
    T = pt.Trees([tops[i] for i in order], [idx[i] for i in order])
    b = np.concatenate([lens[i] for i in order])
    want = pt.pt_batch_branch_grad(ctx, alns, T, b, prec, hess=True)
    monkeypatch.setenv("PT_ARENA_CAP_BYTES", str(4 << 20))
    got = pt.pt_batch_branch_grad(ctx, alns, T, b, prec, hess=True)
    for g, x in zip(got, want):
        assert np.allclose(g, x, rtol=1e-12, atol=0)
