"""GPU tests of the matrix-core likelihood (k_prune) against the FP64 oracle,
and at the edges of tiles against the same patterns one at a time, where its
layout can go wrong: pattern counts around an item (4 to 16 patterns), a wave
and a tile, every padded category count, taxon counts from two up, tip codes
of one, several and all states, the register stack at every depth, and scaled
partials.

Tolerance: lnL is a sum over patterns of logarithms of positive sums; each
update adds a few units of rounding to a pattern, so about n * 1e-15 relative
per pattern and less in the sum: 1e-12 covers 80 taxa tenfold.  That leaves
out the transition matrices, whose entries near zero carry an absolute
rounding of 1e-16 (a difference of exponentials) that a tree of two taxa shows
undiluted (1e-12 relative at t = 1e-5): the tile-edge test, whose trees are
that small, compares every pattern of a tile with the same pattern alone, and
the others cover that one against the oracle."""
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


def problem(n, P, K, rng, ambiguous, mean=0.1):
    """A Yule tree and P random patterns; a third of the codes of several
    states when `ambiguous`."""
    e, b = synth.yule_tree(n, rng, mean=mean)
    tips = (1 << rng.integers(0, 4, size=(n, P))).astype(np.uint8)
    if ambiguous:
        some = rng.random((n, P)) < 0.33
        tips[some] = rng.integers(1, 16, size=int(some.sum())).astype(np.uint8)
    w = rng.integers(1, 5, size=P).astype(np.float64)
    return e, b, tips, w


def by_pattern(ctx, tips, w, K, e, b):
    """lnL as the sum of one-pattern alignments' (a tile's first pattern)."""
    alns = [pt.Alignment(ctx, tips[:, p:p + 1], w[p:p + 1], RATES, FREQS, 0.6, K) for p in range(len(w))]
    t = pt.Trees([e] * len(w), np.arange(len(w)))
    return np.sum(pt.pt_batch_loglik(ctx, alns, t, np.tile(b, len(w))))


def close(got, want, what, tol=1e-12):
    err = np.max(np.abs(np.asarray(got) - want) / np.abs(want))
    print(what, "max rel", err, flush=True)
    assert err <= tol


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("ambiguous", [False, True])
def test_edges_of_tiles(ctx, K, ambiguous):
    rng = np.random.default_rng(500 + 10 * K + ambiguous)
    for n in (2, 3, 4, 9):
        for P in (1, 3, 4, 5, 17, 31, 32, 33, 63, 64, 65, 127, 129, 257, 511, 513):
            e, b, tips, w = problem(n, P, K, rng, ambiguous)
            A = pt.Alignment(ctx, tips, w, RATES, FREQS, 0.6, K)
            got = pt.pt_batch_loglik(ctx, [A], pt.Trees([e]), b)
            want = by_pattern(ctx, tips, w, K, e, b)
            close(got, np.array([want]), "K %d amb %d n %d P %d" % (K, ambiguous, n, P))
            del A


@pytest.mark.parametrize("trees", [1, 40, 700])
def test_batches_of_every_item_count(ctx, trees):
    """Batch sizes that take two, four and eight items per wave, over two
    alignments of different category counts and ragged pattern counts."""
    rng = np.random.default_rng(560 + trees)
    alns, data, tops = [], [], []
    for K, n, P in ((4, 12, 333), (2, 7, 1001)):
        e, b, tips, w = problem(n, P, K, rng, True)
        alns.append(pt.Alignment(ctx, tips, w, RATES, FREQS, 0.6, K))
        data.append(oc.Data(tips, w, RATES, FREQS, 0.6, K))
        tops.append(e)
    idx = np.arange(trees) % 2
    lens = [rng.exponential(0.1, size=len(tops[i])) for i in idx]
    got = pt.pt_batch_loglik(ctx, alns, pt.Trees([tops[i] for i in idx], idx), np.concatenate(lens))
    pick = range(0, trees, max(1, trees // 30))
    want = np.array([oc.loglik(data[idx[t]], tops[idx[t]], lens[t]) for t in pick])
    close(got[list(pick)], want, "batch of %d" % trees)


def balanced(n, rng):
    nodes, nxt, edges = list(range(n)), n, []
    while len(nodes) > 2:
        up = []
        for i in range(0, len(nodes), 2):
            edges += [(nodes[i], nxt), (nodes[i + 1], nxt)]
            up.append(nxt)
            nxt += 1
        nodes = up
    return np.array([(nodes[0], nodes[1])] + edges, np.int32)


@pytest.mark.parametrize("n", [4, 8, 16, 32, 64, 128])
@pytest.mark.parametrize("K", [1, 4, 8])
def test_stack_depths(ctx, n, K):
    """Balanced trees rooted on their middle edge: log2(n) - 1 stack slots."""
    rng = np.random.default_rng(600 + n + K)
    e = balanced(n, rng)
    b = rng.exponential(0.1, size=len(e))
    _, _, tips, w = problem(n, 70, K, rng, False)
    A = pt.Alignment(ctx, tips, w, RATES, FREQS, 0.6, K)
    if n * K == 1024:  # six slots of eight categories: beyond both passes
        with pytest.raises(pt.PTError) as ei:
            pt.pt_batch_loglik(ctx, [A], pt.Trees([e]), b)
        assert ei.value.code == -4
        return
    got = pt.pt_batch_loglik(ctx, [A], pt.Trees([e]), b)
    want = oc.loglik(oc.Data(tips, w, RATES, FREQS, 0.6, K), e, b)
    close(got, np.array([want]), "balanced %d K %d" % (n, K))


@pytest.mark.parametrize("mean", [1e-4, 3.0])
def test_scaled_partials(ctx, mean):
    """Random tips on 300 taxa: every pattern's partials fall below 2^-256,
    in some categories long before the others when the lengths are short.
    Mismatching tips on edges of 1e-7 show the matrices' rounding (above), so
    the bar is the 1e-11 that the library's lnL is held to elsewhere."""
    rng = np.random.default_rng(int(650 + mean))
    for K in (1, 4, 8):
        e, b, tips, w = problem(300 if K < 8 else 150, 41, K, rng, False, mean=mean)
        A = pt.Alignment(ctx, tips, w, RATES, FREQS, 0.3, K)
        got = pt.pt_batch_loglik(ctx, [A], pt.Trees([e]), b)
        want = oc.loglik(oc.Data(tips, w, RATES, FREQS, 0.3, K), e, b)
        close(got, np.array([want]), "scaled K %d mean %g lnL %.1f" % (K, mean, want), 1e-11)


def test_optimised_lnl_of_the_deepest_tree(ctx):
    """The lnL that an optimisation with FP32 partials reports comes from
    k_prune at the final lengths, also beyond the eight stack slots that the
    likelihood calls take: a balanced tree of 1024 taxa needs nine."""
    rng = np.random.default_rng(700)
    n, P = 1024, 21
    e = balanced(n, rng)
    b = rng.exponential(0.05, size=len(e))
    tips = np.repeat((1 << rng.integers(0, 4, size=(1, P))).astype(np.uint8), n, 0)
    change = rng.random((n, P)) < 0.2
    tips[change] = (1 << rng.integers(0, 4, size=int(change.sum()))).astype(np.uint8)
    A = pt.Alignment(ctx, tips, np.ones(P), np.ones(6), np.full(4, 0.25), 1.0, 1)
    mask = np.zeros(len(e), np.uint8)
    mask[[0, 5, 900]] = 1
    lnl, out, passes, status = pt.pt_batch_optimize_branches(ctx, [A], pt.Trees([e]), b, mask, precision=pt.PT_FP32)
    assert status[0] == 0 and np.all(out[mask == 0] == b[mask == 0]) and np.any(out != b)
    want = oc.loglik(oc.Data(tips, np.ones(P), np.ones(6), np.full(4, 0.25), 1.0, 1), e, out)
    close(lnl, np.array([want]), "1024 taxa, lnL %.2f" % want, 1e-11)


def test_two_taxa_under_an_arena_cap(ctx, monkeypatch):
    """Trees of two taxa have no partials, so what a plan of them needs is their
    tiles' words: 16000 patterns in four categories keep within 12000 bytes."""
    rng = np.random.default_rng(710)
    e, b, tips, w = problem(2, 16000, 4, rng, True)
    A = pt.Alignment(ctx, tips, w, RATES, FREQS, 0.6, 4)
    want = pt.pt_batch_loglik(ctx, [A], pt.Trees([e]), b)
    monkeypatch.setenv("PT_ARENA_CAP_BYTES", "12000")
    assert np.array_equal(pt.pt_batch_loglik(ctx, [A], pt.Trees([e]), b), want)
    close(want, np.array([oc.loglik(oc.Data(tips, w, RATES, FREQS, 0.6, 4), e, b)]), "two taxa", 1e-11)
