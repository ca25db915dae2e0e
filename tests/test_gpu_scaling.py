"""GPU tests of the scaling of partials where transition matrices hold negative
entries: U e U^-1 has its zeros to a rounding of either sign (1e-16), so a
partial through an edge of length zero, or of a category whose rate is nearly
zero (Gamma shapes of a few hundredths), has negative entries of that size.
They are no reason not to scale a partial whose other entries have become
small.  Against the FP64 oracle.

Tolerances.  lnL: 1e-9 relative, the library's bar.  Where 70% of the inner edges of
300 taxa have length zero, dozens of random tips meet at one point, and the
likelihood hangs on entries as small as products of three or four substitutions
(1e-16), beside which the matrices' rounding is no longer small: a pattern's
lnL of about -800 may be off by some tenths, so 1e-3 there (the lnL that is
looked for here is not -inf).  Derivatives: with FP32 partials the library's
1e-3, relative to max(1, |d|).  With FP64 the rounding of the entries is what
is left: where two substitutions on edges of about 1e-5 meet at an edge of
length zero, the likelihood hangs on entries of about 1e-10 beside entries of
one, and 1e-16 is 1e-6 of them: 1e-5."""
import numpy as np
import pytest

import paper_1811_11007_amd as pt
import synth
from oracle import core as oc

pytestmark = pytest.mark.gpu

LNL_REL, ZERO_REL, FP64_REL, FP32_REL = 1e-9, 1e-3, 1e-5, 1e-3


@pytest.fixture(scope="module")
def ctx():
    c = pt.Context(0)
    yield c
    c.close()


def problem(n, P, mean, zero, seed):
    """A Yule tree with a part `zero` of its inner edges at length zero, random
    tips and a random model."""
    rng = np.random.default_rng(seed)
    e, b = synth.yule_tree(n, rng, mean=mean)
    b = np.where((e.min(axis=1) >= n) & (rng.random(len(b)) < zero), 0.0, b)
    tips = (1 << rng.integers(0, 4, size=(n, P))).astype(np.uint8)
    rates, freqs = np.exp(rng.normal(0.0, 0.7, size=6)), rng.dirichlet(np.full(4, 8.0))
    return e, b, tips, np.ones(P), rates, freqs


def lnl_error(got, want, what):
    err = abs(got - want) / abs(want)
    print(what, "lnL", got, "rel", err, flush=True)
    return err


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("n,mean,shape,zero", [
    (300, 1e-3, 0.03, 0.0), (300, 1e-3, 0.05, 0.0), (150, 1e-4, 0.02, 0.0), (150, 1e-3, 0.05, 0.0),
    (300, 0.02, 0.5, 0.7)])
def test_likelihood(ctx, n, mean, shape, zero, K):
    # (eight categories: what the LDS of a block takes)
    n = min(n, 150) if K == 8 else n
    worst = 0.0
    for seed in range(4):
        e, b, tips, w, rates, freqs = problem(n, 200, mean, zero, 1000 * K + seed)
        A = pt.Alignment(ctx, tips, w, rates, freqs, shape, K)
        want = oc.loglik(oc.Data(tips, w, rates, freqs, shape, K), e, b)
        what = "K %d n %d mean %g shape %g zero %g seed %d" % (K, n, mean, shape, zero, seed)
        for call in (pt.pt_batch_loglik, pt.pt_batch_loglik_noalloc):
            worst = max(worst, lnl_error(call(ctx, [A], pt.Trees([e]), b)[0], want, what))
    assert worst <= (ZERO_REL if zero else LNL_REL)


@pytest.mark.parametrize("n,K,mean,shape,zero", [
    (150, 4, 0.02, 0.5, 0.5), (150, 8, 0.02, 0.5, 0.5), (64, 4, 1e-3, 0.05, 0.0), (64, 8, 1e-3, 0.05, 0.0),
    (150, 4, 1e-3, 0.03, 0.0)])
def test_gradient(ctx, n, K, mean, shape, zero):
    worst = {}
    for seed in range(3):
        e, b, tips, w, rates, freqs = problem(n, 200, mean, zero, 2000 * K + n + seed)
        A = pt.Alignment(ctx, tips, w, rates, freqs, shape, K)
        want = oc.gradient(oc.Data(tips, w, rates, freqs, shape, K), e, b)
        # (in FP64 the matrices of 150 taxa and eight categories are beyond the LDS)
        for prec in (pt.PT_FP64, pt.PT_FP32) if n * K <= 600 else (pt.PT_FP32,):
            for hess in (False, True):
                got = pt.pt_batch_branch_grad(ctx, [A], pt.Trees([e]), b, prec, hess=hess)
                err = [lnl_error(got[0][0], want[0], "K %d n %d shape %g zero %g seed %d prec %d hess %d"
                                 % (K, n, shape, zero, seed, prec, hess))]
                for g, d in zip(got[1:], want[1:] if hess else want[1:2]):
                    err.append(np.max(np.abs(g - d) / np.maximum(1.0, np.abs(d))))
                print("  derivatives", err[1:], flush=True)
                worst[prec] = np.maximum(worst.get(prec, 0.0), np.pad(err, (0, 3 - len(err))))
    for prec, err in worst.items():
        assert err[0] <= LNL_REL
        assert np.all(err[1:] <= (FP64_REL if prec == pt.PT_FP64 else FP32_REL)), worst
