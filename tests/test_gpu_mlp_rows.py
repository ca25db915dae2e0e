"""GPU tests of the network's one-kernel pass (k_mlp_rows) at the sizes where
its tiles can go wrong: row counts around its 16 rows, hidden layers around a
wave's 64 lanes, inputs and outputs around its groups of eight, networks just
too large for it, and outputs written over the inputs.

Each output sums 1 + n_hidden and each hidden unit 1 + n_in FP32 products, and
each gradient is a FP64 sum of products of such values: against the FP64 oracle
they agree within 1e-4 of the largest entry (the library's bar for the
network)."""
import numpy as np
import pytest
import torch

import paper_1811_11007_amd as pt
from oracle import mlp as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = pt.Context(0)
    yield c
    c.close()


def network(ctx, ni, nh, no, rows):
    rng = np.random.default_rng(ni * 10007 + nh * 101 + no * 13 + rows)
    p = (rng.normal(0, 1, om.n_params(ni, nh, no)) * np.sqrt(1.0 / max(ni, nh))).astype(np.float32)
    x = rng.normal(0, 1, (rows, ni)).astype(np.float32)
    t = rng.normal(0, 0.5, (rows, no)).astype(np.float32)
    return pt.MLP(ctx, ni, nh, no, p), p, x, t


def close(got, want, tol=1e-4):
    assert np.max(np.abs(got - want)) <= tol * max(1e-30, np.max(np.abs(want))), np.max(np.abs(got - want))


# the last three do not fit in a block's LDS: row tiles, and a kernel per step
@pytest.mark.parametrize("ni,nh,no", [(14, 128, 5), (1, 1, 1), (8, 64, 8), (9, 63, 9), (7, 65, 17), (31, 100, 3),
                                      (60, 130, 12), (200, 40, 30), (700, 300, 4)])
def test_sizes_against_oracle(ctx, ni, nh, no):
    for rows in (1, 15, 16, 17, 33, 130, 1000):
        net, p, x, t = network(ctx, ni, nh, no, rows)
        print("net", (ni, nh, no), "rows", rows, flush=True)
        X, T = torch.tensor(x, device="cuda:0"), torch.tensor(t, device="cuda:0")
        p64, x64, t64 = (v.astype(np.float64) for v in (p, x, t))
        close(net.forward(X).cpu().numpy(), om.forward(x64, p64, ni, nh, no)[1])
        g = torch.full((net.n_params,), np.nan, dtype=torch.float32, device="cuda:0")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda:0")
        net.gradient(X, T, g, loss)
        torch.cuda.synchronize()
        close(g.cpu().numpy(), om.gradient(x64, t64, p64, ni, nh, no))
        lo = om.loss(x64, t64, p64, ni, nh, no)
        assert abs(loss.item() / (rows * no) - lo) <= 1e-5 * max(1.0, lo)
        net.close()


def test_outputs_over_inputs(ctx):
    """Predictions may be written over the inputs they are made from."""
    ni, nh, no, rows = 6, 40, 6, 1000
    net, p, x, t = network(ctx, ni, nh, no, rows)
    X = torch.tensor(x, device="cuda:0")
    want = net.forward(X).cpu().numpy()
    pt._lib.check(pt._lib.lib().pt_mlp_forward(net.h, X.data_ptr(), rows, X.data_ptr(), None))
    torch.cuda.synchronize()
    assert np.array_equal(X.cpu().numpy(), want)
    net.close()


@pytest.mark.parametrize("rows", [100, 60000])
def test_start_lengths_over_inputs(ctx, rows):
    """Start lengths may be written over the inputs they are made from, by more
    blocks than the device runs at once too."""
    ni, nh, no = 14, 128, 5
    net, p, x, t = network(ctx, ni, nh, no, rows)
    base = torch.rand(rows, no, dtype=torch.float64, device="cuda:0")
    pos = torch.randperm(rows * no, dtype=torch.int32, device="cuda:0")
    X = torch.tensor(x, device="cuda:0")
    call = pt._lib.lib().pt_mlp_warm_start

    def run(X, brlen):
        pt._lib.check(call(net.h, X.data_ptr(), rows, pos.data_ptr(), base.data_ptr(), 0.01, 1e-8, 100.0,
                           brlen.data_ptr(), None))
        torch.cuda.synchronize()
        return brlen.cpu().numpy()

    want = run(X, torch.zeros(rows * no, dtype=torch.float64, device="cuda:0"))
    for first in (0, rows):  # doubles from the inputs' start
        Y = X.clone()
        got = run(Y, Y.view(-1).view(torch.float64)[first:first + rows * no])
        assert np.array_equal(got, want), first
    net.close()


def test_scratch_of_a_network_that_fits(ctx):
    """A gradient of a network that fits in LDS takes memory for its blocks'
    sums and none for activations (128 MiB here)."""
    ni, nh, no, rows = 14, 128, 5, 1 << 18
    net, p, x, t = network(ctx, ni, nh, no, 1)
    X = torch.zeros(rows, ni, dtype=torch.float32, device="cuda:0")
    T = torch.zeros(rows, no, dtype=torch.float32, device="cuda:0")
    g = torch.zeros(net.n_params, dtype=torch.float32, device="cuda:0")
    net.gradient(X[:16], T[:16], g)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    net.gradient(X, T, g)
    torch.cuda.synchronize()
    taken, sums = free - torch.cuda.mem_get_info()[0], 8 * (rows // 16) * (net.n_params + 1)
    print("taken", taken, "sums", sums, flush=True)
    assert taken <= sums + (32 << 20)
    net.close()
