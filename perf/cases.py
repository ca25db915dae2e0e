"""The work that programs have this library do, as cases that can be timed.

Every case is one call sequence through the public entry points on inputs
drawn from a seed: a random tree, an alignment simulated on it under GTR +
discrete Gamma (or JC69 with one category), and topologies a few NNI moves
away that inherit its lengths, which is what a threshold search over
topologies evaluates all day.  Sizes follow the library's own workloads: 5 to
67 taxa, about 100 to 2000 site patterns, single topologies to a search's
batch of 1024.

  path        what one pass is
  loglik      lnL of a batch of trees: a plan on device lengths, or with
              host = True the host-pointer batch call
  grad        lnL and every edge derivative: a plan call; host = True the
              host-pointer call with the hessian diagonal; autograd = True
              forward and backward of the torch module
  optimize    full branch-length optimisation of a plan's trees (graphs =
              True: replayed from a captured HIP graph on its own stream)
  propose     the search's proposal step: masks of radius 0, a new plan, the
              partial optimisation of every proposal, the plan's release
  mlp_grad    one forward and backward of the warm-start network
  mlp_warm    the network's prediction applied to a batch's start lengths
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1811_11007_amd as pt

# taxa x patterns of the four uneven alignments of a mixed batch
MIXED = [(27, 976), (36, 1187), (50, 938), (64, 861)]
NET = (14, 128, 5)  # features, hidden units, predicted lengths of the warm-start network


def listed():
    base = {"cats": 4, "precision": "fp64"}
    return [
        # scoring one small topology from a host program: latency is all there is
        {"name": "loglik_one_5", "path": "loglik", "host": True, "taxa": 5, "patterns": 90, "trees": 1,
         "cats": 1, "precision": "fp64"},
        # scoring the NNI neighbourhood of one topology, lengths on the device
        dict(base, name="loglik_48_27", path="loglik", taxa=27, patterns=976, trees=48),
        # scoring a batch over several genes at once
        dict(base, name="loglik_mixed_512", path="loglik", mixed=True, trees=512),
        # stationarity and curvature of one topology, from a host program
        dict(base, name="grad_one_27", path="grad", host=True, taxa=27, patterns=976, trees=1),
        # gradient-based inference over many topologies, single-precision partials
        dict(base, name="grad_256_50", path="grad", taxa=50, patterns=1250, trees=256, precision="fp32"),
        # lnL as a node of a torch graph, double precision: forward and backward
        dict(base, name="autograd_48_64", path="grad", autograd=True, taxa=64, patterns=1711, trees=48),
        # visiting the neighbourhood of a topology: the search's main cost
        dict(base, name="optimize_48_27", path="optimize", taxa=27, patterns=976, trees=48, precision="fp32",
             graphs=True),
        # the same where optima are wanted to full precision
        dict(base, name="optimize_48_27_fp64", path="optimize", taxa=27, patterns=976, trees=48),
        # visiting many topologies of several genes in one launch
        dict(base, name="optimize_mixed_256", path="optimize", mixed=True, trees=256, precision="fp32"),
        # one batch of a search's proposals, each optimised on its new edge only
        dict(base, name="propose_1024_64", path="propose", taxa=64, patterns=1711, trees=1024, precision="fp32"),
        # a training step's gradient, and the prediction for a batch of proposals
        {"name": "mlp_grad_4096", "path": "mlp_grad", "rows": 4096},
        {"name": "mlp_warm_1024", "path": "mlp_warm", "rows": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["loglik", "loglik", "grad", "grad", "optimize", "optimize", "propose", "mlp_grad", "mlp_warm"])
    if path.startswith("mlp"):
        return {"path": path, "rows": _log_int(rng, 33, 6000)}
    case = {"path": path, "cats": rng.choice([4, 4, 4, 4, 1, 2, 3, 8]), "precision": rng.choice(["fp32", "fp64"]),
            "taxa": _log_int(rng, 4, 67), "patterns": _log_int(rng, 90, 2000)}
    # few patterns can differ on few taxa; two or more of a handful of taxa stay below this
    case["patterns"] = min(case["patterns"], 20 * case["taxa"] if case["taxa"] < 12 else 2000)
    size = case["taxa"] * case["patterns"] * max(4, case["cats"])  # of one tree
    most = {"loglik": 400e6, "grad": 60e6, "optimize": 8e6, "propose": 400e6}[path]
    top = max(1, min(1024, int(most / size)))
    case["trees"] = _log_int(rng, 1, top) if path != "propose" else _log_int(rng, min(16, top), top)
    if path == "loglik":
        case["host"] = rng.random() < 0.25
    elif path == "grad":
        kind = rng.choice(["plan", "plan", "host", "autograd"])
        case["host"], case["autograd"] = kind == "host", kind == "autograd"
        if kind == "host":
            case["trees"] = min(case["trees"], 8)
    elif path == "optimize":
        case["graphs"] = rng.random() < 0.5
    elif path == "propose":
        case["precision"], case["cats"] = "fp32", 4
    return case


# ------------------------------------------------------------------ inputs

def _tree(n, rng):
    """A random binary topology (lineages joined in random order) with
    exponential lengths of mean 0.05; edges in random order."""
    if n == 2:
        return np.array([[0, 1]], np.int32), rng.exponential(0.05, 1)
    live, edges, nxt = [int(x) for x in rng.permutation(n)], [], n
    while len(live) > 3:
        for _ in range(2):
            edges.append((live.pop(int(rng.integers(len(live)))), nxt))
        live.append(nxt)
        nxt += 1
    edges += [(x, nxt) for x in live]
    e = np.array(edges, np.int32)[rng.permutation(len(edges))]
    flip = rng.random(len(e)) < 0.5
    e[flip] = e[flip][:, ::-1]
    return np.ascontiguousarray(e), rng.exponential(0.05, len(e))


def _model(cats, rng):
    """(exchangeabilities, frequencies): JC69 for one category, else GTR."""
    if cats == 1:
        return np.ones(6), np.full(4, 0.25)
    return rng.dirichlet(np.ones(6)), rng.dirichlet(10.0 * np.ones(4))


def _rate_matrix(rates, freqs):
    q = np.zeros((4, 4))
    for x, (i, j) in zip(rates, [(0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3)]):
        q[i, j], q[j, i] = x * freqs[j], x * freqs[i]
    q -= np.diag(q.sum(1))
    return q / -np.dot(freqs, np.diag(q))


def _walk(edges, n):
    """Edges as (parent, child, edge index) from node n (leaf 0 if n = 2), parents first."""
    at = [[] for _ in range(max(2, 2 * n - 2))]
    for i, (a, b) in enumerate(edges.tolist()):
        at[a].append((b, i))
        at[b].append((a, i))
    root = 0 if n == 2 else n
    out, stack = [], [(root, -1)]
    while stack:
        v, up = stack.pop()
        for c, e in at[v]:
            if c != up:
                out.append((v, c, e))
                stack.append((c, v))
    return root, out


def _alignment(edges, lens, n, patterns, cats, rates, freqs, rng):
    """(tip codes [n][patterns], pattern counts) simulated along the tree,
    continuous Gamma(0.5) site rates, until `patterns` patterns differ."""
    lam, right = np.linalg.eig(_rate_matrix(rates, freqs))
    lam, right = lam.real, right.real
    left = np.linalg.inv(right)
    root, walk = _walk(edges, n)
    seen, order, counts = {}, [], []
    while True:
        s = 2 * patterns + 64
        rate = np.ones(s) if cats == 1 else rng.gamma(0.5, 2.0, s)
        state = np.zeros((max(2, 2 * n - 2), s), np.int8)
        state[root] = rng.choice(4, s, p=freqs)
        for v, c, e in walk:
            rows = (right[state[v]] * np.exp(np.outer(rate * lens[e], lam))) @ left
            cum = np.cumsum(np.maximum(rows, 0.0), 1)
            state[c] = (rng.random(s)[:, None] * cum[:, -1:] >= cum[:, :3]).sum(1)
        for col in np.ascontiguousarray(state[:n].T):
            key = col.tobytes()
            if key in seen:
                counts[seen[key]] += 1
            elif len(order) < patterns:
                seen[key] = len(order)
                order.append(col)
                counts.append(1)
        if len(order) == patterns:
            break
        lens = lens * 1.5  # too few differ: a more divergent set of sites
    codes = np.left_shift(1, np.array(order, np.uint8).T)
    return np.ascontiguousarray(codes, np.uint8), np.array(counts, np.float64)


def _nni(edges, n, rng):
    """(edges after one random NNI move, its central edge)."""
    inner = np.flatnonzero((edges >= n).all(1))
    c = int(rng.choice(inner))
    u, v = (int(x) for x in edges[c])
    at = [[i for i in np.flatnonzero((edges == x).any(1)).tolist() if i != c] for x in (u, v)]
    a, b = int(rng.choice(at[0])), int(rng.choice(at[1]))
    new = edges.copy()
    new[a] = np.where(edges[a] == u, v, edges[a])
    new[b] = np.where(edges[b] == v, u, edges[b])
    return new, c


def _inputs(case, seed):
    rng = np.random.default_rng([int(seed), 1811])
    cats = case["cats"]
    shapes = MIXED if case.get("mixed") else [(case["taxa"], case["patterns"])]
    alns, trees, lens, index, centres = [], [], [], [], []
    for i, (n, patterns) in enumerate(shapes):
        e, b = _tree(n, rng)
        rates, freqs = _model(cats, rng)
        tips, w = _alignment(e, b, n, patterns, cats, rates, freqs, rng)
        alns.append((tips, w, rates, freqs))
        for _ in range(case["trees"] // len(shapes)):
            new, centre = e, 0
            for _ in range(int(rng.integers(1, 4)) if n > 3 else 0):
                new, centre = _nni(new, n, rng)
            trees.append(new)
            centres.append(centre)
            lens.append(b if case["path"] in ("optimize", "propose") else b * rng.uniform(0.5, 2.0, len(b)))
            index.append(i)
    return alns, trees, np.concatenate(lens), np.array(index, np.int32), centres


def _net_inputs(case, seed):
    rng = np.random.default_rng([int(seed), 1811])
    ni, nh, no = NET
    params = np.concatenate([rng.normal(0, ni ** -0.5, ni * nh), np.zeros(nh), rng.normal(0, nh ** -0.5, nh * no),
                             np.zeros(no)]).astype(np.float32)
    x = rng.normal(-2.0, 1.5, (case["rows"], ni)).astype(np.float32)
    y = rng.normal(0, 0.7, (case["rows"], no)).astype(np.float32)
    base = rng.exponential(0.05, (case["rows"], no))
    pos = np.arange(case["rows"])[:, None] * 125 + np.stack(
        [rng.permutation(125)[:no] for _ in range(case["rows"])])
    return params, x, y, base, pos.astype(np.int32)


_PRECISION = {"fp32": pt.PT_FP32, "fp64": pt.PT_FP64}
_KIND = {"loglik": pt.PT_PLAN_LOGLIK, "grad": pt.PT_PLAN_GRAD, "optimize": pt.PT_PLAN_OPTIMIZE}
_ctx = None


def _context():
    """The program's one context."""
    global _ctx
    if _ctx is None:
        _ctx = pt.Context(0)
    return _ctx


def prepare(case, seed):
    ctx, dev = _context(), torch.device("cuda", 0)
    s = {"case": case, "ctx": ctx, "dev": dev}
    if case["path"].startswith("mlp"):
        params, x, y, base, pos = _net_inputs(case, seed)
        s["net"] = pt.MLP(ctx, *NET, params)
        s["x"], s["y"] = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
        s["base"], s["pos"] = torch.tensor(base, device=dev), torch.tensor(pos, device=dev)
        s["grad"] = torch.empty(len(params), dtype=torch.float32, device=dev)
        s["loss"] = torch.empty(1, dtype=torch.float64, device=dev)
        s["brlen"] = torch.full((case["rows"] * 125,), 0.05, dtype=torch.float64, device=dev)
        return s
    alns, trees, lens, index, centres = _inputs(case, seed)
    s["precision"] = _PRECISION[case["precision"]]
    s["alns"] = [pt.Alignment(ctx, tips, w, rates, freqs, 0.5, case["cats"]) for tips, w, rates, freqs in alns]
    s["lens"] = lens
    if case["path"] == "propose":
        s["trees"], s["centres"] = trees, centres
        return s
    s["trees"] = pt.Trees(trees, index)
    if case.get("host"):
        return s
    nt, ne = s["trees"].n_trees, s["trees"].n_edges
    s["b0"] = torch.tensor(lens, dtype=torch.float64, device=dev)
    if case.get("autograd"):
        from paper_1811_11007_amd.autograd import TreeLogLik
        s["module"] = TreeLogLik(ctx, s["alns"], s["trees"], s["precision"]).to(dev)
        return s
    s["plan"] = pt.Plan(ctx, s["alns"], s["trees"], _KIND[case["path"]], s["precision"])
    s["lnl"] = torch.empty(nt, dtype=torch.float64, device=dev)
    if case["path"] == "grad":
        s["grad"] = torch.empty(ne, dtype=torch.float64, device=dev)
    if case["path"] == "optimize":
        s["b"] = torch.empty_like(s["b0"])
        s["passes"] = torch.empty(nt, dtype=torch.int32, device=dev)
        s["status"] = torch.empty(nt, dtype=torch.int32, device=dev)
        s["stream"] = torch.cuda.current_stream(dev)
        if case.get("graphs"):
            s["plan"].set_graphs(True)
            s["stream"] = torch.cuda.Stream(dev)
    torch.cuda.synchronize(dev)
    return s


# -------------------------------------------------------------------- a pass

def run(s):
    case = s["case"]
    path = case["path"]
    if path == "mlp_grad":
        s["net"].gradient(s["x"], s["y"], s["grad"], s["loss"])
        return s["grad"], s["loss"]
    if path == "mlp_warm":
        s["net"].warm_start(s["x"], s["pos"], s["base"], s["brlen"])
        return s["brlen"]
    if path == "loglik" and case.get("host"):
        return pt.pt_batch_loglik(s["ctx"], s["alns"], s["trees"], s["lens"], s["precision"])
    if path == "grad" and case.get("host"):
        return pt.pt_batch_branch_grad(s["ctx"], s["alns"], s["trees"], s["lens"], s["precision"], hess=True)
    if path == "loglik":
        s["plan"].loglik(s["b0"], s["lnl"])
        return s["lnl"]
    if path == "grad" and case.get("autograd"):
        b = s["b0"].detach().requires_grad_(True)
        lnl = s["module"](b)
        lnl.sum().backward()
        return lnl.detach(), b.grad
    if path == "grad":
        s["plan"].grad(s["b0"], s["lnl"], s["grad"])
        return s["lnl"], s["grad"]
    if path == "optimize":
        with torch.cuda.stream(s["stream"]):
            s["b"].copy_(s["b0"])
            s["plan"].optimize(s["b"], s["lnl"], s["passes"], s["status"], stream=s["stream"])
        return s["lnl"], s["b"], s["passes"], s["status"]
    # propose: what the search does with one batch of proposals
    n = case["taxa"]
    mask = None
    if n > 3:
        mask = pt.pt_radius_masks(n, np.stack(s["trees"]), s["centres"], 0).ravel()
    trees = pt.Trees(s["trees"])
    plan = pt.Plan(s["ctx"], s["alns"], trees, pt.PT_PLAN_OPTIMIZE, s["precision"], mask=mask)
    b = torch.tensor(s["lens"], dtype=torch.float64, device=s["dev"])
    lnl = torch.zeros(trees.n_trees, dtype=torch.float64, device=s["dev"])
    passes = torch.zeros(trees.n_trees, dtype=torch.int32, device=s["dev"])
    plan.optimize(b, lnl, passes)
    torch.cuda.synchronize(s["dev"])
    out = lnl.cpu(), b.cpu(), passes.cpu()
    plan.close()
    return out


# -------------------------------------------------- what a pass cannot do without

def work(case):
    if case["path"].startswith("mlp"):
        ni, nh, no = NET
        rows, params = case["rows"], ni * nh + nh + nh * no + no
        macs = ni * nh + nh * no
        if case["path"] == "mlp_grad":
            return {"bytes": 4 * (rows * (ni + no) + 2 * params) + 8, "flops": rows * (4.0 * macs + 2.0 * nh * no)}
        return {"bytes": 4 * (rows * ni + params) + rows * no * (4 + 8 + 8), "flops": 2.0 * rows * macs}
    shapes = MIXED if case.get("mixed") else [(case["taxa"], case["patterns"])]
    per, k = case["trees"] // len(shapes), case["cats"]
    total = {"bytes": 0.0, "flops": 0.0}
    for n, p in shapes:
        edges = max(1, 2 * n - 3)
        prune = (n - 2) * 68.0 + 40.0  # per pattern and category: two 4x4 products and their product per node, the root
        # the derivatives: per node one more product outwards, per edge both sides in the eigenbasis and three sums
        grad = prune + (n - 2) * 36.0 + edges * (2 * 28.0 + 4.0 + 24.0)
        # one pass over the edges: 1.5 partial updates, the eigenbasis table and one evaluation each
        sweep = edges * (1.5 * 68.0 + 60.0 + 24.0)
        flops = {"loglik": prune, "grad": grad, "optimize": prune + 5.0 * sweep, "propose": 2.0 * prune}[case["path"]]
        vectors = {"loglik": 1, "grad": 2, "optimize": 2, "propose": 2}[case["path"]]
        total["bytes"] += p * (n + 8.0) + per * (8.0 * vectors * edges + 8.0 + 8.0 * edges)
        total["flops"] += per * flops * p * k
    return total


# ------------------------------------------------- the values, in 64 bits by torch

def _gamma_means(k):
    """Means of Gamma(0.5, 0.5) over its k equal quantile intervals: with
    X = Z^2, Z standard normal, the quantiles and the truncated mean are
    those of Z."""
    if k == 1:
        return [1.0]
    cdf = lambda z: math.erf(z / math.sqrt(2.0))  # of |Z|
    pdf = lambda z: math.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)
    cut = [0.0]
    for i in range(1, k):
        lo, hi = 0.0, 40.0
        for _ in range(200):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if cdf(mid) < i / k else (lo, mid)
        cut.append(0.5 * (lo + hi))
    part = [cdf(z) - 2.0 * z * pdf(z) for z in cut] + [1.0]  # E[Z^2; |Z| < z]
    return [k * (part[i + 1] - part[i]) for i in range(k)]


def _exact_lnl(edges, t, n, tips, w, lam, right, left, freqs, rate):
    """lnL of one tree by pruning; tips [n][patterns][1][4] of 0 and 1, t its lengths."""
    k = len(rate)
    ex = torch.exp(t[:, None, None] * rate[None, :, None] * lam)  # [edge][k][4]
    prob = torch.matmul(right * ex[:, :, None, :], left)  # [edge][k][4][4]
    root, walk = _walk(edges, n)
    part = {}
    shape = (tips.shape[1], k, 4)
    for v, c, e in reversed(walk):
        x = tips[c].expand(shape) if c < n else part.pop(c)
        y = (x[:, :, None, :] * prob[e]).sum(-1)
        part[v] = part[v] * y if v in part else y
    x = part[root] if root >= n else part[root] * tips[root].expand(shape)
    return (w * torch.log((x * freqs).sum(-1).mean(-1))).sum()


def exact(case, seed):
    dev = torch.device("cuda", 0)
    if case["path"].startswith("mlp"):
        params, x, y, base, pos = _net_inputs(case, seed)
        ni, nh, no = NET
        p = torch.tensor(params, dtype=torch.float64, device=dev, requires_grad=True)
        x = torch.tensor(x, dtype=torch.float64, device=dev)
        w1, b1, w2, b2 = torch.split(p, [ni * nh, nh, nh * no, no])
        out = torch.tanh(x @ w1.view(ni, nh) + b1) @ w2.view(nh, no) + b2
        if case["path"] == "mlp_grad":
            d = (out - torch.tensor(y, dtype=torch.float64, device=dev)).square()
            d.mean().backward()
            return p.grad, d.sum().detach().reshape(1)
        b = torch.full((case["rows"] * 125,), 0.05, dtype=torch.float64, device=dev)
        t = (torch.tensor(base, device=dev) + 1e-4) * torch.exp(out.detach()) - 1e-4
        b[torch.tensor(pos, dtype=torch.int64, device=dev).ravel()] = t.clamp(1e-8, 100.0).ravel()
        return b
    if case["path"] in ("optimize", "propose"):
        return None  # an iterate at a tolerance, not a value
    alns, trees, lens, index, _ = _inputs(case, seed)
    f64 = lambda v: torch.tensor(np.ascontiguousarray(v), dtype=torch.float64, device=dev)
    data = []
    for tips, w, rates, freqs in alns:
        lam, right = np.linalg.eig(_rate_matrix(rates, freqs))
        lam, right = lam.real, right.real
        bits = np.stack([(tips >> j) & 1 for j in range(4)], -1)[:, :, None, :]
        data.append((tips.shape[0], f64(bits), f64(w), f64(lam), f64(right), f64(np.linalg.inv(right)), f64(freqs),
                     f64(_gamma_means(case["cats"]))))
    lnl, grad, hess, at = [], [], [], 0
    for e, i in zip(trees, index):
        n, rest = data[i][0], data[i][1:]
        t = f64(lens[at:at + len(e)])
        at += len(e)
        if case["path"] == "loglik":
            lnl.append(_exact_lnl(e, t, n, *rest))
            continue
        t.requires_grad_(True)
        v = _exact_lnl(e, t, n, *rest)
        g, = torch.autograd.grad(v, t, create_graph=bool(case.get("host")))
        if case.get("host"):
            hess += [torch.autograd.grad(g[j], t, retain_graph=True)[0][j] for j in range(len(e))]
        lnl.append(v.detach())
        grad.append(g.detach())
    lnl = torch.stack(lnl)
    if case["path"] == "loglik":
        return lnl
    return (lnl, torch.cat(grad), torch.stack(hess)) if case.get("host") else (lnl, torch.cat(grad))
