"""The work that is timed: what programs built on this framework ask of it, from the smallest call to the largest.

Kinds of case
  scores    a batch of graphs is scored and each graph's K candidates are selected: the framework's main path.
            The handle (the batch, its tuned SpMV form, the workspace) is kept between passes, as a program that
            scores repeatedly keeps it
  monte     one Monte-Carlo column of the identification-rate experiments: many small graphs, one scores() and one
            topk() call, outputs allocated by the call
  train     one differentiation step: scores and the gradient of the target nodes' summed scores with respect to
            every edge weight, through autograd
  central   subgraph centrality of a candidate set on one graph
  generate  background realizations drawn on the device with the target embedded

Graphs are drawn here with torch, from the seed alone, so that exact() sees the same inputs without the framework.
"""
import math
import random

import numpy as np
import torch

from paper_1409_5000_amd import api

TOL, M_MAX = 1e-6, 60
ADAPTIVE_STEPS = 16  # Krylov steps an adaptive run takes on these graphs (12 to 22 measured), for work()


def listed():
    return [
        # the plain method on a tiny graph: 20 backgrounds of 200 nodes. Latency of one whole call
        dict(name="tiny-er200", kind="scores", family="er", n=200, degree=19.9, graphs=1, reals=20, target="er",
             t=10, inner=0.3, dtype="f64", weights="ones", m=20, reorth=1, tune=False),
        # identification rate, ER 1024 nodes, degree 2, 40 backgrounds, 50 runs of a sparse 20-node target
        dict(name="monte-er1024", kind="monte", family="er", n=1024, degree=2.0, graphs=50, reals=40, target="er",
             t=20, inner=0.11, dtype="f64", weights="none", m=0, reorth=1, tune=False),
        # the same at 9000 nodes, degree 2.1, 20 backgrounds, 10 runs: several row blocks per realization
        dict(name="monte-er9000", kind="monte", family="er", n=9000, degree=2.1, graphs=10, reals=20, target="er",
             t=20, inner=0.11, dtype="f64", weights="none", m=0, reorth=1, tune=False),
        # batched realizations, the benchmark's default workload
        dict(name="batch-er1e5", kind="scores", family="er", n=100_000, degree=20.0, graphs=1, reals=64, target="er",
             t=50, inner=4 / 49, dtype="f32", weights="ones", m=30, reorth=1, tune=True),
        # single background, three graphs of a million nodes (ER, BA, WS), a 30-clique in each
        dict(name="single-1e6", kind="scores", family="mixed", n=1_000_000, n_min=1_000_000, degree=10.0,
             degree_min=10.0, mix=0, graphs=3, reals=1, target="clique", t=30, inner=1.0, dtype="f32",
             weights="ones", m=40, reorth=1, tune=True),
        # an uneven batch: families, sizes and degrees mixed, pattern only, adaptive dimension
        dict(name="uneven-12", kind="scores", family="mixed", n=500_000, n_min=10_000, degree=32.0, degree_min=8.0,
             mix=1409, graphs=12, reals=8, target="clique", t=40, inner=1.0, dtype="f32", weights="none", m=0,
             reorth=1, tune=True),
        # the memory-bounded form at an odd size
        dict(name="bounded-er99991", kind="scores", family="er", n=99_991, degree=15.0, graphs=1, reals=24,
             target="er", t=50, inner=4 / 49, dtype="f32", weights="random", m=30, reorth=0, tune=True),
        # differentiation: forward and backward of 16 realizations of 2e5 nodes
        dict(name="train-er2e5", kind="train", family="er", n=200_000, degree=16.0, graphs=1, reals=16, target="er",
             t=40, inner=3 / 39, dtype="f32", weights="random", m=30, reorth=1, tune=True),
        # refining 50 candidates by their subgraph centrality
        dict(name="central-er1e5", kind="central", family="er", n=100_000, degree=20.0, graphs=1, reals=1,
             target="er", t=50, inner=4 / 49, dtype="f32", weights="ones", m=20, count=50),
        # drawing the benchmark's batch on the device
        dict(name="generate-er1e5", kind="generate", family="er", n=100_000, degree=20.0, reals=64, t=50,
             inner=4 / 49),
        # drawing preferential-attachment backgrounds (hub rows) at an odd size
        dict(name="generate-ba300007", kind="generate", family="ba", n=300_007, degree=16.0, reals=8, t=30,
             inner=1.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["scores", "scores", "scores", "scores", "monte", "monte", "train", "central", "generate",
                       "generate"])
    family = rng.choice(["er", "er", "ba", "ws"])
    if kind == "generate":
        n, degree = int(_log(rng, 1000, 1_000_000)), 2 * rng.randint(1, 16)
        return dict(kind=kind, family=family, n=n, degree=float(degree),
                    reals=max(1, min(64, int(1.2e8 / (n * degree)))), t=rng.randint(10, 60),
                    inner=rng.choice([0.1, 1.0]))
    if kind == "central":
        n = int(_log(rng, 1000, 300_000))
        return dict(kind=kind, family=family, n=n, degree=float(2 * rng.randint(2, 12)), graphs=1, reals=1,
                    target="clique", t=20, inner=1.0, dtype=rng.choice(["f32", "f32", "f64"]),
                    weights=rng.choice(["none", "ones", "random"]), m=rng.randint(12, 30), count=rng.randint(1, 64))
    if kind == "monte":  # the tables' columns: 1024 to 9000 nodes, 1 to 40 backgrounds
        n, degree = int(_log(rng, 1000, 9000)), rng.choice([2.0, 2.9, 3.9, 4.9, 19.3, 39.0])
        reals = rng.choice([1, 2, 6, 20, 40])
        return dict(kind=kind, family=family if degree > 10 else "er", n=n, degree=degree,
                    graphs=max(1, min(rng.randint(1, 100), int(6e6 / (n * degree * reals)) + 1)), reals=reals,
                    target="clique" if degree > 10 else "er", t=20, inner=1.0 if degree > 10 else 0.11,
                    dtype=rng.choice(["f64", "f64", "f32"]), weights="none", m=0, reorth=1, tune=False)
    m = rng.choice([0, 20, 25, 30, 40]) if kind == "scores" else rng.randint(20, 36)
    reorth = rng.choice([0, 1, 1, 1, 1, 2]) if kind == "scores" else 1
    dtype = rng.choice(["f32", "f32", "f32", "f64"])
    n, degree = int(_log(rng, 200, 1_000_000)), rng.uniform(8.0, 32.0)
    entries = (6e7 if dtype == "f32" else 2.5e7) if kind == "scores" else (2.5e7 if dtype == "f32" else 1e7)
    c = dict(kind=kind, family=family, n=n, degree=degree, graphs=1,
             reals=max(1, min(rng.randint(1, 64), int(entries / (n * degree)))), target="clique",
             t=rng.randint(20, 50), inner=1.0, dtype=dtype,
             weights=rng.choice(["none", "ones", "random"]) if kind == "scores" else rng.choice(["ones", "random"]),
             m=m, reorth=reorth, tune=n > 2048)
    if kind == "train":
        c["family"] = "er"
    if kind == "scores" and n >= 20_000 and rng.random() < 0.4:  # an uneven batch
        c.update(family="mixed", n_min=max(10_000, n // 8), degree_min=8.0, mix=rng.randint(1, 1 << 20),
                 graphs=rng.randint(2, 8), reals=max(1, min(8, int(entries / (n * degree * 3)))))
    return c


# ---- the graphs of a case ---------------------------------------------------------------------------------------


def _specs(case):
    """(family, n, degree) of each graph (of all of them alike unless the case is mixed)."""
    if case["family"] != "mixed":
        return [(case["family"], case["n"], case["degree"])] * case["graphs"]
    r, out = random.Random(case["mix"]), []
    for g in range(case["graphs"]):
        n = case["n"] if case["n_min"] == case["n"] else r.randint(case["n_min"], case["n"])
        out.append((("er", "ba", "ws")[g % 3], n, r.uniform(case["degree_min"], case["degree"])))
    return out


def _edges(family, n, degree, R, gen, dev):
    """Edge keys (r n + a) n + b, a < b, of R realizations, unsorted and possibly repeated (ER: some to spare)."""
    if family == "er":
        count = int(1.05 * R * n * degree / 2) + 8 * R * int(degree * degree + 1)
        r = torch.randint(0, R, (count,), generator=gen, device=dev)
        a = torch.randint(0, n, (count,), generator=gen, device=dev)
        b = torch.randint(0, n - 1, (count,), generator=gen, device=dev)
        b += b >= a
    elif family == "ws":  # ring lattice of even degree k, a tenth of the far ends drawn anew
        h = max(1, int(round(degree / 2)))
        a = torch.arange(n, device=dev).repeat_interleave(h)
        b = (a + torch.arange(1, h + 1, device=dev).repeat(n)) % n
        r = torch.arange(R, device=dev).repeat_interleave(n * h)
        a, b = a.repeat(R), b.repeat(R)
        away = (a + 1 + torch.randint(0, n - 1, a.shape, generator=gen, device=dev)) % n
        b = torch.where(torch.rand(a.shape, generator=gen, device=dev) < 0.1, away, b)
    else:  # preferential attachment, k edges per new node: uniform endpoint slots of the earlier edges
        k = max(1, int(round(degree / 2)))
        src = torch.cat([torch.arange(1, k + 1, device=dev),
                         torch.arange(k + 1, n, device=dev).repeat_interleave(k)])
        before = k + (src - (k + 1)) * k
        slot = (torch.rand((R, src.numel()), generator=gen, device=dev, dtype=torch.float64)
                * (2 * before).clamp(min=1)).long()
        end = slot.clone()
        while True:  # an odd slot is the attached end of an earlier edge: follow it to a new node or the seed
            edge = end >> 1
            chase = ((end & 1) == 1) & (edge >= k)
            if not bool(chase.any()):
                break
            end = torch.where(chase, slot.gather(1, edge), end)
        b = torch.where((end & 1) == 0, src[end >> 1], torch.zeros_like(end))
        b[:, :k] = 0
        b = b.reshape(-1)
        a = src.repeat(R)
        r = torch.arange(R, device=dev).repeat_interleave(src.numel())
    return (r * n + torch.minimum(a, b)) * n + torch.maximum(a, b)


def _group(family, n, degree, graphs, reals, t, inner, gen, dev):
    """CSR of graphs x reals realizations of one family and size: row pointers [R, n + 1] of each realization,
    columns, entries per realization, the target nodes [graphs, t] and the pattern's local pairs."""
    R = graphs * reals
    targets = torch.rand((graphs, n), generator=gen, device=dev).argsort(1)[:, :t]
    pa, pb = torch.triu_indices(t, t, 1, device=dev)
    keep = torch.randperm(pa.numel(), generator=gen, device=dev)[: int(round(inner * pa.numel()))]
    pa, pb = pa[keep], pb[keep]
    keys = _edges(family, n, degree, R, gen, dev)
    inside = torch.zeros((graphs, n), dtype=torch.bool, device=dev)
    inside.scatter_(1, targets, True)
    g = keys // (n * n) // reals
    a, b = keys // n % n, keys % n
    keys = keys[(a != b) & ~(inside[g, a] & inside[g, b])]
    del g, a, b
    if family == "er":  # G(n, M): so many of the distinct edges
        keys = torch.unique(keys)
        keys = keys[torch.randperm(keys.numel(), generator=gen, device=dev)[: int(round(R * n * degree / 2))]]
    r = torch.arange(R, device=dev)[:, None]
    x, y = targets[:, pa].repeat_interleave(reals, 0), targets[:, pb].repeat_interleave(reals, 0)
    keys = torch.cat([keys, ((r * n + torch.minimum(x, y)) * n + torch.maximum(x, y)).reshape(-1)])
    keys = torch.unique(keys)
    r, a, b = keys // (n * n), keys // n % n, keys % n
    both = torch.cat([keys, (r * n + b) * n + a])
    del keys, r, a, b
    both = both.sort().values
    rows = both // n
    col = (both % n).to(torch.int32)
    del both
    deg = torch.bincount(rows, minlength=R * n).reshape(R, n)
    del rows
    rp = torch.zeros((R, n + 1), dtype=torch.int64, device=dev)
    torch.cumsum(deg, 1, out=rp[:, 1:])
    return rp, col, rp[:, -1].clone(), targets, torch.stack([pa, pb], 1)


def _weight(case, groups, dtype):
    """Edge weights in CSR order: ones, or symmetric weights in [0.5, 1.5) from the edge's ends."""
    if case["weights"] == "none":
        return None
    out = []
    for rp, col, nnz, *_ in groups:
        if case["weights"] == "ones":
            out.append(torch.ones(col.numel(), dtype=dtype, device=col.device))
            continue
        R, n = rp.shape[0], rp.shape[1] - 1
        row = torch.arange(n, device=col.device).repeat(R).repeat_interleave((rp[:, 1:] - rp[:, :-1]).reshape(-1))
        lo, hi = torch.minimum(row, col.long()), torch.maximum(row, col.long())
        h = (lo * 2654435761 + hi * 40503 + 12345) % 1000003
        h = (h * 69069 + 1) % 1048576
        out.append((0.5 + h.double() / 1048576).to(dtype))
    return torch.cat(out)


def _inputs(case, seed):
    """The case's graphs on the device, in groups of equal size and family."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1000003 + 17)
    specs = _specs(case)
    if case["family"] == "mixed":
        parts = [(f, n, d, 1) for f, n, d in specs]
    else:
        parts = [(*specs[0], case["graphs"])]
    return [_group(f, n, d, g, case["reals"], case["t"], case["inner"], gen, dev) for f, n, d, g in parts]


def _batch(case, seed):
    groups = _inputs(case, seed)
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    gn, gr, sizes, nnz = [], [], [], []
    for rp, col, z, targets, _ in groups:
        gn += [rp.shape[1] - 1] * targets.shape[0]
        gr += [case["reals"]] * targets.shape[0]
        sizes += [rp.shape[1]] * rp.shape[0]
        nnz.append(z.cpu().numpy())
    values = _weight(case, groups, dtype)
    if case["kind"] == "train":
        values.requires_grad_(True)
    b = api.Batch(gn, gr, np.concatenate([[0], np.cumsum(sizes)[:-1]]),
                  np.concatenate([[0], np.cumsum(np.concatenate(nnz))]),
                  torch.cat([g[0].reshape(-1) for g in groups]).to(torch.int32), torch.cat([g[1] for g in groups]),
                  values, case["dtype"])
    return b, values, groups


def _options(case):
    return dict(m=case["m"], tol=TOL, m_max=M_MAX, reorth=case["reorth"])


def _generate_args(case, seed):
    r = np.random.default_rng(int(seed) + 99)
    n, t = case["n"], case["t"]
    targets = r.choice(n, size=t, replace=False)
    a, b = np.triu_indices(t, 1)
    keep = r.random(a.size) < case["inner"]
    args = dict(family=case["family"], n=n, count=case["reals"], seed=int(r.integers(0, 1 << 62)), targets=targets,
                pattern=np.stack([a[keep], b[keep]], 1))
    if case["family"] == "er":
        args["p"] = case["degree"] / (n - 1)
    else:
        half = max(1, int(round(case["degree"] / 2)))
        args.update(k=2 * half, beta=0.1) if case["family"] == "ws" else args.update(k=half)
    return args


# ---- what is timed ----------------------------------------------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "generate":
        args = _generate_args(case, seed)  # the drawn columns go to the program's own arena
        slots = case["reals"] * (case["n"] * case["degree"] + case["t"] ** 2)
        arena = torch.zeros(int(slots + 12 * math.sqrt(2 * slots) + 64), dtype=torch.int32, device="cuda")
        return dict(kind=kind, args=args, arena=arena)
    if kind == "central":
        (group,) = _inputs(case, seed)
        rp, col, _, targets, _ = group
        nodes = targets[0].cpu().numpy()
        more = np.random.default_rng(int(seed)).choice(case["n"], size=case["count"])
        nodes = np.concatenate([nodes, more])[: case["count"]].astype(np.int32)
        dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
        return dict(kind=kind, row_ptr=rp[0].to(torch.int32), col=col, values=_weight(case, [group], dtype),
                    nodes=nodes, m=case["m"], dtype=case["dtype"])
    b, values, groups = _batch(case, seed)
    options = _options(case)
    if case["tune"]:
        b.tune(**options)
    s = dict(kind=kind, batch=b, options=options, K=case["t"])
    if kind == "scores":
        s["handle"] = b.run(**options)
    elif kind == "train":
        s["values"] = values
        s["cotangent"] = _cotangent(b, groups, values.dtype)
    return s


def _cotangent(b, groups, dtype):
    """The gradient of the loss that sums the target nodes' scores."""
    g, at = torch.zeros(b.total_scores, dtype=dtype, device="cuda"), 0
    for rp, _, _, targets, _ in groups:
        for k in range(targets.shape[0]):
            g[at + targets[k]] = 1.0
            at += rp.shape[1] - 1
    return g


def run(state):
    kind = state["kind"]
    if kind == "generate":
        row_ptr, col, nnz = api.generate(**state["args"])
        state["arena"][: col.numel()].copy_(col)
        return dict(row_ptr=row_ptr, columns=state["arena"], nnz=nnz)
    if kind == "central":
        return dict(centrality=api.subgraph_centrality(state["row_ptr"], state["col"], state["values"],
                                                       state["nodes"], m=state["m"], dtype=state["dtype"]))
    b = state["batch"]
    if kind == "train":
        scores, log_scale = api.Communicability.apply(state["values"], b, state["options"])
        (grad,) = torch.autograd.grad(scores, state["values"], state["cotangent"])
        return dict(scores=scores.detach(), log_scale=log_scale, grad=grad)
    out = state["handle"].launch() if kind == "scores" else b.scores(**state["options"])
    idx, val = b.topk(out.scores, state["K"])
    return dict(scores=out.scores, log_scale=out.log_scale, idx=idx, val=val)


def work(case):
    """Bytes and operations of one pass. A realization whose matrix and basis fit one compute unit's local memory reads
    its matrix once. Otherwise each Krylov step reads the matrix once and (with the stored basis) the basis vectors so
    far once, and writes one."""
    if case["kind"] == "generate":  # the CSR, written once
        z = case["reals"] * case["n"] * case["degree"]
        return dict(bytes=4 * z + 4.0 * case["reals"] * (case["n"] + 1), flops=10 * z)
    es = 8 if case["dtype"] == "f64" else 4
    ev = 0 if case["weights"] == "none" else es
    steps = case["m"] or ADAPTIVE_STEPS
    total, flops = 0.0, 0.0
    for family, n, degree in _specs(case):
        z, procs = n * degree, case["reals"]
        csr = 4 * (n + 1) + z * (4 + ev)
        if case["kind"] == "central":  # every process reads the one matrix
            procs = case["count"]
            csr /= procs
        basis = steps * (steps + 1) / 2 * n * es if case.get("reorth", 1) else 4 * steps * n * es
        passes = 2 if case.get("reorth", 1) == 0 or case["kind"] == "train" else 1
        one = passes * (steps * (csr + 2 * n * es) + basis)
        if case["kind"] != "central" and csr + steps * n * es <= 160 * 1024:
            one = csr
        if case["kind"] == "train":  # the forward call, its recomputation for the basis, the adjoint, the gradient
            one += steps * (csr + 2 * n * es) + basis + z * (4 + es) + 2 * steps * n * es
        total += procs * one + n * es
        flops += procs * passes * (steps * 2 * z + 2 * steps * (steps + 1) * n)
    return dict(bytes=total, flops=flops)


# ---- the same in 64 bits, with plain torch ----------------------------------------------------------------------


class _Product:
    """y = A x for R matrices of n rows side by side (x and y: [R, n])."""

    def __init__(self, rp, col, weight):
        self.R, self.n = rp.shape[0], rp.shape[1] - 1
        self.lengths = (rp[:, 1:] - rp[:, :-1]).reshape(-1)
        real = torch.arange(self.R, device=col.device).repeat_interleave(rp[:, -1])
        self.col = real * self.n + col.long()
        self.weight = weight

    def __call__(self, x):
        p = x.reshape(-1)[self.col]
        if self.weight is not None:
            p *= self.weight
        return torch.segment_reduce(p, "sum", lengths=self.lengths, unsafe=True).reshape(self.R, self.n)


def _lanczos(product, start, m):
    """Lanczos with two Gram-Schmidt passes: V [m][R, n], T [R, m + 1, m + 1] (of m steps, and the last beta beside
    them), ||start|| [R]. Once a process has closed its Krylov space, T goes on with a block of its own that
    exp(T) e1 does not see."""
    beta0 = start.norm(dim=1)
    V = [start / beta0[:, None]]
    T = torch.zeros((start.shape[0], m + 1, m + 1), dtype=torch.float64, device=start.device)
    alive = torch.ones_like(beta0, dtype=torch.bool)
    scale = torch.zeros_like(beta0)
    for j in range(m):
        w = product(V[j])
        a = torch.zeros_like(beta0)
        for _ in range(2):
            hs = [(v * w).sum(1) for v in V]
            a = a + hs[-1]
            for v, h in zip(V, hs):
                w = w - h[:, None] * v
        b = w.norm(dim=1)
        scale = torch.maximum(scale, a.abs())
        T[:, j, j] = torch.where(alive, a, torch.full_like(a, -1e4))
        alive = alive & (b > 1e-13 * scale)
        scale = torch.maximum(scale, b)
        b = torch.where(alive, b, torch.zeros_like(b))
        T[:, j, j + 1] = b
        T[:, j + 1, j] = b
        if j + 1 == m:
            break
        V.append(torch.where(alive[:, None], w / b.clamp(min=1e-300)[:, None], torch.zeros_like(w)))
    return V, T, beta0


def _exp_e1(T, adaptive=False):
    """Largest eigenvalue theta and exp(T - theta) e1 of each matrix; adaptive: of its first k rows, k the first where
    beta_k |y_k| / ||y|| is below the tolerance."""
    T = T.cpu()
    R, m = T.shape[0], T.shape[1] - 1
    theta, y = torch.zeros(R, dtype=torch.float64), torch.zeros((R, m), dtype=torch.float64)
    todo = torch.arange(R)
    for k in range(1 if adaptive else m, m + 1):
        w, q = torch.linalg.eigh(T[todo, :k, :k])
        yk = (q * torch.exp(w - w[:, -1:])[:, None, :] * q[:, :1, :]).sum(2)
        stop = T[todo, k - 1, k] * yk[:, -1].abs() < TOL * yk.norm(dim=1)
        if k == m:
            stop[:] = True
        theta[todo[stop]] = w[stop, -1]
        y[todo[stop], :k] = yk[stop]
        todo = todo[~stop]
        if not todo.numel():
            break
    return theta.cuda(), y.cuda()


def exact(case, seed):
    if case["kind"] == "generate":
        return None
    groups = _inputs(case, seed)
    kind, m = case["kind"], case["m"] or M_MAX
    # the weights as the framework gets them, rounded to its type
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32
    if kind == "central":
        rp, col = groups[0][:2]
        weight = _weight(case, groups, dtype)
        product = _Product(rp, col, None if weight is None else weight.double())
        more = np.random.default_rng(int(seed)).choice(case["n"], size=case["count"])
        nodes = np.concatenate([groups[0][3][0].cpu().numpy(), more])[: case["count"]]
        out = []
        for i in nodes:
            e = torch.zeros((1, case["n"]), dtype=torch.float64, device="cuda")
            e[0, int(i)] = 1.0
            theta, y = _exp_e1(_lanczos(product, e, m)[1])
            out.append(torch.exp(theta) * y[:, 0])
        return dict(centrality=torch.cat(out))
    scores, log_scale, grads = [], [], []
    for group in groups:
        rp, col, nnz, targets, _ = group
        weight = _weight(case, [group], dtype)
        product = _Product(rp, col, None if weight is None else weight.double())
        R, n, N = product.R, product.n, case["reals"]
        V, T, beta0 = _lanczos(product, torch.ones((R, n), dtype=torch.float64, device="cuda"), m)
        theta, y = _exp_e1(T, case["m"] == 0)
        u = torch.zeros((R, n), dtype=torch.float64, device="cuda")
        for i, v in enumerate(V):
            u += (beta0 * y[:, i])[:, None] * v
        sigma = theta.reshape(-1, N).max(1).values
        weightk = torch.exp(theta - sigma.repeat_interleave(N))
        scores.append((weightk[:, None] * u).reshape(-1, N, n).sum(1).reshape(-1))
        log_scale.append(sigma)
        if kind == "train":
            grads.append(_gradient(case, group, product, V, T, beta0, theta, sigma))
    out = dict(scores=torch.cat(scores), log_scale=torch.cat(log_scale))
    if kind == "train":
        return dict(out, grad=torch.cat(grads))
    return dict(out, idx=None, val=None)


def _gradient(case, group, product, V, T, beta0, theta, sigma):
    """e^-sigma (W X V')_ij on the pattern, X the upper right block of exp([[S, e1 e1'], [0, T]])."""
    rp, col, nnz, targets, _ = group
    R, n, m, N = product.R, product.n, T.shape[1] - 1, case["reals"]
    g = torch.zeros((R, n), dtype=torch.float64, device="cuda")
    g.scatter_(1, targets.repeat_interleave(N, 0), 1.0)
    W, S, gnorm = _lanczos(product, g, m)
    M = torch.zeros((R, 2 * m, 2 * m), dtype=torch.float64)
    M[:, :m, :m], M[:, m:, m:] = S[:, :m, :m].cpu(), T[:, :m, :m].cpu()
    M[:, 0, m] = 1.0
    shift = torch.maximum(theta, _exp_e1(S)[0])
    M -= shift.cpu()[:, None, None] * torch.eye(2 * m, dtype=torch.float64)
    X = torch.linalg.matrix_exp(M)[:, :m, m:].cuda()
    X *= (torch.exp(shift - sigma.repeat_interleave(N)) * gnorm * beta0)[:, None, None]
    Z = torch.einsum("arn,rab->rnb", torch.stack(W), X).reshape(R * n, m)
    Vn = torch.stack(V, 2).reshape(R * n, m)
    row = torch.arange(R * n, device="cuda").repeat_interleave(product.lengths)
    return torch.cat([(Z[i] * Vn[c]).sum(1) for i, c in zip(row.split(1 << 21), product.col.split(1 << 21))])
