"""The solve of a few row blocks per workgroup, which the automatic schedule takes for batches of mid-sized graphs,
against the schedule of one launch per phase: the same scores, log-scales, diagnostics and checkpoints bit for bit, at
the edges of row blocks, of its LDS, of the ways it sums a row, and of the dot windows."""
import numpy as np
import pytest

from tests.test_gpu_single import api, assert_same, outputs, torch_mod

pytestmark = pytest.mark.gpu


def csr(n, degree, seed, hubs=()):
    rng = np.random.default_rng(seed)
    e = rng.integers(0, n, size=(int(n * degree / 2), 2))
    for row, entries in hubs:
        others = np.setdiff1d(np.arange(n), [row] + [h for h, _ in hubs])
        e = e[(e != row).all(1)]
        e = np.concatenate([e, np.stack([np.full(entries, row), rng.choice(others, entries, replace=False)], 1)])
    e = e[e[:, 0] != e[:, 1]]
    e = np.unique(np.concatenate([e, e[:, ::-1]]), axis=0)
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, e[:, 0] + 1, 1)
    return np.cumsum(rp).astype(np.int32), e[:, 1].astype(np.int32), e


def batch(graphs, dtype, weights):
    rps, cis, vals, noff = [], [], [], [0]
    for rp, ci, e in graphs:
        rps.append(rp)
        cis.append(ci)
        vals.append(0.5 + ((e.sum(1) * 31 + e.min(1) * 7) % 97) / 97.0)
        noff.append(noff[-1] + ci.size)
    roff = np.concatenate([[0], np.cumsum([r.size for r in rps])[:-1]]).astype(np.int64)
    n = [r.size - 1 for r in rps]
    v = np.concatenate(vals).astype(np.float64 if dtype == "f64" else np.float32) if weights else None
    return api().Batch(n, [1] * len(n), roff, np.array(noff, np.int64), np.concatenate(rps), np.concatenate(cis), v,
                       dtype)


def check(b, **kw):
    run = b.run(**kw)
    run.launch()
    assert run.profile()["solve"][1] == 1, "another schedule ran"
    assert_same(outputs(b, hipgraph=False, **kw), outputs(b, schedule="batched", hipgraph=False, **kw))


@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("dtype,n", [("f64", 2049), ("f64", 4096), ("f64", 4097), ("f64", 10200), ("f32", 2049),
                                     ("f32", 6145), ("f32", 14300)])
def test_row_blocks(gpu_lib, dtype, n, weights):
    # mixed sizes down to a single node, and enough realizations for the rule at the largest
    g = csr(n, 3, n)
    b = batch([g] * (160 if n > 5000 else 3) + [csr(max(1, n // 3), 2.5, 5), csr(2100, 3, 6), csr(1, 0, 1)], dtype,
              weights)
    check(b, m=0, tol=1e-8)


@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_rows(gpu_lib, dtype, weights):
    # one thread's rows (up to 128 entries, by eights), one wavefront's, the workgroup's (3072 and 6144 are the
    # stream form's capacities)
    small = csr(2500, 3, 3, [(0, 7), (1, 8), (64, 9), (2499, 128), (700, 129), (701, 192), (702, 193), (1500, 1000)])
    large = csr(7000, 3, 4, [(0, 3071), (17, 3073), (4096, 6144), (6999, 6200)])
    check(batch([small] * 4, dtype, weights), m=0, tol=1e-9)
    check(batch([large] * 150, dtype, weights), m=0, tol=1e-9)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_windows_and_breakdown(gpu_lib, dtype):
    # every dot window of a fixed dimension, an adaptive run to its cap; a graph without edges ends after its first step
    g = csr(2300, 4, 9)
    empty = (np.zeros(2101, np.int32), np.zeros(0, np.int32), np.zeros((0, 2), np.int64))
    b = batch([g] * 140 + [empty], dtype, False)
    for kw in (dict(m=8), dict(m=17), dict(m=33), dict(m=64), dict(m=0, tol=1e-30, m_max=30)):
        check(b, **kw)


@pytest.mark.parametrize("dtype,n,cap", [("f64", 10_000, 3072), ("f32", 14_000, 6144)])
def test_many_rows_beyond_the_capacity(gpu_lib, dtype, n, cap):
    # 133 rows beyond the stream form's capacity in each of 256 realizations, neighbours among them; no bound on their
    # number (fixed and adaptive dimension, with the first product's other order)
    import torch
    rng = np.random.default_rng(7)
    lengths = np.full(n, 2)
    lengths[rng.choice(n - 1, 120, replace=False)] = cap + 1
    lengths[n // 2:n // 2 + 10] = cap + np.arange(1, 20, 2)
    lengths[[0, 1, n - 1]] = [cap + 1, cap + 257, cap + 64]
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths]).astype(np.int32)
    R = 256
    b = api().Batch([n], [R], np.arange(R) * (n + 1), np.arange(R + 1) * ci.size, torch.as_tensor(rp).cuda().repeat(R),
                    torch.as_tensor(ci).cuda().repeat(R), None, dtype)
    check(b, m=8)
    check(b, m=0, tol=1e-8, m_max=40)


@pytest.mark.parametrize("dtype,n,entries,R,weights", [("f64", 4000, 200, 300, False), ("f32", 4000, 39, 300, True)])
def test_dense_graphs_stay_on_the_schedule_of_launches(gpu_lib, dtype, n, entries, R, weights):
    # the workgroup's solve takes 3.4 and 1.2 times as long here
    import torch
    rng = np.random.default_rng(11)
    ci = np.sort(rng.integers(0, n // entries, (n, entries)) + np.arange(entries) * (n // entries), axis=1)
    z = n * entries
    b = api().Batch([n], [R], np.arange(R) * (n + 1), np.arange(R + 1) * z,
                    torch.arange(0, z + 1, entries, dtype=torch.int32, device="cuda").repeat(R),
                    torch.as_tensor(ci.astype(np.int32).reshape(-1)).cuda().repeat(R),
                    torch.full((R * z,), 0.5, device="cuda") if weights else None, dtype)
    run = b.run(m=0)
    run.launch()
    assert run.profile()["solve"][1] == 0


@pytest.mark.parametrize("kw,solves", [(dict(m=1), 0), (dict(m=0, m_max=1), 0), (dict(m=2), 1)])
def test_one_step_of_a_pattern_stays_on_the_schedule_of_launches(gpu_lib, kw, solves):
    # one step of a pattern-only graph needs its degrees alone: no product that the workgroup's solve could save on
    b = api().generated_batch([dict(family="ba", n=5000, count=100, seed=3, k=4)], dtype="f64")
    run = b.run(**kw)
    run.launch()
    assert run.profile()["solve"][1] == solves
