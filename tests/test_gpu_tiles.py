"""The paneled SpMV form's kernels at the sizes where they can go wrong, against the CSR-stream form, bit for
bit, through whole Lanczos runs: rows on both sides of each limit of the long-row path, more panels than one
load of the panel ends covers, bands of no, one and many rows, realizations of very different sizes in one
launch, columns out of order (a share of the stream arithmetic), shares that end early by their entries.

The form adds every row's products in entry order in FP64 as the stream form does, so the tolerance is zero.
"""
import numpy as np
import pytest

from fixtures import graphs as G

pytestmark = pytest.mark.gpu


def api():
    from paper_1409_5000_amd import api as _api
    return _api


def scored(b, **kw):
    import torch
    out = b.scores(schedule=kw.pop("schedule", "batched"), **kw)
    torch.cuda.synchronize()
    return out.scores.cpu().numpy().tobytes(), out.log_scale.cpu().numpy().tobytes(), out.diag_numpy().tobytes()


def csr(n, keys, rng, values):
    rp, ci = G.csr_from_keys(np.unique(keys[(keys // n) != (keys % n)]), n)
    return (rp, ci, 0.5 + rng.random(ci.size)) if values else (rp, ci)


def hubs(n, rows, rng):
    """A sparse background and rows of given lengths."""
    parts = [G.er_keys(n, 5.0 / (n - 1), rng)]
    for h, length in rows:
        parts.append(G.canon(np.full(length, h), rng.choice(n, length, replace=False), n))
    return np.concatenate(parts)


@pytest.mark.parametrize("dtype,values", [("f32", True), ("f32", False), ("f64", True), ("f64", False)])
def test_long_rows(gpu_lib, dtype, values):
    # around the long-row limit (256), a chunk of products (512), the stream form's capacity (6144 FP32,
    # 3072 FP64) and a batch of products (32768 FP32, 16384 FP64), many of them in one group of 64 rows
    n = 50_000
    rng = np.random.default_rng(3)
    rows = [(5, 240), (6, 249), (7, 255), (8, 262), (70, 500), (71, 513), (72, 1030), (9000, 3071), (9001, 3100),
            (9002, 6140), (9003, 6200), (30000, 16400), (30001, 33000), (49999, 40000)]
    rows += [(20000 + i, 300 + 7 * i) for i in range(80)]
    b = api().Batch.from_csr([[csr(n, hubs(n, rows, rng), rng, values)]], dtype=dtype)
    ref = scored(b, m=8, spmv="stream")
    assert scored(b, m=8, spmv="paneled") == ref
    assert scored(b, m=8, spmv="paneled", seg_len=700) == ref  # 72 panels: two loads of panel ends per band
    assert scored(b, m=8, spmv="paneled", schedule="plain") == ref


@pytest.mark.parametrize("dtype,values", [("f32", True), ("f64", False)])
def test_sizes_in_one_launch(gpu_lib, dtype, values):
    # empty, single-node and tiny graphs beside one of several shares; seg_len 100: more than 64 panels
    rng = np.random.default_rng(5)
    graphs = []
    for n in (1, 2, 3, 63, 64, 65, 511, 512, 513, 4097, 12160, 12161, 30011):
        d = min(8.0, max(0, n - 1))
        keys = G.er_keys(n, d / max(1, n - 1), rng) if n > 1 else np.empty(0, np.int64)
        graphs.append([csr(n, keys, rng, values), csr(n, np.empty(0, np.int64), rng, values)])
    b = api().Batch.from_csr(graphs, dtype=dtype)
    ref = scored(b, m=6, spmv="stream")
    for kw in (dict(), dict(seg_len=100), dict(seg_len=8191), dict(hipgraph=False), dict(schedule="plain")):
        assert scored(b, m=6, spmv="paneled", **kw) == ref, kw
    assert scored(b, m=6, spmv="paneled", reorth=0) == scored(b, m=6, spmv="stream", reorth=0)


def test_columns_out_of_order(gpu_lib):
    # two rows with swapped columns: their share takes the stream arithmetic, the other shares stay sorted
    n = 40_000
    rng = np.random.default_rng(7)
    rp, ci, va = csr(n, G.er_keys(n, 12.0 / (n - 1), rng), rng, True)
    for r in (17, 25_000):
        k = int(rp[r])
        assert rp[r + 1] - k >= 2
        ci[[k, k + 1]], va[[k, k + 1]] = ci[[k + 1, k]], va[[k + 1, k]]
    b = api().Batch.from_csr([[(rp, ci, va)]], dtype="f32")
    ref = scored(b, m=10, spmv="stream")
    assert scored(b, m=10, spmv="paneled") == ref
    assert scored(b, m=10, spmv="paneled", seg_len=1000) == ref


def test_shares_that_end_early(gpu_lib):
    # preferential attachment with 40 realizations: heads cut by entries, and the rows per share chosen anew
    n = 30_000
    rng = np.random.default_rng(9)
    reals = [csr(n, G.ba_keys(n, 8, rng), rng, False) for _ in range(40)]
    b = api().Batch.from_csr([reals], dtype="f32")
    ref = scored(b, m=0, tol=1e-6, m_max=40, spmv="stream")
    assert scored(b, m=0, tol=1e-6, m_max=40, spmv="paneled") == ref
    assert scored(b, m=0, tol=1e-6, m_max=40, spmv="paneled") == ref  # a replay


def test_adjoint_on_tiles(gpu_lib):
    # the adjoint's solve starts at the cotangent: step 0 runs the product kernel
    import torch
    n = 26_001
    rng = np.random.default_rng(11)
    rows = [(3, 700), (25_999, 4000)]
    b = api().Batch.from_csr([[csr(n, hubs(n, rows, rng), rng, True) for _ in range(2)]], dtype="f32")
    g = torch.as_tensor(rng.normal(size=n)).to("cuda")
    grads = []
    for form in ("stream", "paneled"):
        out = b.scores(m=12, schedule="batched", spmv=form)
        grads.append(b.scores_backward(out.log_scale, g, m=12, spmv=form).cpu().numpy().tobytes())
    assert grads[0] == grads[1]


@pytest.mark.parametrize("dtype,values", [("f32", True), ("f32", False), ("f64", True)])
def test_rows_with_many_entries_per_panel(gpu_lib, dtype, values):
    # rows of 1 to 250 entries in 1 to 4 neighbouring panels of 1000 columns: every class of entries (1st, 2nd, 3rd,
    # later ones of a row in a panel), at every place in the count's groups of 61, next to the long rows' limit
    n = 9000
    rng = np.random.default_rng(17)
    parts = []
    for h in range(0, n, 3):
        length, at = int(rng.integers(1, 251)), int(rng.integers(0, 5000))
        parts.append(G.canon(np.full(length, h), at + rng.choice(int(rng.integers(250, 4001)), length, replace=False), n))
    b = api().Batch.from_csr([[csr(n, np.concatenate(parts), rng, values)] * 3], dtype=dtype)
    ref = scored(b, m=8, spmv="stream")
    assert scored(b, m=8, spmv="paneled") == ref
    assert scored(b, m=8, spmv="paneled", seg_len=1000) == ref


def test_bands_longer_than_a_segment_of_the_count(gpu_lib):
    # 64 realizations of 20000 nodes, degree 50: bands of about 20000 entries, the count's segments hold 15616
    rng = np.random.default_rng(19)
    g = csr(20_000, G.er_keys(20_000, 50.0 / 19_999, rng), rng, False)
    b = api().Batch.from_csr([[g] * 64], dtype="f32")
    assert scored(b, m=6, spmv="paneled") == scored(b, m=6, spmv="stream")


@pytest.mark.parametrize("values", [True, False])
def test_plain_schedule_of_a_batch_of_many_rounds(gpu_lib, values):
    # 120 realizations of 10 shares: five rounds, so few spare share slots. All entries in 500 or 600 leading rows, long
    # ones or not, and one realization per launch: the shares are cut anew, and a share without a slot would leave its
    # rows' products unwritten (the workspace starts as NaN)
    import torch
    n, R = 100_000, 120
    rng = np.random.default_rng(23)
    for rows, length in ((500, 300), (600, 250)):
        ci = np.sort(rng.integers(0, n // length, (rows, length)) + np.arange(length) * (n // length), axis=1)
        rp = np.minimum(np.arange(n + 1), rows) * length
        va = torch.as_tensor(0.5 + rng.random(rows * length)).cuda().repeat(R) if values else None
        b = api().Batch([n], [R], np.arange(R) * (n + 1), np.arange(R + 1) * rows * length,
                        torch.as_tensor(rp.astype(np.int32)).cuda().repeat(R),
                        torch.as_tensor(ci.astype(np.int32).reshape(-1)).cuda().repeat(R), va, "f32")
        ref = scored(b, m=4, spmv="stream")
        for schedule in ("plain", "batched"):
            run = b.run(m=4, spmv="paneled", schedule=schedule)
            run.ws.fill_(255)
            out = run.launch()
            torch.cuda.synchronize()
            same = (out.scores.cpu().numpy().tobytes(), out.log_scale.cpu().numpy().tobytes(),
                    out.diag_numpy().tobytes()) == ref
            assert same, (rows, schedule)
            del run, out


def test_breakdown_beside_long_rows_of_others(gpu_lib):
    # 320 stars (two steps, then breakdown, found by the product launch of the third) between 320 graphs that go on, a
    # long row or more in each: more batches of long rows than workgroups that take them, stopped ones among them
    n = 700
    rng = np.random.default_rng(29)
    hub = np.arange(1, n)
    star = G.csr_from_keys(np.unique(G.canon(np.zeros(n - 1, np.int64), hub, n)), n)
    graphs = []
    for i in range(320):
        rows = [(int(h), int(rng.integers(280, 600))) for h in rng.choice(n, 1 + i % 3, replace=False)]
        graphs += [[star], [csr(n, hubs(n, rows, rng), rng, False)]]
    b = api().Batch.from_csr(graphs, dtype="f64")
    for kw in (dict(m=9), dict(m=0, tol=1e-8, m_max=30), dict(m=9, reorth=0)):
        ref = scored(b, spmv="stream", **kw)
        same = scored(b, spmv="paneled", **kw) == ref
        assert same, kw


def test_recorded_form_in_the_fixed_array(gpu_lib):
    # a recorded paneled form whose arenas pass the library's 64 MiB: the entry-balanced form, which fits, runs
    from paper_1409_5000_amd import _abi as A
    n = 60_000
    rng = np.random.default_rng(37)
    b = api().Batch.from_csr([[csr(n, G.er_keys(n, 36.0 / (n - 1), rng), rng, True) for _ in range(4)]], dtype="f32")
    assert b.run(m=5, spmv="paneled").ws_bytes > A.NOALLOC_WS_BYTES > b.run(m=5, spmv="balanced").ws_bytes
    b.set_forms(["paneled"])
    import torch
    for schedule in ("auto", "plain"):
        out = b.scores_noalloc(m=5, schedule=schedule)
        torch.cuda.synchronize()
        same = (out.scores.cpu().numpy().tobytes(), out.log_scale.cpu().numpy().tobytes(),
                out.diag_numpy().tobytes()) == scored(b, m=5, spmv="stream")
        assert same, schedule
    # a workspace planned under one schedule serves another
    run = b.run(m=5, schedule="plain")
    run.opts.schedule = api()._SCHED["batched"]
    assert run.launch().scores.cpu().numpy().tobytes() == scored(b, m=5, spmv="stream")[0]
    with pytest.raises(A.EbtcError):
        b.scores_noalloc(m=5, spmv="paneled")  # by name: as asked


@pytest.mark.parametrize("kw", [dict(m=1), dict(m=0, m_max=1), dict(m=1, reorth=0)])
def test_one_step_of_a_pattern_is_not_prepared_for(gpu_lib, kw):
    # it has no product: a recorded paneled form gives way to the balanced one, whose workspace is then enough
    n = 60_000
    rng = np.random.default_rng(59)
    b = api().Batch.from_csr([[csr(n, G.er_keys(n, 12.0 / (n - 1), rng), rng, False)]], dtype="f64")
    ref = scored(b, spmv="stream", **kw)
    need = b.run(spmv="balanced", **kw).ws_bytes
    assert need < b.run(spmv="paneled", **kw).ws_bytes
    b.set_forms(["paneled"])
    run = b.run(hipgraph=False, **kw)
    run.ws_bytes = need
    out = run.launch()
    same = (out.scores.cpu().numpy().tobytes(), out.log_scale.cpu().numpy().tobytes(), out.diag_numpy().tobytes()) == ref
    assert same


@pytest.mark.parametrize("n,R,weighted", [(40, 400_000, True), (6, 2_097_100, False)])
def test_more_places_than_one_launch_takes(gpu_lib, n, R, weighted):
    # two share slots a realization, twelve workgroups of 512 threads each in the sort (less than 2^32 threads a launch:
    # 350000 realizations), one of 1024 in the product (2097020); paths of n nodes with a chord
    import torch
    A = np.diag(np.ones(n - 1), 1)
    A[0, 2] = 1.0
    A = A + A.T
    rp = np.concatenate([[0], np.cumsum((A != 0).sum(1))]).astype(np.int32)
    ci = np.nonzero(A)[1].astype(np.int32)
    va = torch.linspace(0.5, 1.5, R * ci.size, dtype=torch.float32, device="cuda") if weighted else None
    b = api().Batch([n], [R], np.arange(R) * (n + 1), np.arange(R + 1) * ci.size,
                    torch.as_tensor(rp).cuda().repeat(R), torch.as_tensor(ci).cuda().repeat(R), va, "f32")
    kw = dict(m=4, schedule="batched", hipgraph=False)
    outs = []
    for form in ("stream", "paneled"):
        run = b.run(spmv=form, **kw)
        run.ws.fill_(255)
        out = run.launch()
        torch.cuda.synchronize()
        outs.append((out.scores.cpu().numpy().tobytes(), out.log_scale.cpu().numpy().tobytes(), out.diag_numpy().tobytes()))
        del run, out
    same = outs[0] == outs[1]
    assert same
    if weighted:  # the tuner tries the form on such a batch
        api().tune_cache_clear()
        assert "paneled" in b.tune(m=4)["ms_per_launch"]
        api().tune_cache_clear()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_second_pass_of_the_memory_bounded_form(gpu_lib, dtype):
    # step 0 of the second pass comes from the sorted entries: long rows on both sides of the stream form's capacity
    # (whose first product is in entry order, the others not), of a batch of products, and columns out of order
    n = 50_000
    rng = np.random.default_rng(43)
    rows = [(5, 257), (6, 300), (70, 1030), (9000, 3071), (9001, 3100), (9002, 6140), (9003, 6200), (30000, 16400),
            (30001, 33000)] + [(20000 + i, 260 + 9 * i) for i in range(70)]
    rp, ci, va = csr(n, hubs(n, rows, rng), rng, True)
    b = api().Batch.from_csr([[(rp, ci, va), csr(n, hubs(n, rows[:3], rng), rng, True)]], dtype=dtype)
    k = int(rp[40_000])
    assert rp[40_001] - k >= 2
    ci2, va2 = ci.copy(), va.copy()
    ci2[[k, k + 1]], va2[[k, k + 1]] = ci[[k + 1, k]], va[[k + 1, k]]
    c = api().Batch.from_csr([[(rp, ci2, va2)]], dtype=dtype)
    for batch in (b, c):
        for kw in (dict(m=8, reorth=0), dict(m=0, tol=1e-6, m_max=30, reorth=0),
                   dict(m=8, reorth=0, schedule="plain")):
            ref = scored(batch, spmv="stream", **kw)
            same = scored(batch, spmv="paneled", **kw) == ref
            assert same, kw


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("degree", [20, 48])
def test_second_pass_on_rows_of_many_entries(gpu_lib, dtype, degree):
    # the sorted entries give the second pass's step 0 from a mean of 32 entries per row on, the CSR below; columns out
    # of order in one realization, long rows on both sides of the stream form's capacity
    n = 17_000
    rng = np.random.default_rng(53)
    lengths = rng.integers(degree - 8, degree + 8, n)
    lengths[[0, 9, 10, 8000, 16999]] = [400, 3072, 3073, 6200, 9000]
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths]).astype(np.int32)
    va = rng.uniform(0.1, 1.0, rp[-1])
    k = int(rp[12_000])
    ci2, va2 = ci.copy(), va.copy()
    ci2[[k, k + 1]], va2[[k, k + 1]] = ci[[k + 1, k]], va[[k + 1, k]]
    b = api().Batch.from_csr([[(rp, ci, va), (rp, ci2, va2)]], dtype=dtype)
    for kw in (dict(m=6, reorth=0), dict(m=6, reorth=0, schedule="plain")):
        same = scored(b, spmv="paneled", **kw) == scored(b, spmv="stream", **kw)
        assert same, kw


@pytest.mark.parametrize("dtype,degree,long_row", [("f64", 620, 3500), ("f32", 1200, 6500)])
def test_rows_beyond_the_capacity_of_a_dense_graph(gpu_lib, dtype, degree, long_row):
    # six times the mean passes the stream form's capacity here: rows between the two are long rows all the same (the
    # stream form sums them in another order)
    n = 8000
    rng = np.random.default_rng(47)
    lengths = rng.integers(degree - 100, degree + 100, n)
    lengths[[3, 100, 101, 5000, 7999]] = long_row + np.array([0, 1, 2, 400, 64])
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lengths]).astype(np.int32)
    b = api().Batch.from_csr([[(rp, ci, 0.5 + rng.random(ci.size))] * 2], dtype=dtype)
    for kw in (dict(m=6), dict(m=6, reorth=0)):
        ref = scored(b, spmv="stream", **kw)
        same = scored(b, spmv="paneled", **kw) == ref
        assert same, kw
