"""Subgraph centrality of several nodes at once (products formed together) against node by node (one process, the
CSR-stream products): bit for bit the same results, at the edges of the lanes, the tiles, the shares and the long
rows, with processes that end early."""
import numpy as np
import pytest

from tests.test_gpu_parity import api, torch_mod

pytestmark = pytest.mark.gpu


def graph(n, seed, hub_rows=(), degree=6, empty=()):
    """Symmetric CSR: random edges, rows of given numbers of entries, and rows with none."""
    rng = np.random.default_rng(seed)
    e = rng.integers(0, n, size=(n * degree // 2, 2))
    for row, entries in hub_rows:
        others = np.setdiff1d(np.arange(n), [row] + [h for h, _ in hub_rows] + list(empty))
        e = e[(e != row).all(1)]
        e = np.concatenate([e, np.stack([np.full(entries, row), rng.choice(others, entries, replace=False)], 1)])
    e = e[(e[:, 0] != e[:, 1]) & ~np.isin(e, list(empty)).any(1)]
    e = np.unique(np.concatenate([e, e[:, ::-1]]), axis=0)
    rp = np.zeros(n + 1, np.int32)
    np.add.at(rp, e[:, 0] + 1, 1)
    return np.cumsum(rp).astype(np.int32), e[:, 1].astype(np.int32), e


# a long row makes the products formed together the path of every one of these
CASES = [
    (4096, ((0, 1025),), (), 2), (4097, ((4096, 1025),), (0, 1), 16), (4159, ((64, 1100),), (5,), 17),
    (4160, ((63, 1100),), (), 33), (5000, ((7, 1025),), tuple(range(900, 1100)), 64), (4999, ((7, 1025),), (4998,), 65),
    (4099, ((1, 4000),), (), 130),
    (9000, ((0, 1023), (1, 1024), (40, 1025), (41, 1026), (8999, 3073)), (3,), 20),
    (20000, ((17, 6144), (18, 6145), (5000, 3072), (19999, 12000)), (), 50),
    (140000, ((139999, 2000),), (), 9),  # several rounds of shares
]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("n,hubs,empty,count", CASES)
def test_together_equals_one_by_one(gpu_lib, n, hubs, empty, count, weights, dtype):
    torch = torch_mod()
    rp, ci, e = graph(n, 7 * n + count, hubs, empty=empty)
    vals = None
    if weights:
        w = 0.05 + 0.01 * ((e.sum(1) * 37 + e.min(1)) % 89)  # symmetric
        vals = torch.tensor(w, dtype=torch.float64 if dtype == "f64" else torch.float32, device="cuda")
    rng = np.random.default_rng(n + count)
    special = [h for h, _ in hubs] + list(empty)[:2]  # an isolated node's process ends at once
    nodes = np.concatenate([special, rng.integers(0, n, size=count)])[:count].astype(np.int32)
    drp, dci = torch.tensor(rp, device="cuda"), torch.tensor(ci, device="cuda")
    got = api().subgraph_centrality(drp, dci, vals, nodes, m=12, dtype=dtype).cpu().numpy()
    some = range(count) if n <= 5000 else sorted({0, count // 2, count - 1})
    for i in some:
        one = api().subgraph_centrality(drp, dci, vals, nodes[i:i + 1], m=12, dtype=dtype).cpu().numpy()
        assert got[i].tobytes() == one[0].tobytes(), (i, nodes[i], got[i], one[0])


def test_a_workspace_for_the_processes_alone_is_taken(gpu_lib):
    torch = torch_mod()
    import ctypes

    from paper_1409_5000_amd import _abi as A
    n, count, m = 5000, 40, 8
    rp, ci, _ = graph(n, 11, ((7, 1025),))
    drp, dci = torch.tensor(rp, device="cuda"), torch.tensor(ci, device="cuda")
    nd = torch.arange(0, 40 * count, 40, dtype=torch.int32, device="cuda")
    need = ctypes.c_size_t()
    assert gpu_lib.ebtc_subgraph_centrality_ws_bytes(A.EBTC_F32, n, count, m, ctypes.byref(need)) == 0
    got = []
    for size in (need.value, need.value - 1):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out = torch.zeros(count, dtype=torch.float64, device="cuda")
        args = [ctypes.c_void_p(t.data_ptr()) for t in (drp, dci, nd, out, ws)]
        assert gpu_lib.ebtc_subgraph_centrality(A.EBTC_F32, n, args[0], args[1], None, count, args[2], m, args[3],
                                                args[4], size, None) == 0
        torch.cuda.synchronize()
        got.append(out.cpu().numpy().tobytes())
    assert got[0] == got[1]


# Whether one isolated long row makes the products formed together the path is a matter of times. A group of 256 rows that
# the stream form walks in several chunks does: the edges of CASES with eight to twelve long rows side by side.
GROUPS = [
    (4096, 1025, 12, (), 2), (4097, 1025, 12, (3000, 3001), 16), (4159, 1100, 12, (3000,), 17), (4160, 1100, 12, (), 33),
    (5000, 1025, 12, tuple(range(1900, 2100)), 64), (4999, 1025, 12, (4998,), 65), (4099, 4000, 8, (), 130),
    (20000, 6144, 9, (300,), 50), (20000, 3073, 9, (), 3), (140000, 2000, 12, (), 9),
]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("n,length,rows,empty,count", GROUPS)
def test_long_rows_side_by_side(gpu_lib, n, length, rows, empty, count, weights, dtype):
    hubs = tuple((256 + i, length + i % 2) for i in range(rows))
    test_together_equals_one_by_one(None, n, hubs, empty, count, weights, dtype)
