"""GPU generator, assembly from bins of rows against the sorts: row pointers and columns equal the reference
generator's bit for bit (whole numbers: no tolerance) on either side of the rule and at the bins' edges."""
import ctypes

import numpy as np
import pytest

from tests.test_gpu_generate import SEED, check_against_oracle
from tests.test_gpu_parity import api

pytestmark = pytest.mark.gpu


def clique(t):
    return dict(targets=np.arange(t), pattern=[[a, b] for a in range(t) for b in range(a + 1, t)])


CASES = [
    # equal rows per bin (512 at degree 4, 256 at 17): one row short of whole bins, whole bins, one more
    ("er", 1023, 3, True, dict(p=4 / 1022)), ("er", 1024, 3, True, dict(p=4 / 1023)),
    ("er", 1025, 3, True, dict(p=4 / 1024)), ("er", 769, 2, True, dict(p=17 / 768)),
    # rows on both sides of 512 entries, the longest that are ranked; far above; a bin per row
    ("er", 2000, 2, True, dict(p=100 / 1999)), ("er", 2000, 2, True, dict(p=512 / 1999)),
    ("er", 2500, 1, True, dict(p=0.3)), ("er", 4001, 1, True, dict(p=1.0)),
    # more edges of a workgroup's 256 rows than its buffer of 8192
    ("er", 3000, 2, True, dict(p=0.05)),
    # the largest graph that is binned, and the first that is not
    ("er", 2 ** 21, 1, True, dict(p=2.0 ** -21)), ("er", 2 ** 21 + 1, 1, False, dict(p=2.0 ** -21)),
    ("ws", 1024, 3, True, dict(k=6, beta=0.3)), ("ws", 1500, 2, True, dict(k=200, beta=0.5)),
    # bins of equal expected entries: one, several; hubs beyond the LDS (sorted in memory)
    ("ba", 700, 3, True, dict(k=1)), ("ba", 9000, 3, True, dict(k=1)), ("ba", 9001, 2, True, dict(k=7)),
    ("ba", 4000, 2, True, dict(k=300)),
    # a pattern of up to 8192 entries in a bin (91 90 = 8190 and 92 91 = 8372), none of the background's inside
    ("er", 147, 3, True, dict(p=0.2, **clique(91))), ("er", 147, 3, False, dict(p=0.2, **clique(92))),
    ("er", 148, 3, False, dict(p=0.2, **clique(92))), ("ws", 900, 2, False, dict(k=4, beta=0.5, **clique(120))),
    ("ba", 2000, 2, False, dict(k=3, **clique(120))), ("ba", 2000, 2, True, dict(k=3, **clique(60))),
]


@pytest.mark.parametrize("family,n,count,binned,kw", CASES)
def test_bins_bitwise(gpu_lib, family, n, count, binned, kw):
    check_against_oracle(family, n, count, first=5, **kw)
    # the sorts hold at least 60 bytes per candidate edge, the bins 16
    from paper_1409_5000_amd import _abi as A
    spec, keep = api()._gen_spec(family, n, count, SEED, first=5, **kw)
    ws = ctypes.c_size_t()
    A.check(A.lib().ebtc_generate_plan(ctypes.byref(spec), ctypes.byref(ws)))
    per = {"er": kw.get("p", 0) * n * (n - 1) / 2, "ws": n * kw.get("k", 0) / 2, "ba": n * kw.get("k", 0)}[family]
    slots = count * (per + len(kw.get("pattern", ())))
    assert (ws.value < 12 * n * count + 32 * slots + 100_000) == binned


def test_two_threads_draw_graphs_of_different_sizes(gpu_lib):
    # 4096 bins need more than 64 KB of the scatter's LDS, one bin does not: each thread's launches take their own size
    import threading
    import torch
    specs = [dict(family="er", n=2 ** 21, count=1, seed=SEED, p=2.0 ** -20), dict(family="er", n=300, count=1, seed=SEED, p=0.1)]

    def draw(spec):
        rp, ci, nnz = api().generate(**spec)
        torch.cuda.current_stream().synchronize()
        return rp.cpu().numpy().tobytes(), ci.cpu().numpy().tobytes(), np.asarray(nnz).tolist()

    ref = [draw(s) for s in specs]
    wrong = []

    def loop(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(60):
                    if draw(specs[i]) != ref[i]:
                        wrong.append((i, "another graph"))
        except Exception as e:
            wrong.append((i, str(e)))

    threads = [threading.Thread(target=loop, args=(i,)) for i in (0, 1, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
