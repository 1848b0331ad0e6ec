"""GPU: a muon of the compacting form resumed at any step starts with an exact
lookup, whatever bytes lie in the staged tables.  With convex blocks the region
test reads a record of planes; the momentum edges used here are ones that would
pass as such a record around a fresh lane, so that a lane tested against them
would keep flying through empty space."""
import dataclasses

import numpy as np
import pytest

from paper_2512_10520_amd import workloads as W
from tests import _custom as CU
from tests._parity import gpu_run

pytestmark = pytest.mark.gpu
KEYS = ("state", "status", "n_steps", "volume")
EDGES = [(0.18, 400.0, 20), (0.18, 160.0, 95), (0.3, 300.0, 9)]


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    from paper_2512_10520_amd import _lib
    _lib.load()


def _workload(edges, n, max_steps):
    """The blocks workload with other momentum bins (the same histogram in each)."""
    # least plane value and z clearance at (2, 2, 2) of the squared edges read as a
    # record of four float4 planes and a half height
    with np.errstate(all="ignore"):
        r = (W.log_edges(*edges) ** 2).view(np.float32)[:17].astype(np.float64)
        least = np.fmin.reduce(r[:16].reshape(4, 4) @ [2.0, 2.0, 2.0, 1.0])
        assert min(least, r[16] - 2.0) > 0.0
    wl = W.make_workload("blocks", n_muons=n, n_fill=2000)
    h = CU.flat_histograms(n_pbin=edges[2], p_lo=edges[0], p_hi=edges[1])
    wl.hist = dataclasses.replace(h, counts=np.ascontiguousarray(np.repeat(h.counts, 3, axis=0)))
    wl.run = dataclasses.replace(wl.run, max_steps=max_steps)
    return wl


@pytest.mark.parametrize("compact", [1, 32, 100, 128])
@pytest.mark.parametrize("edges", EDGES, ids=str)
def test_any_pass_length(edges, compact):
    # 63 steps: one step to a pass is the most that fits
    wl = _workload(edges, 3000, 63 if compact == 1 else 700)
    a = gpu_run(wl, block=256)
    b = gpu_run(wl, mode="persistent", block=256, compact_every=compact)
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k
    assert len(np.unique(a["volume"])) > (5 if compact > 1 else 0)


def test_default_pass_length_of_a_long_run():
    """Past 8191 steps a pass takes ceil((max_steps + 1) / 64) of them by default
    (141 here), and more than 5 waves a SIMD run in passes."""
    import torch
    n = 5 * 4 * 64 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    wl = _workload(EDGES[0], n, 9000)
    a = gpu_run(wl, block=256)
    b = gpu_run(wl, mode="persistent")
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k
