"""GPU: the kernels for large histogram tables (narrow momentum bins, or many
histograms), against the FP64 oracle and, where every bin holds the same
histogram, against the ordinary kernels on a few wide bins, which then draw the
same losses: the same bits in every launch form."""
import dataclasses

import numpy as np
import pytest

from paper_2512_10520_amd import workloads as W
from tests import _custom as CU
from tests._parity import compare, gpu_run, oracle_run

pytestmark = pytest.mark.gpu
KEYS = ("state", "status", "n_steps", "volume")


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    from paper_2512_10520_amd import _lib
    _lib.load()


def _flat(n_pbin, n_mat):
    """The same histogram in every bin; losses up to 3 %."""
    h = CU.flat_histograms(n_pbin=n_pbin, p_lo=0.18, p_hi=400.0, loss=(0.0, 0.03), scat=(0.0, 5e-3))
    return dataclasses.replace(h, counts=np.ascontiguousarray(np.repeat(h.counts, n_mat, axis=0)))


def _pair(name, n, n_pbin, **kw):
    """The workload with narrow bins (wide kernels) and with 9 bins (ordinary ones)."""
    wl = W.make_workload(name, n_muons=n, n_fill=2000, **kw)
    wl.run = dataclasses.replace(wl.run, max_steps=400, p_min=2.5)   # in the middle of the bins
    m = wl.hist.counts.shape[0]
    return [dataclasses.replace(wl, hist=_flat(p, m)) for p in (n_pbin, 9)]


@pytest.mark.parametrize("sampler", [0, 1], ids=["cdf", "alias"])
@pytest.mark.parametrize("name,opt", [("shield", {}), ("shield", {"interp": 1}),
                                      ("shield", {"stage_field": 1}), ("blocks", {}),
                                      ("block", {}), ("block", {"stage_field": 1})])
@pytest.mark.parametrize("n_pbin", [401, 1024])
def test_launch_forms(name, opt, sampler, n_pbin):
    fine, coarse = _pair(name, 3001, n_pbin)
    for wl in (fine, coarse):
        wl.run = dataclasses.replace(wl.run, sampler=sampler, **opt)
    want = gpu_run(coarse, block=256)
    assert len(np.unique(want["status"])) > 1 and (want["status"] == 1).any()
    for kw in ({}, {"block": 256}, {"mode": "persistent", "block": 64, "compact_every": 37},
               {"mode": "variant_waves"}):
        got = gpu_run(fine, **kw)
        for k in KEYS:
            assert np.array_equal(got[k], want[k]), (kw, k)


@pytest.mark.parametrize("v", [1, 4, 12])
def test_variants(v):
    fine, coarse = _pair("scan", 700, 700, n_variants=v)
    want = gpu_run(coarse, block=256)
    for kw in ({"mode": "variant_waves"}, {"mode": "variant_waves", "block": 1024}, {}):
        got = gpu_run(fine, **kw)
        for k in KEYS:
            assert np.array_equal(got[k], want[k]), (kw, k)


def test_gradients():
    import torch
    from paper_2512_10520_amd import api
    got = []
    for wl in _pair("diff", 1500, 700):
        api.load_workload(wl)
        dm = api.DeviceMuons.from_host(wl.muons)
        sc = torch.linspace(0.9, 1.1, 8, dtype=torch.float32, device="cuda").reshape(1, 8)
        spec = api.RunSpec.from_workload(wl)
        f = api.propagate(dm, spec, scales=sc, ckpt=True)
        gx, gs = api.propagate_backward(dm, spec, f, torch.cos(f.state), scales=sc, n_mag=8)
        got.append((f.state, f.status, f.n_steps, f.volume, gx, gs))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n_mat,n_pbin,p_lo", [(1, 1024, 0.18), (3, 701, 0.5), (40, 95, 0.18),
                                               (4, 1024, 0.18)])
def test_against_the_oracle(n_mat, n_pbin, p_lo):
    """Histograms that differ from bin to bin, so that a wrong bin shows in the cells
    of the trace; enough muons that many histograms select the wide kernels too."""
    rng = np.random.default_rng([12, n_mat, n_pbin])
    counts = rng.integers(0, 40, (n_mat, n_pbin, 6, 5)).astype(np.uint32)
    counts[..., 0, 0] += 1
    hist = W.Histograms(p_edges=W.log_edges(p_lo, 400.0, n_pbin), loss_lo=0.0, loss_hi=0.04,
                        scat_lo=0.0, scat_hi=5e-3, counts=counts)
    box = [[-2, 2, -2, 2, 0.1 * i, 0.1 * i + 0.08] for i in range(60)]
    geom = CU.geometry(box, np.arange(60) % n_mat, b_box=np.tile([[0.1, 1.0, 0.0]], (60, 1)),
                       world=(2.5, 2.5, 5.5))
    n = 300_000 if n_mat == 40 else 2000
    p = np.exp(rng.uniform(np.log(0.4), np.log(60.0), n))
    t = rng.normal(0.0, 0.05, (2, n))
    mu = CU.muons(rng.uniform(-1, 1, n), rng.uniform(-1, 1, n), rng.uniform(0, 3.0, n),
                  p * np.sin(t[0]), p * np.sin(t[1]), p, rng.choice([-1, 1], n))
    wl = CU.workload(hist, geom, mu, max_steps=200, p_min=0.4)
    g = gpu_run(wl, trace_steps=200, n_trace=400)
    o = oracle_run(wl, np.arange(400), trace_steps=200)
    st = compare(g, o, trace_rows=400, label=f"{n_mat} x {n_pbin}")
    assert st["n"] == 400
    for kw in ({}, {"mode": "persistent", "block": 256, "compact_every": 50}):
        a = gpu_run(wl, **kw)
        for k in KEYS:
            assert np.array_equal(a[k], g[k]), (kw, k)
