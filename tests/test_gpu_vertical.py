"""GPU: kernels for vertical fields (every box, block and map field is (0, By,
0)) give the general kernels' results.  A trace request selects the general
kernels, so the same call with and without one must agree."""
import dataclasses

import numpy as np
import pytest

from paper_2512_10520_amd import workloads as W
from tests import _custom as CU
from tests._parity import gpu_run

pytestmark = pytest.mark.gpu
KEYS = ("state", "status", "n_steps", "volume")


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    from paper_2512_10520_amd import _lib
    _lib.load()


def _same(wl, **kw):
    a = gpu_run(wl, **kw)
    b = gpu_run(wl, trace_steps=4, n_trace=1, **kw)
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k
    return a


@pytest.mark.parametrize("sampler", [0, 1], ids=["cdf", "alias"])
@pytest.mark.parametrize("name", ["block", "scan", "logbins", "blocks"])
def test_without_map(name, sampler):
    kw = {"n_variants": 3} if name == "scan" else {}
    wl = W.make_workload(name, n_muons=1537, n_fill=100_000, **kw)
    wl.run = dataclasses.replace(wl.run, sampler=sampler, max_steps=700)
    _same(wl)
    _same(wl, mode="persistent", compact_every=100)
    if name == "scan":
        wl.run = dataclasses.replace(wl.run, stage_field=1)
        _same(wl)


@pytest.mark.parametrize("interp", [0, 1], ids=["trilinear", "nearest"])
@pytest.mark.parametrize("stage", [0, 1], ids=["held", "stages"])
@pytest.mark.parametrize("tilt", [0.0, 1e-30], ids=["vertical", "one node tilted"])
def test_with_map(interp, stage, tilt):
    """A map smaller than the world, negative zeros in the other components; with
    one tiny horizontal value the general kernels must be chosen by themselves
    and see it (here: the same results, it is far below rounding)."""
    rng = np.random.default_rng([7, interp, stage])
    b = np.zeros((9, 6, 7, 3), np.float32)
    b[..., 1] = rng.uniform(-1.5, 1.5, b.shape[:3])
    b[..., 0] = -0.0
    b[4, 3, 2, 2] = tilt
    f = W.FieldMap(lo=np.array([-0.6, -0.5, 0.3]), hi=np.array([0.6, 0.5, 1.9]), b=b)
    geom = CU.geometry([[-1, 1, -1, 1, 0, 1.2], [-1, 1, -1, 1, 1.2, 2.5]], [0, -1],
                       b_box=[[0.0, 0.4, -0.0], [0.0, 0.0, 0.0]], magnet=[0, -1], n_mag=1,
                       world=(1.5, 1.5, 2.4))
    n = 3001
    p = np.exp(rng.uniform(np.log(0.3), np.log(50.0), n))
    t = rng.normal(0.0, 0.2, (2, n))
    mu = CU.muons(rng.uniform(-0.8, 0.8, n), rng.uniform(-0.7, 0.7, n), rng.uniform(-0.1, 2.0, n),
                  p * np.sin(t[0]), p * np.sin(t[1]), p, rng.choice([-1, 1], n))
    wl = CU.workload(CU.flat_histograms(n_pbin=20, p_lo=0.2, p_hi=80.0), geom, mu, max_steps=300,
                     p_min=0.25, field=f, interp=interp, stage_field=stage,
                     scales=np.array([[1.1]], np.float32))
    a = _same(wl)
    assert len(np.unique(a["status"])) > 2
    if tilt == 0.0:
        return
    wl.field = W.FieldMap(lo=f.lo, hi=f.hi, b=np.where(np.abs(b) < 1e-20, 0.0, b).astype(np.float32))
    c = gpu_run(wl)
    for k in KEYS:
        assert np.array_equal(a[k], c[k]), k


@pytest.mark.parametrize("with_map", [False, True], ids=["boxes", "map"])
def test_gradients(with_map):
    """Checkpointed forward and adjoint: one more box with a horizontal field,
    behind the world, selects the general kernels without changing anything."""
    import torch
    from paper_2512_10520_amd import api
    wl = W.make_workload("diff", n_muons=1300, n_fill=100_000)
    if with_map:
        rng = np.random.default_rng(8)
        b = np.zeros((12, 6, 7, 3), np.float32)
        b[..., 1] = rng.uniform(-0.5, 0.5, b.shape[:3])
        wl.field = W.FieldMap(lo=np.array([-0.8, -0.9, 0.2]), hi=np.array([0.8, 0.9, 4.5]), b=b)
    g = wl.geom
    tilted = dataclasses.replace(
        g, box=np.vstack([g.box, [[-1, 1, -1, 1, 50, 51]]]), material=np.append(g.material, -1),
        b_box=np.vstack([g.b_box, [[1, 0, 0]]]).astype(np.float32), magnet=np.append(g.magnet, -1))
    got = []
    for geom in (g, tilted):
        api.load_workload(dataclasses.replace(wl, geom=geom))
        dm = api.DeviceMuons.from_host(wl.muons)
        sc = torch.linspace(0.9, 1.1, 8, dtype=torch.float32, device="cuda").reshape(1, 8)
        spec = api.RunSpec.from_workload(wl, block=64)
        f = api.propagate(dm, spec, scales=sc, ckpt=True)
        gx, gs = api.propagate_backward(dm, spec, f, torch.cos(f.state), scales=sc, n_mag=8)
        got.append((f.state, f.status, f.n_steps, f.volume, gx, gs))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert float(got[0][5].abs().min()) > 0


def test_overflowing_map_is_refused_and_the_loaded_one_stays():
    from paper_2512_10520_amd import api
    wl = W.make_workload("shield", n_muons=500, n_fill=50_000)
    a = gpu_run(wl)
    b = np.zeros((3, 3, 3, 3), np.float32)
    b[1, 1, 1, 1], b[1, 1, 2, 1] = 3e38, -3e38
    with pytest.raises(RuntimeError, match="overflows"):
        api.load_field(W.FieldMap(lo=np.zeros(3), hi=np.ones(3), b=b))
    dm = api.DeviceMuons.from_host(wl.muons)
    r = api.propagate(dm, api.RunSpec.from_workload(wl))
    assert np.array_equal(r.state.cpu().numpy(), a["state"])
