"""GPU: launches that do not fill the chip (muons spread over the wavefronts, the
compacting form as one pass) give the bits of an explicit block size, which
always runs the general launch."""
import dataclasses

import numpy as np
import pytest

from paper_2512_10520_amd import workloads as W

pytestmark = pytest.mark.gpu
KEYS = ("state", "status", "n_steps", "volume")


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    from paper_2512_10520_amd import _lib
    _lib.load()


def _both(torch, wl, n, **kw):
    from paper_2512_10520_amd import api
    api.load_workload(wl)
    dm = api.DeviceMuons.from_host(wl.muons.take(np.arange(n)))
    dm.q[: n // 7] = torch.where(dm.q[: n // 7] > 0, 0, -1).to(torch.int8)    # some invalid
    sc = None
    if wl.run.scales is not None:
        sc = torch.from_numpy(np.ascontiguousarray(wl.run.scales, np.float32)).cuda()
    tally = {"z_det": 30.0, "r_ap": 1.0, "r_scale": 0.01}
    r = [api.propagate(dm, api.RunSpec.from_workload(wl, block=b, **kw), scales=sc, tally=tally)
         for b in (0, 256)]
    for k in KEYS + ("tally",):
        a, b = (getattr(x, k) for x in r)
        assert torch.equal(a.view(torch.int64) if k == "tally" else a,
                           b.view(torch.int64) if k == "tally" else b), (n, k)


# below and at the edges of every number of muons per wavefront (64 / 2^s), of
# the last ragged wavefront, and of the limit without a map (8192 on 256 CUs)
@pytest.mark.parametrize("mode", ["plain", "persistent"])
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 2047, 2049, 4097, 8191, 8192, 8193])
def test_block(n, mode):
    import torch
    _both(torch, W.make_workload("block", n_muons=n, n_fill=100_000), n, mode=mode)


@pytest.mark.parametrize("mode", ["plain", "persistent"])
@pytest.mark.parametrize("name,opt", [("shield", {}), ("shield", {"interp": 1}),
                                      ("shield", {"stage_field": 1}), ("blocks", {}),
                                      ("blocks", {"sampler": 1}), ("logbins", {"sampler": 1}),
                                      ("scan", {})])
@pytest.mark.parametrize("n", [37, 1001, 32_769])
def test_kernels(name, opt, mode, n):
    import torch
    if n > 2000 and (name in ("logbins", "scan") or opt):
        n = 2731
    kw = {"n_variants": 3} if name == "scan" else {}
    wl = W.make_workload(name, n_muons=n, n_fill=100_000, **kw)
    wl.run = dataclasses.replace(wl.run, max_steps=min(wl.run.max_steps, 600), **opt)
    _both(torch, wl, n, mode=mode)


@pytest.mark.parametrize("mode", ["plain", "persistent"])
@pytest.mark.parametrize("general", [True, False])
@pytest.mark.parametrize("opt", [{}, {"interp": 1}, {"sampler": 1}])
def test_few_waves(opt, general, mode):
    """Both sides of the limit of 4 waves a SIMD, where a map's kernels change."""
    wl = _few_waves_workload("shield", opt)
    if general:
        b = wl.field.b.copy()
        b[..., 0] += 0.02 * b[..., 1]
        b[..., 2] += np.float32(0.3) * np.gradient(b[..., 1], axis=0).astype(np.float32)
        wl.field = W.FieldMap(lo=wl.field.lo, hi=wl.field.hi, b=b)
    _few_and_many(wl, mode=mode)


@pytest.mark.parametrize("mode,compact", [("plain", 0), ("persistent", 0), ("persistent", 100)])
@pytest.mark.parametrize("opt,waves", [({}, 4), ({"sampler": 1}, 4), ({}, 5), ({}, 8)])
def test_few_waves_blocks(opt, waves, mode, compact):
    """The limits of 4, 5 and 8 waves a SIMD for convex blocks, in passes too."""
    _few_and_many(_few_waves_workload("blocks", opt, waves), mode=mode, compact_every=compact)


def _few_waves_workload(name, opt, waves=4):
    import torch
    edge = waves * 4 * 64 * torch.cuda.get_device_properties(0).multi_processor_count
    wl = W.make_workload(name, n_muons=edge + 1, n_fill=100_000)
    wl.run = dataclasses.replace(wl.run, max_steps=400, **opt)
    return wl


def _few_and_many(wl, **kw):
    import torch
    from paper_2512_10520_amd import api
    edge = len(wl.muons) - 1
    api.load_workload(wl)
    spec = api.RunSpec.from_workload(wl, **kw)
    dm = api.DeviceMuons.from_host(wl.muons)
    many = api.propagate(dm, spec)
    few = api.propagate(api.DeviceMuons.from_host(wl.muons.take(np.arange(edge))), spec)
    for k in KEYS:
        a, b = getattr(many, k), getattr(few, k)
        assert torch.equal(a[..., :edge], b), k


@pytest.mark.parametrize("n", [1, 65, 5000])
def test_checkpoints_and_gradients(n):
    """The tape and checkpoints of the lone-muon kernel, through the adjoint."""
    import torch
    from paper_2512_10520_amd import api
    wl = W.make_workload("diff", n_muons=n, n_fill=100_000)
    api.load_workload(wl)
    dm = api.DeviceMuons.from_host(wl.muons)
    sc = torch.from_numpy(np.ascontiguousarray(wl.run.scales, np.float32)).cuda()
    out = []
    for b in (0, 256):
        spec = api.RunSpec.from_workload(wl, block=b)
        f = api.propagate(dm, spec, scales=sc, ckpt=True)
        gx, gs = api.propagate_backward(dm, spec, f, torch.ones_like(f.state), scales=sc,
                                        n_mag=wl.geom.n_mag)
        m = int(f.n_steps.min())
        out.append((f.state, f.status, f.n_steps, f.tape[:m], f.ckpt[:m // 16], gx, gs))
    for a, b in zip(*out):
        assert torch.equal(a, b)
