"""GPU: the general plain and compacting launches on few muons.  A small call without
a block size or pass length takes a shape of its own, so these give both: blocks of
256 and passes of 128 steps, against the oracle, against each other, twice, and as a
replayed graph."""
import dataclasses

import numpy as np
import pytest

from paper_2512_10520_amd import workloads as W
from tests._parity import compare, gpu_run, map_deltas, oracle_run

pytestmark = pytest.mark.gpu
PASSES = {"mode": "persistent", "block": 256, "compact_every": 128}


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    from paper_2512_10520_amd import _lib
    _lib.load()


@pytest.mark.parametrize("sampler", [0, 1], ids=["cdf", "alias"])
@pytest.mark.parametrize("name,opt,v", [("block", {}, 1), ("scan", {}, 3), ("scan", {}, 4),
                                        ("shield", {}, 1), ("shield", {"interp": 1}, 1),
                                        ("shield", {"stage_field": 1}, 1), ("blocks", {}, 1),
                                        ("logbins", {}, 1)])
def test_plain_and_passes(name, opt, v, sampler):
    wl = W.make_workload(name, n_muons=1500, n_fill=100_000, **({"n_variants": v} if v > 1 else {}))
    wl.run = dataclasses.replace(wl.run, sampler=sampler, **opt)
    g = gpu_run(wl, block=256)
    for kw in (PASSES, PASSES, {}, {"mode": "persistent"}):
        p = gpu_run(wl, **kw)
        for k in g:
            assert np.array_equal(g[k], p[k]), (kw, k)
    n = 200
    for var in range(v):
        o = oracle_run(wl, np.arange(n), variant=var if v > 1 else None)
        compare(g, o, sel=np.arange(var * 1500, var * 1500 + n), label=f"{name} {opt} v={var}",
                max_tie_frac=0.05, **(map_deltas(wl) if wl.field is not None else {}))


def test_replayed_passes():
    """A captured launch of several passes (survivor counts and lists of its own),
    replayed on other muons in the same buffers with eager work in between."""
    import torch
    from paper_2512_10520_amd import api
    wl = W.make_workload("shield", n_muons=8000, n_fill=100_000)
    api.load_workload(wl)
    all_muons = api.DeviceMuons.from_host(wl.muons)
    dm = api.DeviceMuons(all_muons.state[:, :2000].clone(), all_muons.q[:2000].clone())
    spec = api.RunSpec.from_workload(wl, use_graph=True, **PASSES)
    eager = api.RunSpec.from_workload(wl, mode="plain", block=256)
    out = api.alloc_result(spec, 2000, "cuda")
    for i in range(4):
        dm.state.copy_(all_muons.state[:, 2000 * i:2000 * (i + 1)])
        dm.q.copy_(all_muons.q[2000 * i:2000 * (i + 1)])
        api.propagate(dm, spec, out=out)
        want = api.propagate(dm, eager)
        torch.cuda.synchronize()
        for k in ("state", "status", "n_steps", "volume"):
            assert torch.equal(getattr(out, k), getattr(want, k)), (i, k)


@pytest.mark.parametrize("over", [0, 1], ids=["draws ahead", "many waves"])
def test_variant_waves_over_blocks(over):
    """Both sides of 5 waves a SIMD, where the variant-wave kernel changes."""
    import torch
    n = 5 * 4 * 64 * torch.cuda.get_device_properties(0).multi_processor_count // 8 + over
    wl = W.make_workload("blocks", n_muons=n, n_fill=20_000)
    wl.run = dataclasses.replace(wl.run, max_steps=300, n_variants=8)
    a = gpu_run(wl, mode="variant_waves")
    b = gpu_run(wl, mode="plain", block=256)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
