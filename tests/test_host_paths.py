"""CPU: the library's host code on a HIP runtime of host memory (no kernel runs):
what the loaders keep on the device, and what the launches ask for."""
import dataclasses

import numpy as np
import pytest

from paper_2512_10520_amd import workloads as W
from tests import _custom as CU
from tests import _host_stub

MODES = {"plain": 0, "persistent": 1, "variant_waves": 2}


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return _host_stub.build(tmp_path_factory.mktemp("stub"))


def _tables(n_pbin, n_mat, loss=(0.0, 0.05)):
    h = CU.flat_histograms(n_pbin=n_pbin, p_lo=0.18, p_hi=400.0, loss=loss)
    return dataclasses.replace(h, counts=np.ascontiguousarray(np.repeat(h.counts, n_mat, axis=0)))


def _boxes(n=64):
    return CU.geometry([[-1, 1, -1, 1, i, i + 0.9] for i in range(n)], [0] * n)


def _blocks(n=64):
    q = [-1, -1, 1, -1, 1, 1, -1, 1]
    return CU.geometry([], [0] * n, poly=[[i, i + 0.9] + q + q for i in range(n)])


# ---- staged tables ---------------------------------------------------------
def staged(s, n_pbin, n_mat, blocks, loss, n, limit, wide):
    assert s.histograms(_tables(n_pbin, n_mat, loss)) == 0
    assert s.geometry(_blocks() if blocks else _boxes()) == 0
    for mode in (0, 1):
        assert s.propagate(s.params(mode=mode, block=256), n) == 0
        for l in s.launches():
            if "k_plain" in l.name or "k_pass" in l.name:
                mask = int(l.name.split("ILj")[1].split("E")[0])
                assert l.lds <= limit, l
                assert bool(mask & 4) == wide, l


@pytest.mark.parametrize("n_pbin,n_mat,blocks,loss,n,limit,wide", [
    # the largest tables (limit: edges, totals and geometry alone)
    (1024, 4, False, (0.0, 0.05), 10 ** 6, 30_240, True),
    (1024, 4, True, (0.0, 0.05), 10 ** 6, 44_552, True),
    (95, 43, False, (0.0, 0.05), 10 ** 6, 30_240, True),
    (95, 43, False, (0.0, 0.05), 50_000, 10 ** 6, False),    # all blocks resident at once
    # narrow bins or not, by the losses of a step
    (600, 1, False, (0.0, 0.02), 10 ** 6, 30_240, True),
    (400, 1, False, (0.0, 0.02), 10 ** 6, 30_240, False),
    (1024, 1, False, (0.0, 0.005), 10 ** 6, 30_240, False),
    (95, 3, False, (0.0, 0.05), 10 ** 6, 30_240, False)])
def test_staged_tables(stub, n_pbin, n_mat, blocks, loss, n, limit, wide):
    _host_stub.run(stub, "tests.test_host_paths", "staged", n_pbin, n_mat, blocks, loss, n, limit,
                   wide)


# ---- lone muons ------------------------------------------------------------
def lone(s, n_mat, blocks, n):
    assert s.histograms(_tables(95, n_mat)) == 0
    assert s.geometry(_blocks() if blocks else _boxes()) == 0
    for mode in (0, 1):
        assert s.propagate(s.params(mode=mode), n) == 0
        (l,) = s.launches()
        assert "k_variant_waves" in l.name and l.block == 64
        assert l.grid <= 256 * min(4, 160 * 1024 // l.lds), l


@pytest.mark.parametrize("n", [1, 1000, 2000, 4097, 8192])
@pytest.mark.parametrize("n_mat,blocks", [(1, False), (43, False), (20, True), (43, True)])
def test_lone_muons_are_resident_at_once(stub, n_mat, blocks, n):
    """One wave a SIMD, or as many as the staged tables leave room for."""
    _host_stub.run(stub, "tests.test_host_paths", "lone", n_mat, blocks, n)


# ---- passes ----------------------------------------------------------------
def one_pass(s):
    assert s.histograms(_tables(95, 1)) == 0
    assert s.geometry(_boxes()) == 0
    for max_steps in (0, 1, 1000, 2 ** 31 - 1):
        p = s.params(mode=1, max_steps=max_steps)
        assert s.propagate(p, 10 ** 6, noalloc=True) == 0       # no lists to park muons in
        assert [l.name.count("k_pass") for l in s.launches()] == [1], max_steps
        assert s.propagate(p, 60_000) == 0                      # all resident at once
        assert len(s.launches()) == 1, max_steps
        assert s.propagate(s.params(mode=1, max_steps=max_steps, compact_every=2 ** 31 - 1),
                           10 ** 6) == 0
        names = [l.name for l in s.launches()]
        assert len(names) == (1 if max_steps < 2 ** 31 - 1 else 3), (max_steps, names)


def test_one_pass_at_any_step_cap(stub):
    _host_stub.run(stub, "tests.test_host_paths", "one_pass")


# ---- loaders that fail -----------------------------------------------------
def failing_loads(s, kind):
    """Each allocation and each copy of a load fails in turn: what was loaded keeps
    working, with its own tables."""
    small, large = _tables(20, 1), _tables(95, 8)
    loads = {"histograms": lambda: s.histograms(large), "boxes": lambda: s.geometry(_boxes(60)),
             "blocks": lambda: s.geometry(_blocks(60))}
    runs = [s.params(mode=1, block=256, sampler=k) for k in (0, 1)]

    def launch():
        for p in runs:
            assert s.propagate(p, 500_000) == 0
        got = s.launches()
        assert got and all(l.tables_live for l in got)
        return got

    assert s.histograms(small) == 0 and s.geometry(_boxes(5)) == 0
    launch()
    used, failures = s.c.stub_used(), 0
    for fail in (s.c.stub_fail_alloc, s.c.stub_fail_copy):
        for nth in range(10):
            assert s.histograms(small) == 0 and s.geometry(_boxes(5)) == 0
            before = launch()
            fail(nth)
            rc = loads[kind]()
            fail(-1)
            if rc == 0:
                break
            failures += 1
            assert rc in (-5, -6)
            assert launch() == before, (fail, nth)
    assert failures >= 2
    assert s.histograms(small) == 0 and s.geometry(_boxes(5)) == 0
    assert s.c.stub_used() == used


@pytest.mark.parametrize("kind", ["histograms", "boxes", "blocks"])
def test_a_load_that_fails_leaves_what_was_loaded(stub, kind):
    _host_stub.run(stub, "tests.test_host_paths", "failing_loads", kind)


def tight_histograms(s):
    assert s.histograms(_tables(95, 8)) == 0 and s.geometry(_boxes(5)) == 0
    p = s.params(mode=0, block=256)
    assert s.propagate(p, 500_000) == 0
    before = s.launches()
    used = s.c.stub_used()
    s.c.stub_limit(used + 50_000)                  # no room for two sets of tables
    assert s.histograms(_tables(95, 100)) == -7    # (more than the documented limit)
    assert s.histograms(_tables(95, 40)) == -5     # too large by themselves: the loaded ones stay
    assert s.propagate(p, 500_000) == 0 and s.launches() == before
    assert s.histograms(_tables(95, 8)) == 0       # in place of the loaded ones
    assert s.propagate(p, 500_000) == 0 and s.launches() == before
    assert s.c.stub_used() == used


def test_histograms_that_do_not_fit_beside_the_loaded_ones(stub):
    _host_stub.run(stub, "tests.test_host_paths", "tight_histograms")


# ---- field maps ------------------------------------------------------------
def maps(s):
    assert s.histograms(_tables(95, 1)) == 0 and s.geometry(_boxes(5)) == 0
    assert s.propagate(s.params(block=256), 500_000) == 0      # (with the workspaces)
    s.launches()
    used = s.c.stub_used()

    def field(n, vertical):
        b = np.zeros((n, n, n, 3), np.float32)
        b[..., 1] = 1.0
        b[..., 0] = 0.0 if vertical else 0.5
        return b

    def mask():
        assert s.propagate(s.params(block=256), 500_000) == 0
        (l,) = [l for l in s.launches() if "k_plain" in l.name]
        return int(l.name.split("ILj")[1].split("E")[0]) & (1 | 256)

    general = 128 * 89 ** 3 + 16 * 90 ** 3              # bytes of a map of 90^3 nodes
    vertical = general + 32 * 89 ** 3 + 4 * 90 ** 3
    piece = 12 * 90 ** 3
    # room for one map and the node values in flight
    s.c.stub_limit(used + general + piece + 4096)
    for _ in range(2):
        assert s.field(field(90, False)) == 0           # replaces one of its size
        assert mask() == 1
    assert s.field(field(90, True)) == 0                # its own tables do not fit
    assert mask() == 1
    assert s.field(field(95, False)) == -5              # too large by itself: the loaded one stays
    assert mask() == 1
    s.c.stub_limit(used + vertical + piece + 4096)
    for _ in range(2):
        assert s.field(field(90, True)) == 0
        assert mask() == 1 | 256
    # a map that is refused, and copies and allocations that fail
    b = field(90, True)
    b[0, 0, 1, 1], b[0, 0, 0, 1] = 3e38, -3e38
    assert s.field(b) == -1 and mask() == 1 | 256
    s.c.stub_limit(1 << 40)
    for fail in (s.c.stub_fail_alloc, s.c.stub_fail_copy):
        for nth in range(8):
            fail(nth)
            rc = s.field(field(60, False))
            fail(-1)
            if rc == 0:
                assert mask() == 1
                assert s.field(field(90, True)) == 0
                break
            assert rc in (-5, -6) and mask() == 1 | 256
    s.launches()
    assert s.L.mt_load_field(0, 0, 0, None, None, None) == 0
    assert mask() == 256 and s.c.stub_used() == used


def test_map_that_does_not_fit_beside_the_loaded_one(stub):
    _host_stub.run(stub, "tests.test_host_paths", "maps")


# ---- autotuner -------------------------------------------------------------
def tuned(s, n, cheap, want):
    assert s.histograms(_tables(95, 1)) == 0 and s.geometry(_boxes(5)) == 0
    s.c.stub_cheap(cheap.encode())
    for bad in ({"block": 96}, {"compact_every": -1}, {"step_m": 0.0}):
        assert s.autotune(s.params(mode=1, **bad), n)[0] == -1
    rc, block, compact, ms = s.autotune(s.params(mode=1), n)
    assert rc == 0 and block in (64, 128, 256, 512) and compact in (32, 64, 128, 256, 512, 1 << 30)
    s.launches()
    assert s.propagate(s.params(mode=1), n) == 0
    assert want in s.launches()[-1].name
    assert s.propagate(s.params(mode=1, block=64, compact_every=1 << 30), n) == 0
    assert "k_variant_waves" not in s.launches()[-1].name     # given shapes are not tuned


@pytest.mark.parametrize("n,cheap,want", [(2000, "k_variant_waves", "k_variant_waves"),
                                          (2000, "k_plain", "k_plain"),
                                          (500_000, "k_pass", "k_pass")])
def test_autotune_times_the_untuned_shape(stub, n, cheap, want):
    """Lone muons are a candidate like the others, and remembered if they win."""
    _host_stub.run(stub, "tests.test_host_paths", "tuned", n, cheap, want)


# ---- the entry point that allocates nothing --------------------------------
def same_kernels(s):
    assert s.histograms(_tables(95, 1)) == 0 and s.geometry(_boxes(5)) == 0
    for n in (1, 2000, 8192, 8193, 60_000):
        for mode in (0, 1, 2):
            for block in (0, 128):
                p = s.params(mode=mode, block=block)
                assert s.propagate(p, n) == 0
                want = s.launches()
                used = s.c.stub_used()
                assert s.propagate(p, n, noalloc=True) == 0
                got = s.launches()
                assert s.c.stub_used() == used
                if mode != 1 or block == 0:         # (given a block, passes need lists)
                    assert got == want, (n, mode, block)


def test_noalloc_launches_the_same_kernels(stub):
    _host_stub.run(stub, "tests.test_host_paths", "same_kernels")
