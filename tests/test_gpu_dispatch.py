"""Autotuned calls on both sides of what the LDS-resident sweeps hold (1024
receivers of a shot, 128 sponge cells) against named z sweeps.

Every form has the same operations in the same order.  Two reverse steps per
launch, named or tuned, come with an even snapshot spacing: the named call
takes the tuned one's reverse steps, and all results have the same bits.
"""
import re

import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid, gaussian_anomaly, random_traces, ricker

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,nrec", [(20, 60), (20, 1025), (129, 60)])
def test_tuned_calls_have_the_named_sweeps_bits(N, nrec):
    nx, nz, ns, nt = 200, 90, 3, 118
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 15.0)
    iz, ix = np.divmod(np.arange(nrec, dtype=np.int32), nx)
    geom = Geometry(np.full(ns, 4, np.int32), np.array([5, 100, 190], np.int32),
                    np.arange(ns + 1, dtype=np.int32) * nrec, np.tile(iz, ns), np.tile(ix, ns),
                    np.array([nt, nt - 7, nt - 40], np.int32))
    wav = ricker(14.0, 1e-3, nt).astype(np.float32)
    d = random_traces(geom, nt, seed=5, scale=1e-2)

    def calls(ex):
        return [B.forward(v, wav, grid, geom, ex), B.hessian_diag(v, wav, grid, geom, B.HESS_EQ1, exec_=ex),
                *B.gradient(v, wav, grid, geom, d, "int", ex, hmax=2)]
    tuned = B.make_exec(autotune=1)
    a = calls(tuned)
    steps = B.fwi_exec_query(grid, geom, tuned, B.WS_GRADIENT)["reverse_steps"]
    b = calls(B.make_exec(tile_rows=16, reverse_steps=steps, graph_steps=-1))
    for k, (x, y) in enumerate(zip(a, b)):
        assert bool(torch.isfinite(x).all()) and float(x.abs().max()) > 0, k
        assert torch.equal(x, y), k


def test_lds_resident_calls_are_not_timed(capfd, monkeypatch):
    """Where every sweep of a tuned call runs LDS-resident no candidate is
    timed and the results have the untuned call's bits, snapshot spacing
    included; in a workspace of the z sweeps' size the same call is timed."""
    monkeypatch.setenv("FWI_TUNE_LOG", "1")
    nx, nz, ns, nt = 90, 50, 2, 119    # 11 steps between the snapshots of the first shot, 12 at an even spacing
    grid = Grid(nz, nx, 10.0, 1e-3, nt, 10, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 9.0)
    ix = np.arange(0, nx, 5, dtype=np.int32)
    geom = Geometry(np.full(ns, 3, np.int32), np.array([5, 80], np.int32), np.arange(ns + 1, dtype=np.int32) * len(ix),
                    np.full(ns * len(ix), 1, np.int32), np.tile(ix, ns), np.array([nt, nt - 19], np.int32))
    wav = ricker(14.0, 1e-3, nt).astype(np.float32)
    d = random_traces(geom, nt, seed=5, scale=1e-2)
    tuned = B.make_exec(autotune=1)

    def timed(call):
        out = call()
        torch.cuda.synchronize()
        return out, capfd.readouterr().err.count("[fwi tune]")

    a, n = timed(lambda: B.gradient(v, wav, grid, geom, d, "int", tuned))
    assert n == 0
    b, n = timed(lambda: B.gradient(v, wav, grid, geom, d, "int", None))
    assert n == 0 and all(torch.equal(x, y) for x, y in zip(a[:3], b[:3]))
    ref, n = timed(lambda: B.forward(v, wav, grid, geom, tuned))
    assert n == 0
    size = B.fwi_workspace_bytes(grid, geom, B.make_exec(tile_rows=32), B.WS_FORWARD)
    assert size < B.fwi_workspace_bytes(grid, geom, tuned, B.WS_FORWARD)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    got, n = timed(lambda: B.forward(v, wav, grid, geom, tuned, ws=ws))
    assert n > 0 and torch.equal(got, ref)


@pytest.mark.parametrize("ex", [{}, dict(forward_steps=2, reverse_steps=2)])
def test_the_least_workspace_gives_the_same_bits(ex):
    """The z sweeps without an arrival map, in exactly the bytes that a
    refused call asks for."""
    nx, nz, N, nt = 290, 60, 15, 90
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 15.0)
    ix = np.arange(0, nx, 4, dtype=np.int32)
    geom = Geometry(np.array([3, 40], np.int32), np.array([7, 250], np.int32), np.arange(3, dtype=np.int32) * len(ix),
                    np.full(2 * len(ix), 2, np.int32), np.tile(ix, 2), np.array([nt, nt - 9], np.int32))
    wav = ricker(14.0, 1e-3, nt).astype(np.float32)
    d = random_traces(geom, nt, seed=5, scale=1e-2)
    ex = B.make_exec(**ex)
    for what, call in ((B.WS_GRADIENT, lambda ws: B.gradient(v, wav, grid, geom, d, "int", ex, hmax=2, ws=ws)),
                       (B.WS_EXTIMAGE, lambda ws: B.extended_image(v, wav, grid, geom, d, 2, "int", ex, ws=ws))):
        with pytest.raises(B.FwiError) as e:
            call(torch.empty(16, dtype=torch.uint8, device="cuda"))
        need = int(re.search(r"need (\d+)", str(e.value)).group(1))
        assert need < B.fwi_workspace_bytes(grid, geom, ex, what, 2)
        small, full = call(torch.empty(need, dtype=torch.uint8, device="cuda")), call(None)
        assert all(torch.equal(x, y) for x, y in zip(small, full))


def test_tuned_image_past_the_lds_resident_sizes():
    """An autotuned extended image of 1.8 M cells a step in the workspace that
    is reported for it, against the named call of the tuned steps."""
    nx, nz, ns, nt = 1000, 400, 4, 70
    grid = Grid(nz, nx, 10.0, 1e-3, nt, 20, 2300.0)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 15.0)
    ix = np.arange(0, nx, 10, dtype=np.int32)
    geom = Geometry(np.full(ns, 4, np.int32), np.array([100, 300, 600, 900], np.int32),
                    np.arange(ns + 1, dtype=np.int32) * len(ix), np.full(ns * len(ix), 2, np.int32), np.tile(ix, ns),
                    np.full(ns, nt, np.int32))
    wav = ricker(20.0, 1e-3, nt).astype(np.float32)
    d = random_traces(geom, nt, seed=5, scale=1e-2)
    tuned = B.make_exec(autotune=1)
    a = B.extended_image(v, wav, grid, geom, d, 3, "l2", tuned)
    steps = B.fwi_exec_query(grid, geom, tuned, B.WS_EXTIMAGE)["reverse_steps"]
    b = B.extended_image(v, wav, grid, geom, d, 3, "l2", B.make_exec(tile_rows=16, reverse_steps=steps))
    for x, y in zip(a, b):
        assert float(x.abs().max()) > 0 and torch.equal(x, y)


def test_exact_diagonal_in_workspaces_short_of_the_reported_size():
    """Any size from the one-step z sweeps' on is accepted (the calls then run
    those: the same bits); less is refused, and so is the reported size short
    of less than an alignment unit."""
    grid = Grid(40, 70, 10.0, 1e-3, 100, 8, 2300.0)
    ix = np.arange(0, 70, 14, dtype=np.int32)
    geom = Geometry(np.full(2, 3, np.int32), np.array([5, 60], np.int32), np.arange(3, dtype=np.int32) * len(ix),
                    np.full(2 * len(ix), 1, np.int32), np.tile(ix, 2), np.full(2, 100, np.int32))
    v = gaussian_anomaly(40, 70, 2000.0, 0.12, 9.0)
    wav = ricker(14.0, 1e-3, 100).astype(np.float32)
    full = B.fwi_offset_diag_exact_workspace_bytes(grid, geom, None, 3, 60.0)

    def call(n):
        return B.offset_diag_exact(v, wav, grid, geom, 3, 60.0, None, ws=torch.empty(n, dtype=torch.uint8, device="cuda"))
    with pytest.raises(B.FwiError) as e:
        call(16)
    least = int(re.search(r"need (\d+)", str(e.value)).group(1))
    assert least < full - 512
    ref = call(full)
    for n in (least, least + 1, least + 256, (least + full) // 2, full - 256, full + 100):
        assert torch.equal(call(n), ref), n
    for n in (least - 1, full - 255, full - 1):
        with pytest.raises(B.FwiError) as e:
            call(n)
        assert e.value.code == B.FWI_ERR_WORKSPACE


def test_calls_with_other_candidates_are_tuned_apart(tmp_path, monkeypatch):
    """Born modelling and Gauss-Newton products have no two-step forward sweep:
    they neither give modelling and gradients their settings nor take theirs."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("FWI_TUNE_CACHE", str(cache))
    nx, nz, nt = 120, 40, 41
    grid = Grid(nz, nx, 10.0, 1e-3, nt, 131, 2300.0)   # a sponge that the LDS-resident sweeps do not hold
    ix = np.arange(0, nx, 10, dtype=np.int32)
    geom = Geometry(np.full(2, 3, np.int32), np.array([5, 110], np.int32), np.arange(3, dtype=np.int32) * len(ix),
                    np.full(2 * len(ix), 1, np.int32), np.tile(ix, 2), np.full(2, nt, np.int32))
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, 9.0)
    dv = np.full((nz, nx), 10.0, np.float32)
    wav = ricker(20.0, 1e-3, nt).astype(np.float32)
    d = random_traces(geom, nt, seed=5, scale=1e-2)
    tuned = B.make_exec(autotune=1)
    calls = [lambda: B.born(v, wav, grid, geom, dv, tuned), lambda: B.gn_hvp(v, wav, grid, geom, dv, "int", tuned),
             lambda: B.forward(v, wav, grid, geom, tuned), lambda: B.gradient(v, wav, grid, geom, d, "int", tuned)]
    keys = []
    for call in calls:
        call()
        lines = cache.read_text().splitlines()
        assert len(lines) == len(keys) + 1
        key, choice = lines[-1].split(":")
        keys.append(key)
        if len(keys) <= 2:
            assert choice.split()[-1] == "1"    # forward steps
    assert len(set(keys)) == 4
    B.extended_image(v, wav, grid, geom, d, 2, "int", tuned)   # the gradient's candidates: its entry
    assert len(cache.read_text().splitlines()) == 4
