"""The LDS-resident sweeps (several time steps per launch) against the one-step
z sweeps and the FP64 oracle, at the sizes where their tiling can go wrong: a
grid of one tile, one column more than a tile, tiles in both directions, model
widths that are no multiple of 4, records whose steps are no multiple of a
launch's, snapshots and receivers on the tiles' margins, a free surface.

Both forms make the same operations in the same order per cell, so every
result that does not depend on a tiling has the same bits.
"""
import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid, gaussian_anomaly, random_traces, ricker

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# rows per tile is a setting of the z sweeps only: naming it selects them
Z_SWEEP = dict(tile_rows=16, graph_steps=-1)


def problem(nx, nz, N, nts, fs=False):
    ns, nt = len(nts), max(nts)
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0, fs)
    v = gaussian_anomaly(nz, nx, 2000.0, 0.12, max(3.0, nx / 12), iz0=nz // 2, ix0=nx // 3)
    rec = [(z, x) for z in (1, nz - 1) for x in range(0, nx, 3)] + [(z, nx - 1) for z in range(2, nz - 1, 2)]
    iz = np.array([r[0] for r in rec] * ns, np.int32)
    ix = np.array([r[1] for r in rec] * ns, np.int32)
    six = np.linspace(0, nx - 1, ns).astype(np.int32)
    siz = np.array([(2 + 5 * s) % nz for s in range(ns)], np.int32)
    geom = Geometry(siz, six, np.arange(ns + 1, dtype=np.int32) * len(rec), iz, ix, np.array(nts, np.int32))
    wav = np.stack([ricker(14.0 + s, 1e-3, nt) for s in range(ns)]).astype(np.float32)
    return grid, geom, v, wav


CASES = [
    (24, 16, 8, (150, 61), False),       # 40 x 32: one 64 x 32 region, the whole record in one launch
    (25, 17, 8, (300, 2, 3), False),     # 41 x 33: one 64 x 64 region, two launches, records of one and two steps
    (49, 40, 7, (127, 90), False),       # 63 columns from an unaligned first one
    (53, 50, 7, (100,), False),          # 67 columns, 64 rows: two tiles along x
    (30, 60, 9, (96, 50), False),        # 78 rows: tiles along z only
    (130, 90, 11, (83, 110, 40), False), # tiles both ways, width no multiple of 4
    (131, 70, 12, (121,), True),         # free surface
    (300, 150, 20, (57,) * 9, False),    # several tiles per CU
]


def calls(grid, geom, v, wav, ex):
    d = random_traces(geom, grid.nt_max, seed=3, scale=1e-2)
    dv = np.random.default_rng(4).standard_normal((grid.nz, grid.nx)).astype(np.float32) * 30.0
    out = {"forward": (B.forward(v, wav, grid, geom, ex),),
           "gradient": B.gradient(v, wav, grid, geom, d, "int", ex, hmax=2),
           "l2": B.gradient(v, wav, grid, geom, d, "l2", ex),
           "misfit": (B.misfit_value(v, wav, grid, geom, d, "int", ex),),
           "hessian": (B.hessian_diag(v, wav, grid, geom, B.HESS_EQ1, exec_=ex),),
           "born": (B.born(v, wav, grid, geom, dv, ex),),
           "gn": B.gn_hvp(v, wav, grid, geom, dv, "int", ex),
           "image": B.extended_image(v, wav, grid, geom, d, 3, "int", ex),
           "eq3": B.gradient(v, wav, grid, geom, d, "eq3", ex)}
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("nx,nz,N,nts,fs", CASES)
def test_same_bits_as_the_z_sweeps(nx, nz, N, nts, fs):
    grid, geom, v, wav = problem(nx, nz, N, nts, fs)
    a = calls(grid, geom, v, wav, None)
    b = calls(grid, geom, v, wav, B.make_exec(**Z_SWEEP))
    for name in a:
        for k, (x, y) in enumerate(zip(a[name], b[name])):
            assert (x is None) == (y is None)
            if x is not None:
                assert bool(torch.isfinite(x).all()), (name, k)
                assert torch.equal(x, y), (name, k)
    assert float(a["gradient"][1].abs().max()) > 0 and float(a["born"][0].abs().max()) > 0


def test_exact_diagonal_same_bits():
    """Captured series in chunks of 64 updates, tiles both ways."""
    grid, geom, v, wav = problem(70, 40, 8, (150, 150))
    for sif in (3, 64):
        a = B.offset_diag_exact(v, wav, grid, geom, 3, 60.0, B.make_exec(shots_in_flight=sif))
        b = B.offset_diag_exact(v, wav, grid, geom, 3, 60.0, B.make_exec(shots_in_flight=sif, tile_rows=16))
        assert torch.equal(a, b)


def test_workspace_of_the_z_sweeps_size_is_enough():
    """A workspace of the size the z sweeps need holds every call that it held
    before (the call then runs those), and gives the same bits."""
    grid, geom, v, wav = problem(130, 90, 11, (83, 110, 40))
    d = random_traces(geom, grid.nt_max, seed=3, scale=1e-2)
    n = B.fwi_workspace_bytes(grid, geom, B.make_exec(tile_rows=64), B.WS_GRADIENT)
    full = B.fwi_workspace_bytes(grid, geom, None, B.WS_GRADIENT)
    assert n < full
    small = B.gradient(v, wav, grid, geom, d, "int", None, ws=torch.empty(n, dtype=torch.uint8, device="cuda"))
    ref = B.gradient(v, wav, grid, geom, d, "int", None)
    for x, y in zip(small, ref):
        assert (x is None and y is None) or torch.equal(x, y)
