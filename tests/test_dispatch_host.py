"""Host checks of the rules that choose a call's sweeps (no GPU needed)."""
import numpy as np
import pytest

from paper_1406_1864_amd import binding as B
from paper_1406_1864_amd.synthetic import Geometry, Grid


def problem(nx, nz, N, ns, nrec, nt=64, fs=False):
    grid = Grid(nz, nx, 10.0, 1e-3, nt, N, 2300.0, fs)
    iz, ix = np.divmod(np.arange(nrec, dtype=np.int32), nx)
    geom = Geometry(np.zeros(ns, np.int32), (np.arange(ns, dtype=np.int32) * 7) % nx,
                    np.arange(ns + 1, dtype=np.int32) * nrec, np.tile(iz, ns), np.tile(ix, ns), np.full(ns, nt, np.int32))
    return grid, geom


@pytest.mark.parametrize("N,nrec", [(20, 1025), (129, 30)])
def test_tuned_calls_keep_two_steps_past_the_lds_tables(N, nrec):
    """A shot with more receivers, or a sponge wider, than the LDS-resident
    sweeps hold: a tuned call keeps the two-step sweeps' levels, as an untuned
    one does, however few its cells."""
    grid, geom = problem(300, 150, N, 2, nrec)
    for what in (B.WS_FORWARD, B.WS_HESSIAN, B.WS_GRADIENT, B.WS_AUTOGRAD):
        tuned = B.fwi_workspace_bytes(grid, geom, B.make_exec(autotune=1), what)
        untuned = B.fwi_workspace_bytes(grid, geom, None, what)
        assert tuned >= untuned, what
