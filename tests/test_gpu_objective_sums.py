"""Objective sums at the sizes where the one-launch reduction can go wrong: no dome
sites, one, a few blocks, and more items than the largest grid has threads; step after
step, so that a counter left over from one launch would spoil the next.

Against the FP64 oracle at the repository's tolerance for the objective (1e-5)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from oracle.adjoint import Adjoint, Objective  # noqa: E402
from oracle.lbgk import LBGK  # noqa: E402
from paper_1906_11925_amd import LB  # noqa: E402

pytestmark = pytest.mark.gpu

T, W = 5, (1, 5)


@pytest.mark.parametrize("lattice", [15, 19])
@pytest.mark.parametrize("Z,dome_sites", [(12, 0), (12, 1), (64, 1000), (1200, None)])
def test_objective_sums(Z, dome_sites, lattice):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if dome_sites is None and lattice == 19:
        pytest.skip("the size is covered once")
    g = wl.pipe(Z=Z)
    o = LBGK(g, lattice)
    _, has = o.wall_normals()
    at = np.flatnonzero(has)[:dome_sites]
    if dome_sites is None:
        assert len(at) > 256 * 256  # the grid-stride loop takes a second pass
    dome = np.zeros(g.n_sites, dtype=bool)
    dome[at] = True
    d0 = wl.random_deviations(lattice, g.n_sites, 5, 1e-3).astype(np.float32).astype(np.float64)
    obj = Objective(1, 0.05, dome, 2.0, W)
    J, _, q = Adjoint(o, obj).forward(o.rest_state() + d0, T)
    lb = LB.from_geometry(g, lattice=lattice)
    lb.set_objective(obj.outlet, obj.q_target, obj.dome, obj.lam, obj.window)
    lb.set_deviations(torch.from_numpy(d0), t=0)
    lb.step(T)
    got, flux, wss = lb.objective_value()
    q = np.asarray(q)
    print(f"Z={Z} dome={len(at)}: J {got:.6e} against {J:.6e}", flush=True)
    assert abs(got - J) <= 1e-5 * abs(J)
    assert np.abs(lb.objective_flux() - q).max() <= 1e-5 * np.abs(q).max()
    assert (wss == 0.0) == (len(at) == 0)
