"""Sites with links past several iolets, in every direction.

A step loads what a site's iolet links name a few links at a time, and the first link's
iolet only once; the links are decoded from ghost records in LDS.  The lattices make the
edges of that: a sheet one site thick between a Ladd inlet and a pressure outlet (each site
has links of both), a porous box whose empty points are wall or one of three iolets at
random (every set of directions and iolets, several ghost blocks a group), one site with
iolets all around.  Two steps against the FP64 oracle, the second on what the first wrote;
and five steps bit for bit against the tables and against several steps per launch.

The bound for two steps: one step errs by at most e = 2 q^2 a 2^-24 (a = 1e-3 the deviations'
size).  In the second, a pressure iolet's value carries at most 3.5 e (u errs by at most 10
e, and 3 w_i |c_i| 10 e <= 3.5 e), and collision at tau = 0.7 multiplies by at most
|1 - 1/tau| + (1/tau) w_i sum_j (1 + 3 |c_i . c_j|) < 8.6; 3.5 * 8.6 + 1 < 32.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from oracle.lbgk import LBGK  # noqa: E402
from paper_1906_11925_amd import LB  # noqa: E402
from workloads.geometry import Geometry, Iolet  # noqa: E402

from lbtest import quantize  # noqa: E402

pytestmark = pytest.mark.gpu

IOLETS = [Iolet("velocity", direction=(0.0, 0.6, 0.8), mean=0.02, cos=(0.003,), sin=(0.002,), period=40.0),
          Iolet("pressure", mean=1.002), Iolet("pressure", mean=0.999)]


def _sheet():
    lab = np.zeros((13, 12, 3), dtype=np.uint8)
    lab[1:-1, 1:-1, 1] = 1
    lab[:, :, 0], lab[:, :, 2] = 2, 3
    return Geometry("sheet", (11, 10, 1), lab, iolets=IOLETS[:2], tau=0.7)


def _porous():
    rng = np.random.default_rng(12)
    shape = (14, 13, 11)
    lab = rng.choice([0, 2, 3, 4], size=tuple(s + 2 for s in shape), p=[0.4, 0.2, 0.2, 0.2]).astype(np.uint8)
    inner = lab[1:-1, 1:-1, 1:-1]
    inner[rng.random(shape) < 0.55] = 1
    return Geometry("porous", shape, lab, iolets=IOLETS, tau=0.7)


def _alone():
    lab = np.full((3, 3, 3), 4, dtype=np.uint8)
    lab[1, 1, 1], lab[0], lab[2] = 1, 2, 3
    return Geometry("alone", (1, 1, 1), lab, iolets=IOLETS, tau=0.7)


GEOMS = {"sheet": _sheet, "porous": _porous, "alone": _alone}


def _start(g, q, storage):
    return quantize(wl.random_deviations(q, g.n_sites, 31, 1e-3), q, storage)


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("name", sorted(GEOMS))
@pytest.mark.parametrize("q", [15, 19])
@pytest.mark.parametrize("addressing", ["blocks", "table32"])
def test_two_steps_against_the_oracle(monkeypatch, name, q, addressing):
    _gpu()
    monkeypatch.setenv("HEMELB_FUSE", "0")
    g = GEOMS[name]()
    o = LBGK(g, q)
    d = _start(g, q, "f32")
    lb = LB.from_geometry(g, lattice=q, addressing=addressing)
    lb.set_deviations(torch.from_numpy(d), t=9)
    A = o.lat.w[:, None] + d
    for t in (9, 10):
        lb.step(1)
        A, _ = o.step(A, t)
    gpu = lb.get_deviations().cpu().numpy().astype(np.float64)
    lb.close()
    assert np.abs(gpu - (A - o.lat.w[:, None])).max() < 32 * 2.0 * q * q * 1e-3 * 2.0 ** -24


@pytest.mark.parametrize("name", sorted(GEOMS))
@pytest.mark.parametrize("q,storage", [(15, "f32"), (19, "f32"), (15, "f16"), (19, "bf16")])
def test_forms_give_the_same_bits(monkeypatch, name, q, storage):
    _gpu()
    g = GEOMS[name]()
    d = torch.from_numpy(_start(g, q, storage))
    want = None
    for fuse, tiles, addressing in (("0", 0, "table32"), ("0", 0, "table16"), ("0", 0, "blocks"),
                                    ("0", 4, "blocks"), ("0", 8, "blocks"), ("2,1,512,0", 0, "blocks")):
        monkeypatch.setenv("HEMELB_FUSE", fuse)
        monkeypatch.setenv("HEMELB_STAGE_TILES", str(tiles))
        lb = LB.from_geometry(g, lattice=q, storage=storage, addressing=addressing)
        lb.set_deviations(d, t=9)
        lb.step(5)
        got = [x.cpu().contiguous().view(torch.uint8) for x in (lb.get_state()[0], *lb.observables())]
        lb.close()
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(want, got)), (fuse, tiles, addressing)
