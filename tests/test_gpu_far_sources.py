"""Block addressing on a lattice whose populations pass 2^30 elements, against the table.

There a group of four tiles finds its sources by 32-bit references within a window around
it, and a group with sources beyond the window (the ghost slots at the end of the buffer,
neighbours across a large Morton boundary) by site numbers.  The int32 table knows neither,
so it is the reference: the same arithmetic on the same values, hence the same bits.  A
straight vessel of 75M sites with a pulsating Ladd inlet and a pressure outlet; steps with
collision, all outputs, and a reverse sweep with recomputed segments.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from paper_1906_11925_amd import LB, links  # noqa: E402
from paper_1906_11925_amd import lib as L  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vessel():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = wl.pipe(X=456, Y=456, Z=470, r2=226.0 ** 2, inlet_velocity=(0.02, (0.003,), (0.002,), 40.0))
    tables = {}

    def of(q):
        if q not in tables:
            tables.clear()  # one lattice's table at a time
            tables[q] = (*links(g.labels, g.shape, g.periodic, q), g.site_weight())
            print(f"vessel D3Q{q}: {len(tables[q][0])} sites", flush=True)
        return (g, *tables[q])

    return of


def _handle(vessel, q, storage, addressing, alpha=None):
    g, coords, nbr, weight = vessel(q)
    assert len(coords) * q > 2 ** 30
    lb = LB(nbr, g.tau, lattice=q, storage=storage, coords=coords, iolets=list(g.iolets),
            site_weight=weight, addressing=addressing, alpha=alpha)
    assert lb.info()["addressing"] == {"blocks": L.ADDR_BLOCKS, "table32": L.ADDR_TABLE32}[addressing]
    print(f"D3Q{q} {storage} {addressing}", flush=True)
    return lb


def _start(n, q):
    gen = torch.Generator(device="cuda").manual_seed(29)
    return torch.rand((q, n), generator=gen, device="cuda").sub_(0.5).mul_(2e-3)


def _steps(vessel, q, storage, addressing):
    lb = _handle(vessel, q, storage, addressing)
    lb.set_deviations(_start(lb.n, q), t=7)
    lb.step(3)
    out = [lb.get_state()[0], *lb.observables()]
    lb.close()
    return [x.view(torch.int16) if x.dtype == torch.bfloat16 else x for x in out]


@pytest.mark.parametrize("q,storage,forms", [(15, "f32", ("8", "4", "0")), (15, "f16", ("4",)),
                                             (19, "f32", ("4", "16"))])
def test_steps_and_outputs_equal_the_table(vessel, q, storage, forms, monkeypatch):
    want = _steps(vessel, q, storage, "table32")
    for form in forms:
        monkeypatch.setenv("HEMELB_STAGE_TILES", form)
        got = _steps(vessel, q, storage, "blocks")
        for name, a, b in zip(("state", "p", "u", "wss"), want, got):
            assert torch.equal(a, b), (form, name)
        del got


@pytest.mark.parametrize("q,storage", [(15, "f32"), (15, "f16")])
def test_reverse_sweep_equals_the_table(vessel, q, storage):
    """Two segments of two steps: paired launches (the recompute half staged in FP32),
    single reverse steps and the segments' ends."""
    res = []
    for addressing in ("table32", "blocks"):
        n = len(vessel(q)[1])
        alpha = np.full(n, 0.004, dtype=np.float32)
        lb = _handle(vessel, q, storage, addressing, alpha)
        lb.set_objective(1, 0.5, (np.arange(n) % 97 == 0).astype(np.uint8), 1e4, (0, 4))
        lb.set_deviations(_start(n, q), t=0)
        checkpoints = []
        for t0 in (0, 2):
            checkpoints.append((t0, 2, lb.get_state()[0]))
            lb.step(2)
        lb.adjoint_begin(2)
        lb.adjoint_run(checkpoints)
        dtheta, dalpha = lb.adjoint_grads()
        res.append((lb.get_adjoint(), dtheta[0], dalpha, lb.objective_value()))
        lb.close()
        del lb, checkpoints
    (ga, ta, aa, ja), (gb, tb, ab, jb) = res
    assert torch.equal(ga, gb)
    assert np.array_equal(aa, ab) and np.array_equal(ta, tb) and ja == jb
    assert np.abs(ta).max() > 0 and np.abs(aa).max() > 0
