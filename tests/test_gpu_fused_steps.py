"""Several steps per launch give the bits of single steps.

Small lattices make up to four steps in one launch (HEMELB_FUSE chooses the form when a
handle is created; 0: single steps).  Each site is then computed from the same values by
the same arithmetic, so states, observables and times must be equal bit for bit, however
the steps are asked for.  Cases at the edges of the form: a lattice smaller than a tile, a
ragged last tile, vessels thinner than a group's surroundings, periodic cells (the sites
around a group wrap onto it), interpolated walls, Brinkman damping, iolets of both kinds
with a time series; step counts that leave every remainder; calls that need a step by
itself (a check interval, the objective's window), a cancelled request and a captured one.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from paper_1906_11925_amd import LB, HemelbError  # noqa: E402
from paper_1906_11925_amd import lib as L  # noqa: E402

pytestmark = pytest.mark.gpu

WAVE = (0.02, (0.0, 0.003), (0.01, 0.002), 40.0)
GEOMS = {
    "speck": lambda: wl.closed_box(X=3, Y=5, Z=2),
    "odd_pipe": lambda: wl.pipe(X=23, Y=21, Z=37, r2=97.0, inlet_velocity=WAVE),
    "pressure_pipe": lambda: wl.pipe(X=12, Y=13, Z=19, r2=30.0),
    "thin_tree": lambda: wl.tree(box=72, r0=4.0, root=(36.0, 36.0, 2.0), generations=5, seed=2),
    "couette": lambda: wl.couette(H=9, Lx=5, Lz=3),
    "channel": lambda: wl.channel(H=7, L=31, Lx=5),
}
FORMS = ["2,1,64,0", "2,3,512,1", "3,1,512,1", "4,1,1024,2"]


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _bits(*ts):
    return [t.cpu().contiguous().view(torch.uint8) for t in ts]


def _same(a, b):
    return len(a) == len(b) and all(torch.equal(x, y) for x, y in zip(a, b))


def _run(g, form, monkeypatch, q=15, storage="f32", bfl=False, alpha=None, counts=(1, 2, 3, 4, 7, 13)):
    monkeypatch.setenv("HEMELB_FUSE", form)
    lb = LB.from_geometry(g, lattice=q, storage=storage, bfl=bfl, alpha=alpha)
    d = wl.random_deviations(q, g.n_sites, 7, 1e-3).astype(np.float32)
    lb.set_deviations(torch.from_numpy(d), t=0)
    out = []
    for k in counts:
        lb.step(k)
        out += _bits(lb.get_state()[0], *lb.observables())
    assert lb.time == sum(counts)
    lb.close()
    return out


@pytest.mark.parametrize("name", sorted(GEOMS))
@pytest.mark.parametrize("q,storage", [(15, "f32"), (19, "f32"), (15, "f16"), (19, "bf16")])
def test_fused_steps_give_the_bits_of_single_steps(name, q, storage, monkeypatch):
    _gpu()
    g = GEOMS[name]()
    want = _run(g, "0", monkeypatch, q, storage)
    for form in FORMS:
        assert _same(_run(g, form, monkeypatch, q, storage), want), form
    monkeypatch.delenv("HEMELB_FUSE")
    lb = LB.from_geometry(g, lattice=q, storage=storage)  # the default form
    lb.close()


@pytest.mark.parametrize("q", [15, 19])
def test_fused_steps_with_interpolated_walls_and_damping(q, monkeypatch):
    _gpu()
    g = GEOMS["odd_pipe"]()
    alpha = np.random.default_rng(3).uniform(0.0, 0.3, g.n_sites).astype(np.float32)
    for kw in (dict(bfl=True), dict(alpha=alpha), dict(bfl=True, alpha=alpha)):
        want = _run(g, "0", monkeypatch, q, **kw)
        for form in ("2,2,512,1", "3,1,512,2"):
            assert _same(_run(g, form, monkeypatch, q, **kw), want), (form, list(kw))


def test_default_form_on_a_lattice_of_each_size_class(monkeypatch):
    _gpu()
    for radius, length in ((7.0, 40), (12.0, 60), (18.0, 110), (22.0, 120)):
        g = wl.pipe(X=2 * int(radius) + 5, Y=2 * int(radius) + 5, Z=length, r2=radius ** 2,
                    inlet_velocity=WAVE)
        for storage in ("f32", "f16"):
            want = _run(g, "0", monkeypatch, storage=storage, counts=(11, 4))
            monkeypatch.delenv("HEMELB_FUSE")
            lb = LB.from_geometry(g, storage=storage)
            d = wl.random_deviations(15, g.n_sites, 7, 1e-3).astype(np.float32)
            lb.set_deviations(torch.from_numpy(d), t=0)
            got = []
            for k in (11, 4):
                lb.step(k)
                got += _bits(lb.get_state()[0], *lb.observables())
            lb.close()
            assert _same(got, want), (g.n_sites, storage)


def test_calls_that_need_single_steps(monkeypatch):
    """A check interval, kernel timing and the objective's window fall inside a request."""
    _gpu()
    g = GEOMS["odd_pipe"]()
    got = {}
    for form in ("0", "3,1,512,1"):
        monkeypatch.setenv("HEMELB_FUSE", form)
        lb = LB.from_geometry(g)
        lb.set_objective(1, 0.1, np.ones(g.n_sites, dtype=np.uint8), 2.0, (5, 12))
        lb.set_check(4)
        lb.step(19)
        lb.sync()
        lb.set_check(0)
        lb.kernel_timing(3)
        lb.step(7)
        assert lb.kernel_time()[1] == 3
        lb.kernel_timing(0)
        lb.step(8)
        got[form] = (lb.objective_value(), lb.objective_flux().tolist(), lb.totals().tolist(),
                     _bits(lb.get_state()[0], *lb.observables()), lb.time)
        lb.close()
    a, b = got.values()
    assert a[:3] == b[:3] and a[4] == b[4] == 34 and _same(a[3], b[3])


def test_cancelled_request_leaves_a_usable_state(monkeypatch):
    _gpu()
    g = GEOMS["pressure_pipe"]()
    monkeypatch.setenv("HEMELB_FUSE", "3,1,512,1")
    lb = LB.from_geometry(g)
    lb.step(5)
    lb.cancel()  # seen by the next request before its first step
    with pytest.raises(HemelbError) as e:
        lb.step(10)
    assert e.value.code == L.ECANCELLED if hasattr(L, "ECANCELLED") else True
    lb.step(9)
    t, got = lb.time, _bits(lb.get_state()[0], *lb.observables())
    lb.close()
    monkeypatch.setenv("HEMELB_FUSE", "0")
    lb = LB.from_geometry(g)
    lb.step(t)
    assert t == 14 and _same(_bits(lb.get_state()[0], *lb.observables()), got)
    lb.close()


def test_captured_steps_replay(monkeypatch):
    """Captured steps stay single launches, whose buffers an even count restores."""
    _gpu()
    g = GEOMS["pressure_pipe"]()
    res = {}
    for form in ("0", "3,1,512,1"):
        monkeypatch.setenv("HEMELB_FUSE", form)
        stream = torch.cuda.Stream()
        lb = LB.from_geometry(g, stream=stream)
        lb.step(8)
        lb.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            lb.step(4)
        out = []
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            out += _bits(lb.get_state()[0])
            torch.cuda.synchronize()
        res[form] = out
        lb.close()
    monkeypatch.setenv("HEMELB_FUSE", "0")
    lb = LB.from_geometry(g)
    lb.step(8)
    want = []
    for _ in range(3):
        lb.step(4)
        want += _bits(lb.get_state()[0])
    lb.close()
    assert _same(res["0"], want) and _same(res["3,1,512,1"], want)


def test_captured_output_follows_eager_steps(monkeypatch):
    """Observables captured once are replayed between requests of an even step count."""
    _gpu()
    g = GEOMS["pressure_pipe"]()
    res = []
    for form in ("0", "3,1,512,1"):
        monkeypatch.setenv("HEMELB_FUSE", form)
        stream = torch.cuda.Stream()
        lb = LB.from_geometry(g, stream=stream)
        lb.step(7)
        out = [torch.empty(s, device="cuda") for s in ((g.n_sites,), (g.n_sites, 3), (g.n_sites,))]
        lb.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            lb.observables_into(*out)
        got = []
        for k in (10, 6, 14):
            lb.step(k)
            lb.sync()
            graph.replay()
            torch.cuda.synchronize()
            got += _bits(*out)
        res.append(got)
        lb.close()
    assert _same(*res)
