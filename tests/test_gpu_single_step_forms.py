"""The forms of the single step give the same bits, with several steps per launch off.

Small lattices make several steps per launch by default, in a kernel that knows
neither the addressing nor the staging of the single step.  Here HEMELB_FUSE=0 turns that
off, so that every step is one launch of the form under test: the staged copies of 4, 8 and
16 tiles, by loads that write LDS directly and through registers, in every storage; the
three addressings; and the decode of links for thin vessels, ragged tiles and iolets.  30
steps (3 for the decode) from a seeded random state; states and outputs equal bit for bit.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from paper_1906_11925_amd import LB  # noqa: E402
from paper_1906_11925_amd import lib as L  # noqa: E402

pytestmark = pytest.mark.gpu

WAVE = (0.02, (0.0, 0.003), (0.01, 0.002), 40.0)
GEOMS = {
    "aneurysm_half": lambda: wl.aneurysm(half=True),
    "tree_small": lambda: wl.tree(box=96, r0=6.0, root=(48.0, 48.0, 4.0), generations=3, seed=1),
    "odd_pipe": lambda: wl.pipe(X=23, Y=21, Z=37, r2=97.0, inlet_velocity=WAVE),
    "thin_tree": lambda: wl.tree(box=72, r0=4.0, root=(36.0, 36.0, 2.0), generations=5, seed=2),
}
# (HEMELB_STAGE_TILES, HEMELB_LDS_DMA); the first is the unstaged reference
FORMS = [(0, 1), (4, 1), (8, 1), (16, 1), (4, 0), (8, 0), (16, 0)]


def _run(monkeypatch, g, q, storage, steps, addressing="auto", form=None):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("HEMELB_FUSE", "0")
    if form is not None:
        monkeypatch.setenv("HEMELB_STAGE_TILES", str(form[0]))
        monkeypatch.setenv("HEMELB_LDS_DMA", str(form[1]))
    lb = LB.from_geometry(g, lattice=q, storage=storage, addressing=addressing)
    info = lb.info()
    lb.set_deviations(torch.from_numpy(wl.random_deviations(q, g.n_sites, 23, 1e-3).astype(np.float32)), t=5)
    lb.step(steps)
    out = [lb.get_state()[0], *lb.observables()]
    out = [x.cpu().contiguous().view(torch.uint8) for x in out]
    lb.close()
    return info, out


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b, strict=True))


@pytest.mark.parametrize("name", ["aneurysm_half", "tree_small"])
@pytest.mark.parametrize("q,storage", [(15, "f32"), (19, "f32"), (15, "f16"), (19, "bf16")])
def test_staged_forms(monkeypatch, name, q, storage):
    g = GEOMS[name]()
    info, want = _run(monkeypatch, g, q, storage, 30, form=FORMS[0])
    assert info["addressing"] == L.ADDR_BLOCKS
    for form in FORMS[1:]:
        assert _same(want, _run(monkeypatch, g, q, storage, 30, form=form)[1]), form


@pytest.mark.parametrize("name", ["aneurysm_half", "odd_pipe"])
@pytest.mark.parametrize("q,storage", [(15, "f32"), (19, "f32"), (15, "f16"), (19, "f16")])
def test_addressings(monkeypatch, name, q, storage):
    g = GEOMS[name]()
    runs = {a: _run(monkeypatch, g, q, storage, 30, addressing=a) for a in ("table32", "table16", "blocks")}
    want = {"table32": L.ADDR_TABLE32, "table16": L.ADDR_TABLE16, "blocks": L.ADDR_BLOCKS}
    for a, (info, out) in runs.items():
        assert info["addressing"] == want[a]
        assert _same(runs["table32"][1], out), a


@pytest.mark.parametrize("name", ["odd_pipe", "thin_tree"])
@pytest.mark.parametrize("q,storage", [(15, "f32"), (19, "bf16")])
def test_decode_over_several_steps(monkeypatch, name, q, storage):
    g = GEOMS[name]()
    want = _run(monkeypatch, g, q, storage, 3, addressing="table32", form=(0, 1))[1]
    for tiles in (0, 4, 8, 16):
        got = _run(monkeypatch, g, q, storage, 3, addressing="blocks", form=(tiles, 1))[1]
        assert _same(want, got), tiles
