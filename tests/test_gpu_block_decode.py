"""Links decoded from a group's staged block records against the int32 table.

One step with the collision off moves every population along one link, so its bits
show each link's source; three more steps with collision and iolets show the next
steps' iolet populations too.  The lattices are chosen for the decode's edges: vessels
so thin that a group of four tiles has more own blocks than its LDS holds (those
groups use the global records), a ragged last tile, one lattice smaller than a tile,
iolet planes inside and across blocks.  Equality is exact.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from paper_1906_11925_amd import LB  # noqa: E402
from paper_1906_11925_amd import lib as L  # noqa: E402

pytestmark = pytest.mark.gpu

GEOMS = {
    "thin_tree": lambda: wl.tree(box=72, r0=4.0, root=(36.0, 36.0, 2.0), generations=5, seed=2),
    "wide_tree": lambda: wl.tree(box=96, r0=12.0, root=(48.0, 48.0, 6.0), generations=4, seed=3),
    "speck": lambda: wl.closed_box(X=3, Y=5, Z=2),
    "odd_pipe": lambda: wl.pipe(X=23, Y=21, Z=37, r2=97.0),
}


def _run(g, q, storage, addressing, stage, monkeypatch, d):
    monkeypatch.setenv("HEMELB_STAGE_TILES", str(stage))
    out = []
    for tau, steps in ((float("inf"), 1), (0.7, 3)):
        lb = LB.from_geometry(g, lattice=q, storage=storage, addressing=addressing, tau=tau)
        lb.set_deviations(torch.from_numpy(d), t=0)
        lb.step(steps)
        out += [lb.get_state()[0].cpu(), *(x.cpu() for x in lb.observables())]
        lb.close()
    return out


@pytest.mark.parametrize("name", sorted(GEOMS))
@pytest.mark.parametrize("q,storage", [(15, "f32"), (19, "f32"), (15, "f16"), (19, "bf16")])
def test_staged_decode_equals_the_table(name, q, storage, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = GEOMS[name]()
    d = wl.random_deviations(q, g.n_sites, 6, 1e-3).astype(np.float32)
    want = _run(g, q, storage, "table32", 0, monkeypatch, d)
    for stage in (0, 4, 8):
        got = _run(g, q, storage, "blocks", stage, monkeypatch, d)
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(want, got)), stage


def test_thin_tree_has_groups_beyond_the_staged_records():
    """The fallback is reached: some group of 256 sites spans more than 24 blocks."""
    g = GEOMS["thin_tree"]()
    c = g.coords.astype(np.int64)
    key = np.zeros(len(c), dtype=np.int64)
    for bit in range(6):
        for a, shift in ((2, 0), (1, 1), (0, 2)):
            key |= ((c[:, a] >> (2 + bit)) & 1) << (3 * bit + shift)
    key = np.sort(key)
    spans = [len(np.unique(key[s:s + 256])) for s in range(0, len(key), 256)]
    assert max(spans) > 24
