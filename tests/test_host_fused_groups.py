"""Planning of the groups that make several steps per launch, on the CPU.

Whether a plan holds them shows in its device bytes: without them (HEMELB_FUSE=0) a plan
has neither the third population buffer nor the groups' data.
"""

import numpy as np
import pytest

import workloads as wl
from paper_1906_11925_amd import links, plan
from paper_1906_11925_amd.lb import lattice_vectors


def _opp(i):
    return i + 1 if i % 2 else i - 1


def _star(q, children, grandchildren, n):
    """Reciprocal table of n sites in which one tile's 64 sites reach `children` others
    each, and each of these `grandchildren` of its own; all other links are walls."""
    nbr = np.full((n, q), -1, dtype=np.int32)
    free = n - 1  # far from the first tile, so that no group holds both
    for s in range(64):
        for i in range(1, children + 1):
            c, free = free, free - 1
            nbr[s, i], nbr[c, _opp(i)] = c, s
            left = grandchildren
            for k in range(1, q):
                if left and k != _opp(i):
                    g, free, left = free, free - 1, left - 1
                    nbr[c, k], nbr[g, _opp(k)] = g, c
    assert free >= 1024
    return nbr


def _bytes(monkeypatch, nbr, form, **kw):
    if form is None:
        monkeypatch.delenv("HEMELB_FUSE", raising=False)
    else:
        monkeypatch.setenv("HEMELB_FUSE", form)
    return plan(nbr, 0.8, **kw)["device_bytes"]


# 64 + 64 * 13 = 896 sites fill a D3Q19 row of class 2; what reaches them counts to 896 +
# 896 + 14592 of 2^14 four-byte places with 16 links each at most (832 * 16 + 896 = 14208)
@pytest.mark.parametrize("grandchildren,fits", [(16, True), (17, False)])
def test_codes_of_a_row_stay_within_16_bits(monkeypatch, grandchildren, fits):
    nbr = _star(19, 13, grandchildren, 140096)
    single = _bytes(monkeypatch, nbr, "0", lattice=19)
    assert (_bytes(monkeypatch, nbr, "2,8,1024,2", lattice=19) > single) == fits


def _pipe(radius, length):
    w = 2 * int(np.ceil(radius)) + 3
    return wl.pipe(X=w, Y=w, Z=length, r2=radius ** 2)


GEOMS = {
    "pipe13k": wl.pipe,
    "pipe75k": lambda: _pipe(16.0, 94),
    "pipe140k": lambda: _pipe(19.0, 123),
    "aneurysm_half": lambda: wl.aneurysm(half=True),
    "tree230k": lambda: wl.tree(170, 21.5, (85.0, 85.0, 10.75), 6, seed=5),
    "pipe255k": lambda: _pipe(23.0, 154),
}


# measured on the GPU: where several steps per launch are faster than single ones
@pytest.mark.parametrize("name,q,storage,bfl,several", [
    ("pipe13k", 15, "f32", False, True),
    ("pipe13k", 19, "bf16", True, True),
    ("pipe75k", 19, "f32", False, True),
    ("pipe75k", 15, "f32", True, True),
    ("pipe75k", 19, "f32", True, False),
    ("aneurysm_half", 15, "f32", False, True),
    ("aneurysm_half", 15, "f16", False, True),
    ("aneurysm_half", 19, "f32", False, False),
    ("aneurysm_half", 19, "f16", False, True),
    ("tree230k", 15, "f32", False, False),
    ("pipe140k", 15, "f32", False, False),
    ("pipe140k", 15, "f16", False, True),
    ("pipe140k", 19, "f16", False, False),
    ("tree230k", 15, "f16", False, False),
    ("tree230k", 19, "f16", False, False),
    ("pipe255k", 15, "f32", False, False),
    ("pipe255k", 15, "bf16", False, False),
    ("pipe255k", 19, "f32", False, False),
])
def test_default_choice(monkeypatch, name, q, storage, bfl, several):
    g = GEOMS[name]()
    coords, nbr = links(g.labels, g.shape, g.periodic, q)
    kw = dict(lattice=q, storage=storage, coords=coords, iolets=list(g.iolets),
              wall_q=g.wall_fractions(lattice_vectors(q)) if bfl else None)
    assert (_bytes(monkeypatch, nbr, None, **kw) > _bytes(monkeypatch, nbr, "0", **kw)) == several


@pytest.mark.parametrize("form", ["2,8,1024,0", "2,3,512,1", "3,4,128,1", "4,6,512,2"])
@pytest.mark.parametrize("q", [15, 19])
def test_groups_hold_as_many_tiles_as_fit(monkeypatch, q, form):
    """The plan's bytes are those of groups grown here by definition: whole tiles, as many as
    leave the inner sites within a row and a site a thread (fewer than 2048 sites, which one
    task plans, in the caller's order)."""
    steps, tiles, threads, row = (int(x) for x in form.split(","))
    g = wl.pipe(X=13, Y=12, Z=19, r2=29.0)
    _, nbr = links(g.labels, g.shape, g.periodic, q)
    n = len(nbr)
    assert 1024 < n < 2048
    pitch = (2048, 3072, 4096 if q == 15 else 3584)[row] // 4

    def grow(a, b):
        inside, counts = set(range(64 * a, min(n, 64 * b))), []
        for _ in range(steps):
            counts.append(len(inside))
            inside |= {int(v) for s in inside for v in nbr[s, 1:] if v >= 0}
        return counts + [len(inside)]

    words, t, fits = 0, 0, True
    while 64 * t < n and fits:
        for take in range(min(tiles, (n + 63) // 64 - t), 0, -1):
            c = grow(t, t + take)
            fits = c[steps - 1] <= pitch and (steps == 2 or c[steps - 2] <= threads)
            if fits:
                break
        words += 16 + c[steps] + c[steps - 1] * (8 if q == 15 else 12)
        t += take
    kw = dict(lattice=q, iolets=list(g.iolets))
    single = _bytes(monkeypatch, nbr, "0", **kw)
    monkeypatch.setenv("HEMELB_FUSE", form)
    info = plan(nbr, 0.8, **kw)
    assert info["device_bytes"] - single == (q * info["pitch"] * 4 + 4 * words if fits else 0)
