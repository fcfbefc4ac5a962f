"""Frames of sites in clusters with empty blocks between them: gaps around one block, the
largest distance that the renderer's maps hold (16 blocks) and beyond, crossed in either
direction, along an axis and at a slant, against the oracle's marcher.

Tolerance as for every frame: FP32 compositing rounds three times a sample, 4 K 2^-24 after
K samples; pixels whose ray meets no site are zero on both sides."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from oracle.render import render as oracle_render  # noqa: E402
from paper_1906_11925_amd import LB  # noqa: E402
from workloads.camera import orbit_view, ramp_lut  # noqa: E402

pytestmark = pytest.mark.gpu


def _clusters(gaps, axis):
    """Random voxels in 8-wide cells on the axis, `gaps` empty blocks apart."""
    rng = np.random.default_rng(3)
    starts, at = [], 0
    for gap in list(gaps) + [0]:
        starts.append(at)
        at += 8 + 4 * gap
    shape = [12, 12, 12]
    shape[axis] = at
    lab = np.zeros([n + 2 for n in shape], dtype=np.uint8)
    for s in starts:
        lo = [2, 2, 2]
        lo[axis] = s
        cell = rng.random((8, 8, 8)) < 0.4
        lab[tuple(slice(1 + lo[a], 9 + lo[a]) for a in range(3))] = cell
    return wl.Geometry("clusters", tuple(shape), lab)


@pytest.mark.parametrize("filt", ["nearest", "trilinear"])
@pytest.mark.parametrize("gaps,axis", [((1, 2, 15), 2), ((16, 17), 0), ((14, 1, 33), 1)])
def test_frames_across_gaps(gaps, axis, filt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = _clusters(gaps, axis)
    vals = np.random.default_rng(7).uniform(0.0, 1.0, g.n_sites).astype(np.float32)
    lb = LB.from_geometry(g)
    c = g.coords
    mid = (c.min(axis=0) + c.max(axis=0)) / 2.0
    size = float(np.linalg.norm(c.max(axis=0) - c.min(axis=0)))
    lut = ramp_lut()
    for angles in ((0, 0), (180, 0), (90, 0), (270, 0), (0, 90), (0, -90), (37, 21), (215, -8)):
        for pixel in (0.5, size / 24.0):
            v = orbit_view(mid, size, angles[0], angles[1], 25, 23, pixel=pixel, step=0.7)
            v["filter"] = filt
            img = lb.render(torch.from_numpy(vals).cuda(), v, lut, scale=1.0, offset=0.0)
            ref = oracle_render(c, vals, v, lut, scale=1.0, offset=0.0)
            img = img.cpu().numpy().astype(np.float64)
            assert np.array_equal(img[..., 3] == 0, ref[..., 3] == 0), (angles, pixel)
            assert np.abs(img - ref).max() <= 4.0 * max(1, v["steps"]) * 2.0 ** -24, (angles, pixel)
