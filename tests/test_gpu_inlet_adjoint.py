"""Inlet-coefficient adjoints where their sums can go wrong: segments of fewer, as many
and more steps than one launch of the summing kernel covers (64), sites whose links
belong to several iolets of different kinds and harmonic counts, either addressing.

Against the FP64 oracle's adjoint at the repository's adjoint tolerance (max |error| <=
1e-4 of the largest entry: FP32 adjoint populations, FP64 sums); runs that differ only in
how steps are grouped give the same bits."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from oracle.adjoint import Adjoint, Objective  # noqa: E402
from oracle.lbgk import LBGK  # noqa: E402
from paper_1906_11925_amd import LB  # noqa: E402

pytestmark = pytest.mark.gpu


def _vessel():
    """Short pipe whose inlet plane holds two velocity iolets and a pressure iolet, and
    whose outlet plane holds two pressure iolets."""
    g = wl.pipe(X=8, Y=8, Z=12, r2=9.0, tau=0.7,
                inlet_velocity=(0.02, (0.0, 0.003), (0.01, 0.002), 40.0))
    lab, cls = g.labels, type(g.iolets[0])
    for plane, old, parts in ((0, 2, (4, 5)), (-1, 3, (6,))):
        p = lab[:, :, plane]
        xs = np.arange(p.shape[0])[:, None] + 0 * np.arange(p.shape[1])[None, :]
        ys = xs.T if p.shape[0] == p.shape[1] else np.broadcast_to(np.arange(p.shape[1]), p.shape)
        p[(p == old) & (xs >= 5)] = parts[0]
        if len(parts) > 1:
            p[(p == parts[0]) & (ys >= 5)] = parts[1]
    g.iolets += [cls("velocity", direction=(0.0, 0.0, 1.0), mean=0.015, cos=(0.004,), sin=(0.001,),
                     period=30.0),
                 cls("pressure", mean=1.002), cls("pressure", mean=0.999)]
    return g


@pytest.fixture(scope="module")
def problems():
    g = _vessel()
    n = g.n_sites
    alpha = np.random.default_rng(4).uniform(0.0, 0.01, n).astype(np.float32)
    o = LBGK(g, 15, alpha=alpha.astype(np.float64))
    _, has = o.wall_normals()
    dome = has & (g.coords[:, 2] >= 4) & (g.coords[:, 2] <= 7)
    made = {}

    def make(T):
        if T not in made:
            obj = Objective(1, 0.05, dome, 1.0, (T - 15, T))
            adj = Adjoint(o, obj)
            _, tape, _ = adj.forward(o.rest_state(), T)
            made[T] = (obj, *adj.backward(tape, T))
        return (g, alpha) + made[T]

    return make


def _run(g, alpha, obj, T, K, how, addressing="auto"):
    lb = LB.from_geometry(g, alpha=alpha, addressing=addressing)
    lb.set_objective(obj.outlet, obj.q_target, obj.dome, obj.lam, obj.window)
    if how == "recorded":
        lb.record(T)
        lb.step(T)
        lb.adjoint_begin(1)
        lb.adjoint_recorded()
    else:
        cks = []
        for t0 in range(0, T, K):
            cks.append((t0, min(K, T - t0), lb.get_state()[0].clone()))
            lb.step(min(K, T - t0))
        lb.adjoint_begin(K)
        if how == "run":
            lb.adjoint_run(cks)
        else:
            for t0, k, ck in reversed(cks):
                lb.adjoint_segment(ck, t0, k)
    return lb.adjoint_grads()


@pytest.mark.parametrize("T", [63, 64, 65, 140])
def test_inlet_sums_match_the_oracle(problems, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g, alpha, obj, theta, ahat, _ = problems(T)
    runs = [_run(g, alpha, obj, T, T, "segment"), _run(g, alpha, obj, T, 9, "run"),
            _run(g, alpha, obj, T, 66, "run"), _run(g, alpha, obj, T, T, "recorded")]
    runs = [([t[k] for k in sorted(t)], d) for t, d in runs]
    th, da = runs[0]
    ref = [theta[k] for k in sorted(theta)]
    assert len(th) == len(ref) == 2 and [len(x) for x in th] == [5, 3]
    for a, b in zip(th, ref):
        err = np.abs(np.asarray(a) - b).max() / np.abs(b).max()
        print(f"T={T}: e_theta={err:.2e}", flush=True)
        assert err <= 1e-4
    assert np.abs(da - ahat).max() <= 1e-4 * np.abs(ahat).max()
    for other_th, other_da in runs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(th, other_th))
        assert np.array_equal(da, other_da)
    for addressing in ("table16", "table32"):
        t2, d2 = _run(g, alpha, obj, T, 40, "run", addressing)
        for a, b in zip([t2[k] for k in sorted(t2)], ref):
            assert np.abs(np.asarray(a) - b).max() <= 1e-4 * np.abs(b).max()
        assert np.abs(d2 - ahat).max() <= 1e-4 * np.abs(ahat).max()
