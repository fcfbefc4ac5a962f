"""A request cancelled from another thread leaves a state and outputs that single steps give."""

import threading

import pytest

torch = pytest.importorskip("torch")

import workloads as wl  # noqa: E402
from paper_1906_11925_amd import LB, HemelbError  # noqa: E402
from paper_1906_11925_amd import lib as L  # noqa: E402

pytestmark = pytest.mark.gpu


def _bits(lb):
    return [x.cpu().contiguous().view(torch.uint8) for x in (lb.get_state()[0], *lb.observables())]


@pytest.mark.parametrize("form", ["2,2,512,0", "3,1,512,1"])
def test_cancelled_in_the_middle_of_a_request(form, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = wl.pipe(X=23, Y=21, Z=37, r2=97.0, inlet_velocity=(0.02, (0.0, 0.003), (0.01, 0.002), 40.0))
    monkeypatch.setenv("HEMELB_FUSE", form)
    lb = LB.from_geometry(g)
    timer = threading.Timer(0.02, lb.cancel)
    timer.start()
    with pytest.raises(HemelbError) as e:
        lb.step(100000)  # some 0.4 s
    timer.join()
    assert e.value.code == L.HEMELB_ECANCELLED
    t = lb.time
    assert 0 < t < 100000
    got = _bits(lb)
    lb.close()
    monkeypatch.setenv("HEMELB_FUSE", "0")
    lb = LB.from_geometry(g)
    lb.step(t)
    want = _bits(lb)
    lb.close()
    assert all(torch.equal(a, b) for a, b in zip(want, got))
