"""The network's kernels where a work-group takes several tiles: more than 65536 5D
sites of a parity (the layers' 512 work-groups step several times over their run,
reusing the links staged per wave; the weight gradients' 256 step over their sites),
a last tile that is partial, and for 8 -> 8 channels more than 256 MB (streamed
output). Compared with the 64-bit evaluation of perf/cases.py.

Tolerances as on small lattices: 1e-5 of the largest output (FP32 products and sums
of six layers), 1e-4 of a layer's largest gradient (sums over all sites).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from perf import cases

pytestmark = pytest.mark.gpu

DIMS, LS = (10, 14, 18, 22), 6
SITES = 10 * 14 * 18 * 22 // 2 * LS


def case(kind, channels):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert SITES > 2 * 65536 and SITES % 64 != 0 and 96 * SITES * (2 * 8 + 8) > 256 << 20
    c = dict(kind=kind, lx=DIMS[0], ly=DIMS[1], lz=DIMS[2], lt=DIMS[3], ls=LS, prec="fp32", nrhs=1, eps=0.5, m1=0.04,
             m2=1.0, gparity=False, channels=channels, residual=False)
    return c


@pytest.mark.parametrize("channels", ["1,8,8,1", "1,3,5,1"])
def test_apply(channels):
    c = case("net_apply", channels)
    state = cases.prepare(c, 31)
    state["out"].fill_(255)  # NaN
    got = cases.run(state).double()
    assert bool(torch.isfinite(got).all())
    ref = cases.exact(c, 31)
    assert float((got - ref).abs().max()) < 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("channels", ["1,8,8,1", "1,2,3,1"])
def test_gradients(channels):
    c = case("net_grad", channels)
    loss, grads = cases.run(cases.prepare(c, 32))
    lref, gref = cases.exact(c, 32)
    assert abs(loss - lref) < 1e-5 * abs(lref)
    for g, ref in zip(grads, gref):
        assert np.abs(g - ref).max() < 1e-4 * np.abs(ref).max()
