"""More right-hand sides than a launch grid's second extent may count: Dslash on the
smallest lattice, against single launches (the same kernel and sums: equal).
"""
import pytest

torch = pytest.importorskip("torch")

from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32])
def test_dslash(prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dims, Ls, n, half = (2, 2, 2, 2), 2, 65536 + 40, 40000
    ctx = eofa.Context(eofa.make_action(dims, Ls, 1.8, 1.5, 0.5), torch.from_numpy(synth.gauge_field(dims, 0.5, 3)).cuda())
    f = synth.fermion_torch(dims, Ls, 4, nrhs=n)
    pin, pout = ctx.new_packed(prec, n), ctx.new_packed(prec, n)
    one = ctx.packed_bytes(prec, 1)
    for a, b in ((0, half), (half, n)):
        ctx.eofa_pack(f[a:b], pin[a * one:b * one], 1, prec, nrhs=b - a)
    systems = [(0.01 * (1 + r % 7), 0.0, 0.0, 0.0, 1) for r in range(n)]
    pout.fill_(255)  # NaN
    ctx.eofa_dslash(systems, pin, pout, 0, 0, prec, nrhs=n)
    assert bool(torch.isfinite(pout.view(torch.float64 if prec == eofa.FP64 else torch.float32)).all())
    k = 2048  # beyond the eight-wave form's range
    for a in (0, 30000, 63000, n - k):
        ref = ctx.new_packed(prec, k)
        ctx.eofa_dslash(systems[a:a + k], pin[a * one:(a + k) * one], ref, 0, 0, prec, nrhs=k)
        assert torch.equal(ref, pout[a * one:(a + k) * one]), a
