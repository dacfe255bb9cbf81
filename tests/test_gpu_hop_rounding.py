"""The eight-wave form of the hop (hop_small.hip) rounds where the general form
(kernels.hip) does. One system takes the first, the same system batched until
the tiles exceed its range the second.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

M5 = 1.8
DIMS = (4, 4, 4, 4)


def context(Ls, U, b5=1.5):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return eofa.Context(eofa.make_action(DIMS, Ls, M5, b5, b5 - 1.0), torch.from_numpy(U).cuda())


def batch(Ls):
    """Right-hand sides that take the general form: more than 1024 tiles in all."""
    g = 64 // Ls
    tiles = (int(np.prod(DIMS)) // 2 + g - 1) // g
    return 1024 // tiles + 1


def both_forms(ctx, f, prec, dag, m=0.03):
    """Dslash of f alone and as the first of a batch: canonical fields."""
    n = batch(ctx.Ls)
    out = []
    for k in (1, n):
        pin, pout = ctx.new_packed(prec, k), ctx.new_packed(prec, k)
        ctx.eofa_pack(f.expand((k,) + f.shape[1:]).contiguous(), pin, 1, prec, nrhs=k)
        ctx.eofa_dslash([(m, 0.0, 0.0, 0.0, 1)] * k, pin, pout, 0, dag, prec, nrhs=k)
        full = torch.zeros((k,) + f.shape[1:], dtype=f.dtype, device="cuda")
        ctx.eofa_unpack(pout, full, 0, prec, nrhs=k)
        out.append(full[0])
    return out


# One component of one 5D site on unit links: every output is that component
# times the premix factor (c-d)/(c+d) (or 1, or -m times it across the wrap)
# times the leading factor, all other terms exact zeros, so the forms agree to
# the bit if each forms the two factors alike.
@pytest.mark.parametrize("b5", [1.5, 1.6, 1.7, 1.8, 1.95, 2.3])
@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32])
@pytest.mark.parametrize("Ls", [8, 12, 16])
def test_premix_factor(Ls, prec, b5):
    ctx = context(Ls, synth.unit_gauge(DIMS), b5)
    for s, c in ((Ls // 2, 1), (Ls - 1, 4), (0, 9)):  # inside, and both wraps
        f = torch.zeros((1, Ls) + DIMS[::-1] + (4, 3), dtype=torch.complex128, device="cuda")
        f[0, s, 1, 2, 1, 1, c // 3, c % 3] = 1.0
        small, general = both_forms(ctx, f, prec, 0)
        assert int((general != 0).sum()) > 16
        assert torch.equal(small, general), (s, c)


# One 5D site in FP16S: a single direction reaches each output site (extents of
# 4), so the FP32 sum over the directions has one term, (unit times the leading
# factor) times the product, rounded once in either form, and the encoding of it
# is the same bits.
@pytest.mark.parametrize("dag", [0, 1])
@pytest.mark.parametrize("Ls", [6, 8, 10, 12, 16, 20, 24, 32])
def test_half_spinors_fp16s(Ls, dag):
    ctx = context(Ls, synth.gauge_field(DIMS, 0.5, 81))
    x = synth.fermion(DIMS, Ls, 82)
    for s in (0, Ls // 2, Ls - 1):
        f = torch.zeros((1, Ls) + DIMS[::-1] + (4, 3), dtype=torch.complex128, device="cuda")
        f[0, s, 1, 2, 1, 1] = torch.from_numpy(x[s, 1, 2, 1, 1]).cuda()
        small, general = both_forms(ctx, f, eofa.FP16S, dag)
        assert int((general != 0).sum()) > 64
        assert torch.equal(small, general), s


# FP32 iterations at Ls = 16, where the general form sums the series of the
# inverse with one rounding per term. The root mean square distance from the same
# iterations in FP64 is that of the general form or less, up to the scatter of such
# a mean over 4096 5D sites of 24 numbers each, of which at least the 4096 round
# independently: 1 / sqrt(2 x 4096) = 1.1 % a system, 1.1 / sqrt(3) = 0.64 % over
# three, sqrt(2) of it for the ratio of two, and three times that: 2.7 %.
def test_series_rounding():
    Ls = 16
    ctx = context(Ls, synth.gauge_field(DIMS, 0.4, 83))
    kinds = [(1.0, 0.04, 1.0, -1.0, 1), (0.04, 0.04, 1.0, -0.5, -1), (0.1, 0.0, 0.0, 0.0, 1)]
    n = 3 * (batch(Ls) // 3 + 1)
    f = synth.fermion_torch(DIMS, Ls, 84, nrhs=3)
    many, systems = f.repeat((n // 3,) + (1,) * 7), kinds * (n // 3)

    def iterate(prec, sys, phi):
        psi = torch.zeros_like(phi)
        ctx.eofa_cg_solve(sys, phi, psi, eofa.make_params(fixed_iters=3, inner_prec=prec))
        return psi

    general = iterate(eofa.FP32, systems, many)[:3]
    err = [0.0, 0.0]
    for r in range(3):
        one = f[r:r + 1].contiguous()
        exact = iterate(eofa.FP64, kinds[r:r + 1], one)[0]
        small = iterate(eofa.FP32, kinds[r:r + 1], one)[0]
        for k, got in enumerate((small, general[r])):
            err[k] += float((got - exact).abs().square().sum() / exact.abs().square().sum())
    assert (err[0] / err[1]) ** 0.5 < 1.027, err
