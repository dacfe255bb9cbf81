"""The two forms of the hop kernel against each other. A launch over few tiles
takes the form that shares a tile among eight waves (hop_small.hip); the same
systems batched over enough right-hand sides take the general form
(kernels.hip). Dslash and its adjoint, and a few fixed CG iterations of both the
Cayley and the dense form (every role of a solve: source, normal operator with
shift on either chirality, residual update, reconstruction, true residual) must
agree, for Ls with one, two and three prime factors, the row form (16) and
columns that leave lanes idle.

Tolerances: FP64, the same sums in another order, 1e-13 for the hop and 1e-11
after the iterations (alpha and beta from sums over the whole lattice); FP32
inner, 2e-6 and, through the iterations' rounding, 1e-4.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

M5, B5, C5 = 1.8, 1.5, 0.5
DIMS = (4, 2, 6, 4)


def setup(Ls):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.gauge_field(DIMS, 0.5, 71)
    ctx = eofa.Context(eofa.make_action(DIMS, Ls, M5, B5, C5), torch.from_numpy(U).cuda())
    g = 64 // Ls
    tiles = (int(np.prod(DIMS)) // 2 + g - 1) // g
    n = 1100 // tiles + 1  # beyond 1024 tiles in all: the general form
    kinds = [(1.0, 0.04, 1.0, -1.0, 1), (0.04, 0.04, 1.0, -0.5, -1), (0.1, 0.0, 0.0, 0.0, 1)]
    systems = [kinds[r % 3] for r in range(n)]
    f = synth.fermion_torch(DIMS, Ls, seed=72, nrhs=n)
    return ctx, systems, f, n


def rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("Ls", [2, 6, 8, 12, 16, 20, 32])
@pytest.mark.parametrize("prec,tol", [(eofa.FP64, 1e-13), (eofa.FP32, 2e-6)])
def test_dslash(Ls, prec, tol):
    ctx, systems, f, n = setup(Ls)
    for dag in (0, 1):
        pin, pout = ctx.new_packed(prec, n), ctx.new_packed(prec, n)
        ctx.eofa_pack(f, pin, 1, prec, nrhs=n)
        ctx.eofa_dslash(systems, pin, pout, 0, dag, prec, nrhs=n)
        out = torch.zeros_like(f)
        ctx.eofa_unpack(pout, out, 0, prec, nrhs=n)
        for r in (0, 1, 2, n - 1):
            one, two = ctx.new_packed(prec), ctx.new_packed(prec)
            ctx.eofa_pack(f[r:r + 1].contiguous(), one, 1, prec)
            ctx.eofa_dslash(systems[r:r + 1], one, two, 0, dag, prec)
            ref = torch.zeros_like(f[:1])
            ctx.eofa_unpack(two, ref, 0, prec)
            assert rel(out[r], ref[0]) < tol, (dag, r)


@pytest.mark.parametrize("Ls", [2, 6, 8, 12, 16, 20, 32])
@pytest.mark.parametrize("prec,tol", [(eofa.FP64, 1e-11), (eofa.FP32, 1e-4)])
@pytest.mark.parametrize("form", [0, 1])
def test_fixed_iterations(Ls, prec, tol, form):
    ctx, systems, f, n = setup(Ls)
    prm = eofa.make_params(fixed_iters=10, inner_prec=prec, form=form)
    psi = torch.zeros_like(f)
    ctx.eofa_cg_solve(systems, f, psi, prm)
    for r in (0, 1, 2, n - 1):
        one = torch.zeros_like(f[:1])
        _, st = ctx.eofa_cg_solve(systems[r:r + 1], f[r:r + 1].contiguous(), one, prm)
        assert np.isfinite(st[0]["true_resid"])
        assert rel(psi[r], one[0]) < tol, r


# FP16S: both forms take the same halves through the same products and differ in
# the order of the FP32 sums alone, which now and then rounds a stored half the
# other way: by 2^-11 of the site's largest value at most, in each of the two
# parts, in few components. Iterations: such a step in each of the ten.
@pytest.mark.parametrize("Ls", [2, 6, 8, 12, 16, 20, 32])
def test_dslash_fp16s(Ls):
    ctx, systems, f, n = setup(Ls)
    prec = eofa.FP16S
    for dag in (0, 1):
        pin, pout = ctx.new_packed(prec, n), ctx.new_packed(prec, n)
        ctx.eofa_pack(f, pin, 1, prec, nrhs=n)
        ctx.eofa_dslash(systems, pin, pout, 0, dag, prec, nrhs=n)
        out = torch.zeros_like(f)
        ctx.eofa_unpack(pout, out, 0, prec, nrhs=n)
        for r in (0, 1, 2, n - 1):
            one, two = ctx.new_packed(prec), ctx.new_packed(prec)
            ctx.eofa_pack(f[r:r + 1].contiguous(), one, 1, prec)
            ctx.eofa_dslash(systems[r:r + 1], one, two, 0, dag, prec)
            ref = torch.zeros_like(f[:1])
            ctx.eofa_unpack(two, ref, 0, prec)
            assert rel(out[r], ref[0]) < 2 ** -10.5 + 2e-6, (dag, r)
            far = (out[r] - ref[0]).abs() > 2e-6 * ref.abs().max()
            assert float(far.float().mean()) < 0.01, (dag, r)


@pytest.mark.parametrize("Ls", [2, 6, 8, 12, 16, 20, 32])
@pytest.mark.parametrize("form", [0, 1])
def test_fixed_iterations_fp16s(Ls, form):
    ctx, systems, f, n = setup(Ls)
    prm = eofa.make_params(fixed_iters=10, inner_prec=eofa.FP16S, form=form)
    psi = torch.zeros_like(f)
    ctx.eofa_cg_solve(systems, f, psi, prm)
    for r in (0, 1, 2, n - 1):
        one = torch.zeros_like(f[:1])
        _, st = ctx.eofa_cg_solve(systems[r:r + 1], f[r:r + 1].contiguous(), one, prm)
        assert np.isfinite(st[0]["true_resid"])
        assert rel(psi[r], one[0]) < 10 * 2 ** -11, r
