"""The site-local kernels (fifth-dimension matrices, packing) at the edges of
their work-group tiles: Ls from 2 to 32 (columns that leave threads of a
work-group over, tiles of one to many sites), lattices whose last tile is
partial, several right-hand sides, every precision.

Tolerances (relative to the largest entry): matrices, 10 x the rounding of a
sum of Ls products (FP64 1e-13, FP32 1e-5) and, stored as FP16S, 1e-3 (half
precision 2^-11 of the site's largest entry, in and out); packing there and
back is exact in FP64 and rounds once in FP32 (6e-8) and FP16S (5e-4).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import fifth
from oracle.dwf import System
from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

M5, B5, C5 = 1.8, 1.5, 0.5
TOL = {eofa.FP64: 1e-13, eofa.FP32: 1e-5, eofa.FP16S: 1e-3}
PACK_TOL = {eofa.FP64: 0.0, eofa.FP32: 6e-8, eofa.FP16S: 5e-4}
SHAPES = [((2, 2, 2, 2), 2), ((6, 2, 4, 2), 10), ((2, 4, 2, 10), 18), ((10, 2, 2, 2), 32), ((4, 6, 2, 4), 16)]


def make(dims, Ls):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.unit_gauge(dims)
    return eofa.Context(eofa.make_action(dims, Ls, M5, B5, C5), torch.from_numpy(U).cuda())


@pytest.mark.parametrize("dims,Ls", SHAPES)
@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32, eofa.FP16S])
def test_mooee_inverse_two_rhs(dims, Ls, prec):
    ctx = make(dims, Ls)
    systems = [System(1.0, 0.04, 1.0, -1.0, +1), System(0.1, 0.04, 1.0, -0.5, -1)]
    psi = synth.fermion(dims, Ls, seed=4, nrhs=2)
    f = torch.from_numpy(psi).cuda()
    pin, pout = ctx.new_packed(prec, 2), ctx.new_packed(prec, 2)
    for dag in (0, 1):
        out = torch.zeros_like(f)
        for par in (0, 1):
            ctx.eofa_pack(f, pin, par, prec, nrhs=2)
            ctx.eofa_mooee_inv(systems, pin, pout, dag, prec, nrhs=2)
            ctx.eofa_unpack(pout, out, par, prec, nrhs=2)
        got = out.cpu().numpy()
        for r, q in enumerate(systems):
            mats = [np.linalg.inv(a) for a in fifth.mee_blocks(Ls, M5, 0.5 * (B5 + C5), 0.5 * (B5 - C5), q.m_op, q.beta,
                                                               q.chi, q.m_a, q.m_b)]
            if dag:
                mats = [a.T for a in mats]
            ref = np.empty_like(psi[r])
            ref[..., :2, :] = np.tensordot(mats[0], psi[r][..., :2, :], axes=1)
            ref[..., 2:, :] = np.tensordot(mats[1], psi[r][..., 2:, :], axes=1)
            assert np.abs(got[r] - ref).max() < TOL[prec] * np.abs(ref).max(), (dag, r)


@pytest.mark.parametrize("dims,Ls", SHAPES)
@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32, eofa.FP16S])
@pytest.mark.parametrize("g5r5", [0, 1])
def test_pack_and_back(dims, Ls, prec, g5r5):
    ctx = make(dims, Ls)
    n = 3
    psi = synth.fermion(dims, Ls, seed=5, nrhs=n)
    f = torch.from_numpy(psi).cuda()
    out = torch.full_like(f, float("nan"))
    for par in (0, 1):
        p = ctx.new_packed(prec, n)
        p.fill_(255)
        ctx.eofa_pack(f, p, par, prec, nrhs=n, g5r5=g5r5)
        ctx.eofa_unpack(p, out, par, prec, nrhs=n)
    ref = psi[:, ::-1].copy() if g5r5 else psi
    if g5r5:
        ref[..., 2:, :] *= -1
    got = out.cpu().numpy()
    big = np.abs(ref).max(axis=(-1, -2), keepdims=True)
    assert np.all(np.abs(got - ref) <= PACK_TOL[prec] * big)
