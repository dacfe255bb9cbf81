"""The hop on a lattice beyond the sweep threshold of the traversal order
(1.5 M 5D sites of a parity: the XCDs share each t slab) and beyond the MALL
(non-temporal output stores in FP64 and FP32), with extents whose t slabs do
not divide into eighths or into whole work-group tiles: every site of the
output is written, and sampled sites agree with the oracle's one-site
evaluation (FP64 rounding 1e-13, FP32 rounding 2e-6 of the largest entry).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import site
from oracle.dwf import Action
from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

M5, B5, C5 = 1.8, 1.5, 0.5


@pytest.fixture(scope="module")
def big():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dims, Ls = (18, 14, 22, 26), 24
    act = Action(dims, Ls, M5, B5, C5, (1, 1, 1, -1))
    U = synth.gauge_field(dims, 0.5, seed=1011)
    ctx = eofa.Context(eofa.make_action(dims, Ls, M5, B5, C5), torch.from_numpy(U).cuda())
    psi = synth.fermion_torch(dims, Ls, seed=2011, nrhs=1)
    yield act, U, ctx, psi
    ctx.close()


@pytest.mark.parametrize("prec,dag,tol", [(eofa.FP64, 0, 1e-13), (eofa.FP64, 1, 1e-13), (eofa.FP32, 0, 2e-6)])
def test_every_site_written_and_sampled(big, prec, dag, tol):
    act, U, ctx, psi = big
    m = 0.03
    pin, pout = ctx.new_packed(prec), ctx.new_packed(prec)
    ctx.eofa_pack(psi, pin, 1, prec)
    pout.fill_(255)  # NaN in either precision
    ctx.eofa_dslash([(m, 0.0, 0.0, 0.0, 1)], pin, pout, 0, dag, prec)
    vals = pout.view(torch.float64 if prec == eofa.FP64 else torch.float32)
    assert bool(torch.isfinite(vals).all())
    out = torch.zeros_like(psi)
    ctx.eofa_unpack(pout, out, 0, prec)
    got, ph = out[0].cpu().numpy(), psi[0].cpu().numpy()
    f = site.dslash_dag_column if dag else site.dslash_column
    rng = np.random.default_rng(7)
    xs = [tuple(int(rng.integers(0, L)) for L in act.dims) for _ in range(24)]
    xs += [(0, 0, 0, 0), tuple(L - 1 for L in act.dims)]
    for x in xs:
        if sum(x) % 2 == 0:
            ref = f(act, U, m, ph, x)
            assert np.abs(got[:, x[3], x[2], x[1], x[0]] - ref).max() < tol * np.abs(ref).max(), x


@pytest.mark.parametrize("prec,n", [(eofa.FP64, 3), (eofa.FP64, 4), (eofa.FP32, 5)])
def test_right_hand_sides_beyond_the_mall_together(prec, n):
    """Fields that fit the MALL one by one and exceed it together (streamed output,
    two right-hand sides per work-group, an odd one left over): the same bits as
    one launch each."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dims, Ls = (18, 14, 20, 12), 12
    ctx = eofa.Context(eofa.make_action(dims, Ls, M5, B5, C5),
                       torch.from_numpy(synth.gauge_field(dims, 0.5, seed=1012)).cuda())
    one = ctx.packed_bytes(prec, 1)
    assert 2 * one < 256 << 20 < 2 * n * one
    f = synth.fermion_torch(dims, Ls, seed=2012, nrhs=n)
    systems = [(0.02 + 0.01 * r, 0.0, 0.0, 0.0, 1) for r in range(n)]
    pin, pout = ctx.new_packed(prec, n), ctx.new_packed(prec, n)
    ctx.eofa_pack(f, pin, 1, prec, nrhs=n)
    for dag in (0, 1):
        pout.fill_(255)
        ctx.eofa_dslash(systems, pin, pout, 0, dag, prec, nrhs=n)
        for r in range(n):
            ref = ctx.new_packed(prec)
            ctx.eofa_dslash(systems[r:r + 1], pin[r * one:(r + 1) * one], ref, 0, dag, prec)
            assert torch.equal(pout[r * one:(r + 1) * one], ref), (dag, r)
    ctx.close()
