"""The general form of the hop kernels (kernels.hip) in whole solves on lattices
small enough for the oracle. A given launch shape (waves, rhs_block) asks for that
form at any size, and the statistics report the shape that was launched.

* FP64 fixed iterations, every Ls of one to three prime factors and the row form
  (16), against the oracle's mirror-mode CGNR for a shift on either chirality
  and none: 1e-12, for one, two and four waves, and with graph replays (beta step
  in a launch of its own);
* several right-hand sides per work-group, one of them halted: the others agree
  with single solves;
* FP32 and FP16S solves reach a true residual of 1e-10, re-measured by the oracle.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import eo
from oracle.dwf import Action, System, H_system
from oracle.lattice import norm2
from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

M5, B5, C5 = 1.8, 1.5, 0.5
SYSTEMS = [System(1.0, 0.04, 1.0, -1.0, +1), System(0.04, 0.04, 1.0, -0.5, -1), System(0.1)]
DIMS = (4, 2, 2, 4)
ITERS = 20
_SET = {}


def setup(Ls):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if Ls not in _SET:
        act = Action(DIMS, Ls, M5, B5, C5, (1, 1, 1, -1))
        U = synth.gauge_field(DIMS, 0.4, seed=110 + Ls)
        phi = synth.fermion(DIMS, Ls, 120 + Ls, nrhs=3)
        ctx = eofa.Context(eofa.make_action(DIMS, Ls, M5, B5, C5), torch.from_numpy(U).cuda())
        _SET[Ls] = (act, U, phi, ctx)
    return _SET[Ls]


def solve(ctx, systems, phis, **kw):
    ph = torch.from_numpy(np.ascontiguousarray(phis)).cuda()
    psi = torch.zeros_like(ph)
    rc, st = ctx.eofa_cg_solve(systems, ph, psi, eofa.make_params(**kw))
    return rc, st, psi.cpu().numpy()


def rel2(a, b):
    return np.sqrt(norm2(a - b) / norm2(b))


@pytest.mark.parametrize("Ls", [2, 6, 8, 10, 12, 16, 20, 32])
def test_mirror_mode(Ls):
    act, U, phi, ctx = setup(Ls)
    ref = [eo.solve_mirror(act, U, s, phi[r], iters=ITERS)["psi"] for r, s in enumerate(SYSTEMS)]
    for waves, rb, graph in ((1, 3, 0), (2, 2, 0), (4, 1, 0), (2, 3, 1)):
        if Ls == 2 and waves == 4:
            continue  # 128 sites a work-group: beyond the LDS
        _, st, got = solve(ctx, SYSTEMS, phi, fixed_iters=ITERS, waves=waves, rhs_block=rb, use_graph=graph,
                           check_every=4, ring_slots=4)
        assert (st[0]["waves"], st[0]["rhs_block"]) == (waves, rb)
        for r in range(3):
            assert rel2(got[r], ref[r]) < 1e-12, (waves, rb, graph, r)


@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32, eofa.FP16S])
def test_given_shape_takes_the_general_form(prec):
    """A batch beyond the eight-wave form's range and one system of it alone, the same
    shape given for both: the same kernels and sums, the same bits."""
    Ls, n = 8, 300  # 4 tiles each
    act, U, phi, ctx = setup(Ls)
    kw = dict(fixed_iters=5, inner_prec=prec, waves=2, rhs_block=1)
    many = solve(ctx, [SYSTEMS[0]] * n, np.repeat(phi[:1], n, axis=0), **kw)[2]
    one = solve(ctx, SYSTEMS[:1], phi[:1], **kw)[2]
    assert np.array_equal(one[0], many[0]) and np.array_equal(one[0], many[n - 1])


@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("prec", [eofa.FP32, eofa.FP16S])
@pytest.mark.parametrize("Ls", [10, 12, 16])
def test_converged(Ls, prec, form):
    act, U, phi, ctx = setup(Ls)
    rc, st, got = solve(ctx, SYSTEMS, phi, tol=1e-10, inner_prec=prec, form=form, waves=1, rhs_block=3)
    assert rc == eofa.EOFA_OK, st
    for r, s in enumerate(SYSTEMS):
        assert (st[r]["waves"], st[r]["rhs_block"], st[r]["converged"]) == (1, 3, 1)
        assert np.sqrt(norm2(H_system(act, U, s, got[r]) - phi[r]) / norm2(phi[r])) <= 1.05e-10


@pytest.mark.parametrize("prec", [eofa.FP64, eofa.FP32, eofa.FP16S])
@pytest.mark.parametrize("Ls", [12, 16])
def test_one_halted_in_a_shared_work_group(Ls, prec):
    """A zero source halts its right-hand side before the first iteration; the two
    it shares work-groups with take the iterates of a batch without it (the same
    kernels and sums: 1e-13)."""
    act, U, phi, ctx = setup(Ls)
    mid = phi.copy()
    mid[1] = 0.0
    kw = dict(fixed_iters=12, inner_prec=prec, waves=2)
    _, st, got = solve(ctx, SYSTEMS, mid, rhs_block=3, **kw)
    _, _, ref = solve(ctx, [SYSTEMS[0], SYSTEMS[2]], phi[[0, 2]], rhs_block=2, **kw)
    assert st[0]["waves"] == 2 and st[0]["rhs_block"] == 3
    assert np.all(got[1] == 0.0)
    assert rel2(got[0], ref[0]) < 1e-13 and rel2(got[2], ref[1]) < 1e-13


@pytest.mark.parametrize("noalloc", [False, True])
def test_shape_reported_for_few_tiles(noalloc):
    """Without a given shape few tiles take the eight-wave form, nothing to tune."""
    act, U, phi, ctx = setup(8)
    ph = torch.from_numpy(phi).cuda()
    psi = torch.zeros_like(ph)
    call = ctx.eofa_cg_solve_noalloc if noalloc else ctx.eofa_cg_solve
    rc, st = call(SYSTEMS, ph, psi, eofa.make_params(tol=1e-10))
    assert rc == eofa.EOFA_OK
    assert all((s["waves"], s["rhs_block"]) == (8, 1) for s in st)


@pytest.mark.parametrize("Ls,dims,n,few", [(32, (4, 2, 2, 2), 32, True), (32, (4, 2, 2, 2), 33, False),
                                           (24, (4, 2, 2, 2), 85, True), (24, (4, 2, 2, 2), 86, False),
                                           (8, (4, 2, 2, 2), 512, True), (8, (4, 2, 2, 2), 513, False)])
def test_dense_roles_line(Ls, dims, n, few):
    """The dense form leaves the eight-wave kernels at fewer tiles the larger Ls is (256
    tiles at 32, 16384 / Ls below); the Cayley form of the same batch stays."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = eofa.Context(eofa.make_action(dims, Ls, M5, B5, C5), torch.from_numpy(synth.unit_gauge(dims)).cuda())
    phi = synth.fermion_torch(dims, Ls, 5, nrhs=n)
    psi = torch.empty_like(phi)
    for form in (0, 1):
        _, st = ctx.eofa_cg_solve([SYSTEMS[2]] * n, phi, psi,
                                  eofa.make_params(fixed_iters=1, inner_prec=eofa.FP32, form=form))
        assert (st[0]["waves"] == 8) == (few or (form == 0 and Ls != 8)), form
    ctx.close()
