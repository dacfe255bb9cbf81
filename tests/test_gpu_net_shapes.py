"""The network layer's kernels over channel counts and shapes where they can go
wrong, against the network oracle: channel pairs on both sides of the line
between the one-thread-per-site and the matrix-core kernels (odd counts, whose
last channel pair is half empty, and 1, 4, 5, 8), tiles of 16 5D sites that
span many 4D sites (Ls = 2) or parts of them (Ls = 6, 10), and lattices whose
last tile is partial.

The weight gradients' channel blocks are checked the same way (1e-4, sums over
all sites of FP32 products, as for the other gradient tests).

Tolerance: bfloat16 weights (the same rounded values in the oracle), FP32
products and sums; each of the six layer applications of N = B^dag B adds a
few 2^-24 of its largest terms, about 1e-6 in all: 1e-5 of the largest entry.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nn
from oracle.dwf import Action
from oracle.lattice import restrict
from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

M5, B5, C5 = 1.8, 1.5, 0.5
BC = (1, 1, 1, -1)


@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((2, 4, 6, 2), 6), ((6, 2, 2, 4), 10)])
@pytest.mark.parametrize("chans", [[1, 4, 5, 1], [1, 3, 2, 1], [1, 5, 8, 1], [1, 8, 3, 1], [1, 2, 4, 1], [1, 7, 1]])
def test_forward_matches_oracle(dims, Ls, chans):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.gauge_field(dims, 0.5, 17)
    ctx = eofa.Context(eofa.make_action(dims, Ls, M5, B5, C5, BC), torch.from_numpy(U).cuda())
    rng = np.random.default_rng(3)
    W = [0.4 * (rng.standard_normal((nn.NTERMS, co, ci)) + 1j * rng.standard_normal((nn.NTERMS, co, ci)))
         for ci, co in zip(chans[:-1], chans[1:])]
    net = eofa.Net(ctx, chans, seed=1)
    net.set_weights(W)
    Wb = [nn.bf16_round(w.astype(np.complex64).astype(np.complex128)) for w in W]
    r = restrict(synth.fermion(dims, Ls, 5), dims, 1).astype(np.complex64).astype(np.complex128)
    pin, pout = ctx.new_packed(eofa.FP32), ctx.new_packed(eofa.FP32)
    ctx.eofa_pack(torch.from_numpy(r[None].copy()).cuda(), pin, 1, eofa.FP32)
    net.apply(ctx, pin, pout)
    full = torch.zeros(ctx.full_shape(1), dtype=torch.complex128, device="cuda")
    ctx.eofa_unpack(pout, full, 1, eofa.FP32)
    got = full[0].cpu().numpy()
    ref = nn.forward(U, Wb, r, dims, BC)[0]
    assert np.abs(got - ref).max() < 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 2), ((6, 2, 2, 4), 10)])
@pytest.mark.parametrize("chans", [[1, 3, 2, 1], [1, 5, 8, 1], [1, 6, 1]])
def test_gradients_match_oracle(dims, Ls, chans):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.gauge_field(dims, 0.5, 18)
    ctx = eofa.Context(eofa.make_action(dims, Ls, M5, B5, C5, BC), torch.from_numpy(U).cuda())
    rng = np.random.default_rng(4)
    W = [0.3 * (rng.standard_normal((nn.NTERMS, co, ci)) + 1j * rng.standard_normal((nn.NTERMS, co, ci)))
         for ci, co in zip(chans[:-1], chans[1:])]
    net = eofa.Net(ctx, chans, seed=1)
    net.set_weights(W)
    Wb = [nn.bf16_round(w.astype(np.complex64).astype(np.complex128)) for w in W]
    f = [restrict(synth.fermion(dims, Ls, k), dims, 1).astype(np.complex64).astype(np.complex128) for k in (6, 7)]
    packed = []
    for x in f:
        packed.append(ctx.new_packed(eofa.FP32))
        ctx.eofa_pack(torch.from_numpy(x[None].copy()).cuda(), packed[-1], 1, eofa.FP32)
    loss, grads = net.loss_grad(ctx, packed[0], packed[1], 1)
    Lref, gref = nn.loss_and_grads(U, Wb, [tuple(f)], dims, BC)
    assert abs(loss - Lref) < 1e-5 * Lref
    for g, ref in zip(grads, gref):
        assert np.abs(g - ref).max() < 1e-4 * np.abs(ref).max()
