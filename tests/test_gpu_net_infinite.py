"""An activation that overflows FP32 stays infinite through the next layer, as in
plain FP32 products, and touches no output that does not depend on it.

N = B^dag B with 1 -> C -> 1 channels, all layers on the matrix cores. The source is
scaled so that one real number of the third layer's output (the C channels of
B^dag) exceeds the FP32 range by a factor of about 1.4 and the next largest stays
below 0.8 of it, as do the terms of its sum that are not its own real part: channel ``big`` at one odd site and s, one component. The last
layer's same-site terms then give w (inf, y) = (Re w inf, Im w inf) at that 5D
site and, through the s shift, at its s neighbour; its transports reach even sites
alone, which N does not return. Every other output is finite and agrees with the
oracle to the tolerance of the layer tests (1e-5 of the largest).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import nn
from oracle.lattice import restrict
from paper_1706_05843_amd import eofa, synth

pytestmark = pytest.mark.gpu

DIMS, LS, BC = (4, 4, 2, 2), 4, (1, 1, 1, -1)
S, SITE, SPIN, COL = 2, (1, 0, 1, 1), 1, 2  # (t, z, y, x), an odd site


# big: inside, and the last of an odd number of channels (whose pair is half empty)
@pytest.mark.parametrize("C,big", [(5, 1), (5, 4), (7, 6), (8, 7)])
def test_overflow_stays_infinite(C, big):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.gauge_field(DIMS, 0.5, 17)
    ctx = eofa.Context(eofa.make_action(DIMS, LS, 1.8, 1.5, 0.5, BC), torch.from_numpy(U).cuda())
    rng = np.random.default_rng(1)
    W = []
    for ci, co in ((1, C), (C, 1)):
        w = 0.02 * (rng.standard_normal((20, co, ci)) + 1j * rng.standard_normal((20, co, ci)))
        w[:2] += 0.25 * (1 + 0.1j)
        W.append(w)
    W[1][:2, 0, big] *= 8
    Wb = [nn.bf16_round(w.astype(np.complex64).astype(np.complex128)) for w in W]
    net = eofa.Net(ctx, [1, C, 1], seed=1)
    net.set_weights(W)

    r = restrict(synth.fermion(DIMS, LS, 5), DIMS, 1)
    r[(S,) + SITE + (SPIN, COL)] = 200.0
    hidden = nn.forward(U, Wb, r, DIMS, BC)[1][1][1]
    top = np.sort(np.abs(np.stack([hidden.real, hidden.imag])).ravel())[::-1]
    r = r * (1.4 * float(np.finfo(np.float32).max) / top[0])
    r = r.astype(np.complex64).astype(np.complex128)
    ref, (X, Y) = nn.forward(U, Wb, r, DIMS, BC)
    over = np.argwhere(np.abs(np.stack([Y[1].real, Y[1].imag])) > np.finfo(np.float32).max)
    assert over.tolist() == [[0, big, S, *SITE, SPIN, COL]] and top[1] * 1.4 < 0.8 * top[0]

    pin, pout = ctx.new_packed(eofa.FP32), ctx.new_packed(eofa.FP32)
    ctx.eofa_pack(torch.from_numpy(r[None].copy()).cuda(), pin, 1, eofa.FP32)
    net.apply(ctx, pin, pout)
    full = torch.zeros(ctx.full_shape(1), dtype=torch.complex128, device="cuda")
    ctx.eofa_unpack(pout, full, 1, eofa.FP32)
    got = full[0].cpu().numpy()
    reached = np.zeros(got.shape, dtype=bool)
    for s, t in ((S, 0), (S - 1, 18)):  # P_+ at the same s, and the adjoint of psi(s - 1)
        k = (s,) + SITE + (SPIN, COL)
        reached[k] = True
        w = np.conj(Wb[0][t, big, 0]) * np.sign(Y[1][(big, S) + SITE + (SPIN, COL)].real)
        assert np.isinf(got[k].real) and np.sign(got[k].real) == np.sign(w.real), (s, got[k])
        assert np.isinf(got[k].imag) and np.sign(got[k].imag) == np.sign(w.imag), (s, got[k])
    assert np.isfinite(got[~reached]).all()
    assert np.abs(got - ref)[~reached].max() < 1e-5 * np.abs(ref).max()


# Activations near the bottom of the FP32 range (the low parts of whose splits are not
# normal numbers): N is linear, and a source scaled by a power of two gives the scaled
# result to the rounding of the layers, 1e-5 of the largest as above, as long as the
# source itself is represented (its largest entries are normal numbers).
@pytest.mark.parametrize("k", [100, 112, 120])
@pytest.mark.parametrize("channels", [[1, 5, 1], [1, 8, 8, 1]])
def test_tiny_activations(channels, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.gauge_field(DIMS, 0.5, 18)
    ctx = eofa.Context(eofa.make_action(DIMS, LS, 1.8, 1.5, 0.5, BC), torch.from_numpy(U).cuda())
    net = eofa.Net(ctx, channels, seed=2, init_scale=0.25)
    r = torch.from_numpy(synth.fermion(DIMS, LS, 6)[None]).cuda()
    out = []
    for f in (1.0, 2.0 ** -k):
        pin, pout = ctx.new_packed(eofa.FP32), ctx.new_packed(eofa.FP32)
        ctx.eofa_pack(r * f, pin, 1, eofa.FP32)
        net.apply(ctx, pin, pout)
        out.append(pout.view(torch.float32).double() / f)
    assert float((out[1] - out[0]).abs().max()) < 1e-5 * float(out[0].abs().max())
