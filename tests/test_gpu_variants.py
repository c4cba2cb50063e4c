"""Every product of a layer -- set-up, the step in its forms, the Gram-form step, the forward -- on shapes chosen for the GEMM
instantiations they run (tests/parity_cases.py, VARIANT_SHAPES), against float64 products on the device.

The soft-quantised weights are taken from the library (their own tests compare them with the oracle), rounded to bf16 as its steps
store them, so that no boundary flip of theirs is in the way; what remains per element is float32 accumulation and the bf16
rounding of the output, and in the gradient of a step's own dY the rounding of dY, whose flips move a row of it."""
import pytest
import torch

from parity_cases import VARIANT_SHAPES

pytestmark = pytest.mark.gpu

import paper_2603_22370_amd as faar  # noqa: E402
from paper_2603_22370_amd import binding as fb  # noqa: E402

U8, EPS = 2.0 ** -8, 2.0 ** -24
LAMBDA, BETA, ADAM = 0.01, 12.0, (5e-3, 0.9, 0.999, 1e-8)


def _bf16(x):
    return x.float().to(torch.bfloat16).double()


def _mm(a, b):
    return a.contiguous() @ b.contiguous()


def _check_gradient(m, G, W, sg, scales, V):
    """m of a first step against (1 - beta1) dV, dV by the library's own chain from G to V (tested on its own)."""
    _, want, _ = faar.faar_softquant_fwd_bwd(W, sg, scales, V, BETA, dWt=G.float(), lambda_round=LAMBDA)
    got, want = m.double() / (1 - ADAM[1]), want.double()
    rms = want.pow(2).mean().sqrt()
    assert float((got - want).norm()) <= 3e-4 * float(want.norm())
    assert float((got - want).abs().max() / rms) <= 2e-2 + 2.0 ** -7 * float(want.abs().max() / rms)
    # row by row: a tile, a row or a slice left out or taken twice is an error of order one in its rows
    assert bool(((got - want).norm(dim=1) <= 5e-3 * want.norm(dim=1) + 1e-3 * rms * want.shape[1] ** 0.5).all())


@pytest.mark.parametrize("O,K,T", VARIANT_SHAPES)
def test_all_products_of_a_layer(O, K, T):
    gen = torch.Generator(device="cuda").manual_seed(O * 31 + K * 7 + T)
    W = (0.02 * torch.randn((O, K), generator=gen, device="cuda")).to(torch.bfloat16)
    X = torch.randn((T, K), generator=gen, device="cuda").to(torch.bfloat16)
    Xd, Wd = X.double(), W.double()
    clean = _mm(Xd, Wd.T)
    Y = (clean + 0.05 * torch.randn((T, O), generator=gen, device="cuda")).to(torch.bfloat16)
    sg, scales, _, _ = faar.faar_quant_rtn(W)
    V0 = 0.05 + 0.9 * torch.rand((O, K), generator=gen, device="cuda")
    Wq = faar.faar_softquant_fwd_bwd(W, sg, scales, V0, BETA)[0].double()
    delta = faar.faar_softquant_fwd_bwd(W, sg, scales, V0, BETA, emit_delta=True)[0].double()

    # set-up: C (the bound of one rounding per term), H from the C that was written, ||C||^2
    Xt, C, icodes, H, c_norm2 = faar.faar_layer_prepare(W, sg, scales, X, Y, gradient_constant=True)
    c = C.flatten()[:(T + 3) // 4 * 4 * O].view(-1, O, 4).permute(0, 2, 1).reshape(-1, O).double()
    assert not bool(c[T:].any())
    c = c[:T]
    assert bool(((c - (Y.double() - clean)).abs() <= (K + 2) * EPS * (Y.double().abs() + _mm(Xd.abs(), Wd.abs().T))).all())
    h = H.view(O, K).double()
    assert bool(((h - _mm(c.T, Xd)).abs() <= (3 * T + 4) * EPS * _mm(c.abs().T, Xd.abs())).all())
    assert float(c_norm2) == pytest.approx(float((c * c).sum()), rel=1e-6)

    # the step, on its own and inside a chain, with C and with H
    alpha = 1.0 / (T * O)
    A = _mm(Xd, delta.T)
    R = A - c
    loss = alpha * float((R * R).sum())
    dY_ext = (1e-3 * torch.randn((T, O), generator=gen, device="cuda")).to(torch.bfloat16)
    for chained, own in ((False, False), (True, False), (True, True)):     # own: dX of the step's own dY
        for with_h in (False, True):
            V, m, u = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
            losses = torch.zeros(3, dtype=torch.float32, device="cuda")
            dX = torch.empty((T, K), dtype=torch.bfloat16, device="cuda") if chained else None
            faar.faar_layer_step(W, sg, scales, V, m, u, X, Xt, C, icodes, BETA, LAMBDA, alpha, *ADAM, 1, losses,
                                 faar.layer_step_workspace(O, K, T, chained=chained), dY_ext=None if own or not chained else dY_ext, dX=dX,
                                 H=H if with_h else None, c_norm2=c_norm2 if with_h else None)
            assert float(losses[0]) == pytest.approx(loss, rel=2e-5)
            if chained:
                dY = _bf16(2.0 * alpha * R) if own else dY_ext.double()
                G = _mm(dY.T, Xd)
                want = _mm(dY, Wq)
                # the output's rounding; the step forms W_q in a pass of its own, which may round a value on a bf16 boundary the other
                # way: two such terms of the largest size (two more of its own dY); and one float32 rounding per term
                d = dY.abs()
                flips = (4.0 if own else 2.0) * U8 * d.amax(dim=1, keepdim=True) * Wq.abs().amax(dim=0, keepdim=True)
                assert bool(((dX.double() - want).abs() <= U8 * want.abs() + flips + (O + 2) * EPS * _mm(d, Wq.abs())).all())
                assert float((dX.double() - want).norm()) <= 2.5e-3 * float(want.norm())
            elif with_h:
                G = _mm(_bf16(2.0 * alpha * A).T, Xd) - 2.0 * alpha * h
            else:
                G = _mm(_bf16(2.0 * alpha * R).T, Xd)
            _check_gradient(m, G, W, sg, scales, V0)

    # the Gram form, from the matrix as it is stored
    gram, gram_lo = fb.faar_gram_prepare(Xt, T)
    Gm = gram.view(K, K).double() + torch.diag(gram_lo.double())
    mag = _mm(Xd.abs().T, Xd.abs())
    assert bool(((Gm - _mm(Xd.T, Xd)).abs() <= U8 * _mm(Xd.T, Xd).abs() + (T + 2) * EPS * mag).all())
    V, m, u = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
    losses = torch.zeros(3, dtype=torch.float32, device="cuda")
    fb.faar_layer_step_gram(W, sg, scales, V, m, u, icodes, H, c_norm2, gram, gram_lo, BETA, LAMBDA, alpha, *ADAM, 1, losses,
                            fb.layer_step_gram_workspace(O, K))
    dG = _mm(delta, Gm)
    assert float(losses[0]) == pytest.approx(alpha * float((dG * delta).sum() - 2.0 * (delta * h).sum() + (c * c).sum()), rel=2e-5)
    _check_gradient(m, 2.0 * alpha * (dG - h), W, sg, scales, V0)

    # the forward of a joint step
    got = faar.faar_linear_forward(W, sg, scales, V0, BETA, X).double()
    want = _mm(Xd, Wq.T)
    assert bool(((got - want).abs() <= U8 * want.abs() + (K + 2) * EPS * _mm(Xd.abs(), Wq.abs().T)).all())
