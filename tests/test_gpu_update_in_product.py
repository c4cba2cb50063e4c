"""Products that end in the pass over V (dW where the plan does not split it, the Gram form's on large layers): every tile shape with both
weight types against float64 products on the device, and steps chained through the forward that they leave against steps that make
their own."""
import pytest
import torch

import paper_2603_22370_amd as faar
from paper_2603_22370_amd import binding as fb
from test_gpu_variants import ADAM, BETA, LAMBDA, _bf16, _check_gradient, _mm

pytestmark = pytest.mark.gpu

# (O, K, T, alone on the device): N64, S64, M64, L64 on transposed operands, the three token-major tiles; ragged edges in both directions;
# 1600 tiles of 256x256, for which there are slots for the next step's partial sums, and 2160 of 192x256, for which there are not
DW = [(1056, 656, 64, False), (648, 2816, 64, False), (648, 5408, 64, False), (7176, 1088, 65, False), (7176, 1088, 64, False),
      (7176, 1088, 64, True), (6224, 1808, 64, True), (5120, 20480, 64, True)]
# M64, S64, then L64: 256x256, 192x256, 256x192; contractions that end inside a slice and that do not
GRAM = [(8872, 592), (8432, 624), (8200, 640), (6496, 1232), (8192, 512), (8256, 1552), (8256, 1584), (8256, 1600), (7176, 1088), (6632, 1232),
        (7040, 1664), (8128, 1376)]


def _layer(O, K, T, dtype):
    gen = torch.Generator(device="cuda").manual_seed(O * 31 + K * 7 + T)
    W = (0.02 * torch.randn((O, K), generator=gen, device="cuda")).to(dtype)
    X = torch.randn((T, K), generator=gen, device="cuda").to(torch.bfloat16)
    Y = (X.float() @ W.float().T + 0.05 * torch.randn((T, O), generator=gen, device="cuda")).to(torch.bfloat16)
    sg, scales, _, _ = faar.faar_quant_rtn(W)
    V = 0.05 + 0.9 * torch.rand((O, K), generator=gen, device="cuda")
    return W, X, Y, sg, scales, V, gen


def _steps(step, V0, prepared, betas=(BETA, 13.0, 14.5)):
    """Three steps, each on a forward of its own or on the one the step before left; t from 2, so that both turns of the Gram form's
    buffers come first."""
    V, m, u = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
    out = []
    for i, beta in enumerate(betas):
        losses = torch.zeros(3, dtype=torch.float32, device="cuda")
        nxt = betas[i + 1] if prepared and i + 1 < len(betas) else 0.0
        extra = step(V, m, u, beta, 2 + i, losses, nxt, prepared and i > 0)
        out += [losses, *(x.clone() for x in extra)]
    return [V, m, u, *out]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("O,K,T,alone", DW)
def test_weight_gradient_that_updates_v(O, K, T, alone, dtype):
    assert fb.faar_gemm_plan(fb.K_GEMM_DW, O, K, T)[3] == 1
    assert fb.faar_gemm_form(fb.K_GEMM_DW, O, K, T) == fb.FORM_UPDATES_V | fb.FORM_UPDATES_V_WITH_DX
    W, X, Y, sg, scales, V0, gen = _layer(O, K, T, dtype)
    Xt, C, icodes, H, c_norm2 = faar.faar_layer_prepare(W, sg, scales, X, Y, gradient_constant=True)
    alpha = 1.0 / (T * O)
    dY = (1e-3 * torch.randn((T, O), generator=gen, device="cuda")).to(torch.bfloat16)

    def step(chained, own, ws, V, m, u, beta, t, losses, nxt, ready):
        dX = torch.empty((T, K), dtype=torch.bfloat16, device="cuda") if chained else None
        faar.faar_layer_step(W, sg, scales, V, m, u, X, Xt, C, icodes, beta, LAMBDA, alpha, *ADAM, t, losses, ws,
                             dY_ext=dY if chained and not own else None, dX=dX, beta_next=nxt, forward_ready=ready, H=H, c_norm2=c_norm2,
                             whole_device=alone)
        return [dX] if chained else []

    delta = faar.faar_softquant_fwd_bwd(W, sg, scales, V0, BETA, emit_delta=True)[0].double()
    for chained, own in ((False, False), (True, False), (True, True)):      # own: dX of the step's own gradient
        ws = faar.layer_step_workspace(O, K, T, chained=chained)
        V, m, u = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
        step(chained, own, ws, V, m, u, BETA, 1, torch.zeros(3, device="cuda"), 0.0, False)
        if own:
            c = C.flatten()[:(T + 3) // 4 * 4 * O].view(-1, O, 4).permute(0, 2, 1).reshape(-1, O).double()[:T]
            G = _mm(_bf16(2.0 * alpha * (_mm(X.double(), delta.T) - c)).T, X.double())
        elif chained:
            G = _mm(dY.double().T, X.double())
        else:
            G = _mm(_bf16(2.0 * alpha * _mm(X.double(), delta.T)).T, X.double()) - 2.0 * alpha * H.view(O, K).double()
        _check_gradient(m, G, W, sg, scales, V0)
        runs = [_steps(lambda *a: step(chained, own, ws, *a), V0, prepared) for prepared in (False, True)]
        for k, (a, b) in enumerate(zip(*runs)):
            if a.dtype == torch.float32 and a.numel() == 3:      # the same terms, added up in other groups
                assert torch.allclose(a, b, rtol=2e-7, atol=0.0), (k, a, b)
            else:
                assert torch.equal(a, b), k
        # told of another step's forward: NaN losses, nothing touched, and no forward is left for anyone
        state = [V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)]
        step(chained, own, ws, *state, BETA, 5, torch.zeros(3, device="cuda"), 13.0, False)
        snap = [x.clone() for x in state]
        for t in (7, 6):
            bad = torch.zeros(3, dtype=torch.float32, device="cuda")
            step(chained, own, ws, *state, 13.0, t, bad, 0.0, True)
            assert bool(torch.isnan(bad).all()) and all(torch.equal(x, y) for x, y in zip(state, snap))


@pytest.mark.parametrize("T", [64, 65])
def test_input_gradient_in_the_place_of_the_activations(T):
    """dX comes before the product that updates V where that is faster, but not where it would overwrite an operand of it."""
    O, K = 7176, 1088
    W, X, Y, sg, scales, V0, gen = _layer(O, K, T, torch.bfloat16)
    Xt, C, icodes = faar.faar_layer_prepare(W, sg, scales, X, Y)
    dY = (1e-3 * torch.randn((T, O), generator=gen, device="cuda")).to(torch.bfloat16)
    ws = faar.layer_step_workspace(O, K, T, chained=True)
    runs = []
    for in_place in (False, True):
        x, state = X.clone(), [V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)]
        dX = x if in_place else torch.empty_like(x)
        faar.faar_layer_step(W, sg, scales, *state, x, Xt, C, icodes, BETA, LAMBDA, 1.0 / (T * O), *ADAM, 1,
                             torch.zeros(3, dtype=torch.float32, device="cuda"), ws, dY_ext=dY, dX=dX)
        runs.append([*state, dX])
    assert all(torch.equal(a, b) for a, b in zip(*runs))


def _distance_from_64_bits(O, K, T, alone):
    """Of the gradient in m after a first step on an upstream gradient, relative to its norm; dL/dV is affine in the gradient, its factor
    taken from the library's own backward pass (float32: about 3e-7 of every distance)."""
    W, X, Y, sg, scales, V, gen = _layer(O, K, T, torch.bfloat16)
    Xt, C, icodes = faar.faar_layer_prepare(W, sg, scales, X, Y)
    dY = torch.randn((T, O), generator=gen, device="cuda").to(torch.bfloat16)
    G = _mm(dY.double().T, X.double())
    _, factor, _ = faar.faar_softquant_fwd_bwd(W, sg, scales, V, BETA, dWt=torch.ones_like(V))
    want = G * factor.double() + LAMBDA / (O * K) * (4.0 - 8.0 * V.double())
    m, u = torch.zeros_like(V), torch.zeros_like(V)
    faar.faar_layer_step(W, sg, scales, V, m, u, X, Xt, C, icodes, BETA, LAMBDA, 1.0 / (T * O), *ADAM, 1,
                         torch.zeros(3, dtype=torch.float32, device="cuda"), faar.layer_step_workspace(O, K, T, chained=True), dY_ext=dY,
                         whole_device=alone)
    return float((m.double() / (1 - ADAM[1]) - want).norm() / want.norm())


@pytest.mark.parametrize("alone", [False, True])
@pytest.mark.parametrize("O,K", [(6144, 2048), (4096, 3072)])
def test_planned_splits_stay_split(O, K, alone):
    """Over 16384 tokens the plan has partial sums over at most 8192 of them, over 8192 a single sum: rounding errors grow with the root of
    a sum's length, so the former are no further from 64 bits than the latter."""
    assert fb.faar_gemm_plan(fb.K_GEMM_DW, O, K, 16384)[3] > 1 and fb.faar_gemm_plan(fb.K_GEMM_DW, O, K, 8192)[3] == 1
    assert _distance_from_64_bits(O, K, 16384, alone) <= _distance_from_64_bits(O, K, 8192, alone)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("O,K", GRAM)
def test_gram_product_that_updates_v(O, K, dtype):
    T = 192
    assert O * K >= 1 << 22 and fb.faar_gemm_plan(fb.K_GEMM_GRAM, O, K, 1)[3] == 1
    assert fb.faar_gemm_form(fb.K_GEMM_GRAM, O, K, 1) == fb.FORM_UPDATES_V
    W, X, Y, sg, scales, V0, _ = _layer(O, K, T, dtype)
    Xt, C, icodes, H, c_norm2 = faar.faar_layer_prepare(W, sg, scales, X, Y, gradient_constant=True)
    gram, gram_lo = fb.faar_gram_prepare(Xt, T)
    alpha = 1.0 / (T * O)
    ws = fb.layer_step_gram_workspace(O, K)
    ws.fill_(0xA5)

    def step(V, m, u, beta, t, losses, nxt, ready):
        fb.faar_layer_step_gram(W, sg, scales, V, m, u, icodes, H, c_norm2, gram, gram_lo, beta, LAMBDA, alpha, *ADAM, t, losses, ws,
                                beta_next=nxt, forward_ready=ready)
        return []

    V, m, u = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
    losses = torch.zeros(3, dtype=torch.float32, device="cuda")
    step(V, m, u, BETA, 1, losses, 0.0, False)
    delta = faar.faar_softquant_fwd_bwd(W, sg, scales, V0, BETA, emit_delta=True)[0].double()
    h = H.view(O, K).double()
    dG = _mm(delta, gram.view(K, K).double() + torch.diag(gram_lo.double()))
    want = alpha * float((dG * delta).sum() - 2.0 * (delta * h).sum() + c_norm2.double())
    assert float(losses[0]) == pytest.approx(want, rel=2e-5)
    _check_gradient(m, 2.0 * alpha * (dG - h), W, sg, scales, V0)
    runs = [_steps(step, V0, prepared) for prepared in (False, True)]
    for k, (a, b) in enumerate(zip(*runs)):
        if a.numel() == 3:
            assert torch.allclose(a, b, rtol=2e-7, atol=0.0), (k, a, b)
        else:
            assert torch.equal(a, b), k
    # a step told of a forward that is another step's: NaN losses, nothing touched, and no forward is left for anyone
    state = [V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)]
    first = torch.zeros(3, dtype=torch.float32, device="cuda")
    step(*state, BETA, 5, first, 13.0, False)
    snap = [x.clone() for x in state]
    for t in (7, 6):
        bad = torch.zeros(3, dtype=torch.float32, device="cuda")
        step(*state, 13.0, t, bad, 0.0, True)
        assert bool(torch.isnan(bad).all()) and all(torch.equal(x, y) for x, y in zip(state, snap))
