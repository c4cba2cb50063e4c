"""Steps of small layers, which are one launch: sizes around its tiles (16 rows, 32 columns a wavefront, 16 and 64 tokens), both weight
types, with the constant in C and as H, against float64 products; and chained through prepared forwards, the check of its tag included."""
import pytest
import torch

import paper_2603_22370_amd as faar
from paper_2603_22370_amd import binding as fb
from test_gpu_update_in_product import _layer, _steps
from test_gpu_variants import ADAM, BETA, LAMBDA, _bf16, _check_gradient, _mm

pytestmark = pytest.mark.gpu

SHAPES = [(1, 16, 1), (16, 32, 16), (250, 256, 64), (256, 256, 64), (33, 240, 65), (1024, 256, 64), (1000, 144, 113),
          (16, 32, 400), (9, 16, 960), (256, 256, 128), (256, 272, 64), (90, 320, 61), (256, 128, 129), (4090, 128, 256)]
# more activations than it takes, more columns a wavefront than it is fast with, or more workgroups than there are slots for the next
# step's sums
BEYOND = [(64, 1024, 16), (256, 512, 32), (64, 336, 64), (256, 272, 65), (256, 256, 129), (17, 48, 63), (9, 16, 961), (128, 16, 1024), (512, 80, 200)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("O,K,T", SHAPES + BEYOND)
def test_small_step(O, K, T, dtype):
    assert fb.faar_gemm_form(fb.K_GEMM_RESIDUAL, O, K, T) == (fb.FORM_WHOLE_STEP if (O, K, T) in SHAPES else 0)
    W, X, Y, sg, scales, V0, _ = _layer(O, K, T, dtype)
    Xt, C, icodes, H, c_norm2 = faar.faar_layer_prepare(W, sg, scales, X, Y, gradient_constant=True)
    alpha = 1.0 / (T * O)
    c = C.flatten()[:(T + 3) // 4 * 4 * O].view(-1, O, 4).permute(0, 2, 1).reshape(-1, O).double()[:T]
    delta = faar.faar_softquant_fwd_bwd(W, sg, scales, V0, BETA, emit_delta=True)[0].double()
    A = _mm(X.double(), delta.T)
    for with_h in (False, True):
        ws = faar.layer_step_workspace(O, K, T)
        ws.fill_(0xA5)

        def step(V, m, u, beta, t, losses, nxt, ready):
            faar.faar_layer_step(W, sg, scales, V, m, u, X, Xt, C, icodes, beta, LAMBDA, alpha, *ADAM, t, losses, ws, beta_next=nxt,
                                 forward_ready=ready, H=H if with_h else None, c_norm2=c_norm2 if with_h else None)
            return []

        V, m, u = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
        losses = torch.zeros(3, dtype=torch.float32, device="cuda")
        step(V, m, u, BETA, 1, losses, 0.0, False)
        R = A - c
        assert float(losses[0]) == pytest.approx(alpha * float((R * R).sum()), rel=2e-5)
        assert float(losses[1]) == pytest.approx(float((1 - (2 * V0.double() - 1) ** 2).mean()), rel=1e-5)
        if with_h:
            G = _mm(_bf16(2.0 * alpha * A).T, X.double()) - 2.0 * alpha * H.view(O, K).double()
        else:
            G = _mm(_bf16(2.0 * alpha * R).T, X.double())
        _check_gradient(m, G, W, sg, scales, V0)
        runs = [_steps(step, V0, prepared) for prepared in (False, True)]
        for k, (a, b) in enumerate(zip(*runs)):
            if k >= 3:
                assert torch.allclose(a, b, rtol=2e-7, atol=0.0), (k, a, b)
            else:
                assert torch.equal(a, b), k
        # the bits of the products on their own, which a step with dX of its own gradient takes
        if not with_h and O % 8 == 0:
            V2, m2, u2 = V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)
            faar.faar_layer_step(W, sg, scales, V2, m2, u2, X, Xt, C, icodes, BETA, LAMBDA, alpha, *ADAM, 1, torch.zeros_like(losses),
                                 faar.layer_step_workspace(O, K, T, chained=True), dX=torch.empty_like(X))
            assert torch.equal(V, V2) and torch.equal(m, m2) and torch.equal(u, u2)
        # told of another step's forward: NaN losses, nothing touched, and no forward is left for anyone
        state = [V0.clone(), torch.zeros_like(V0), torch.zeros_like(V0)]
        step(*state, BETA, 5, losses, 13.0, False)
        snap = [x.clone() for x in state]
        for t in (7, 6):
            bad = torch.zeros(3, dtype=torch.float32, device="cuda")
            step(*state, 13.0, t, bad, 0.0, True)
            assert bool(torch.isnan(bad).all()) and all(torch.equal(x, y) for x, y in zip(state, snap))
