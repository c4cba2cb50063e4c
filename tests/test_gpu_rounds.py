"""Products whose workgroups walk several tiles: ragged in both directions, few and odd numbers of slices, both epilogues, against float64
products on the device; and the widths that they do not take."""
import pytest
import torch

import paper_2603_22370_amd as faar
from paper_2603_22370_amd import binding as fb
from test_gpu_update_in_product import _layer
from test_gpu_variants import ADAM, BETA, EPS, LAMBDA, U8, _bf16, _check_gradient, _mm

pytestmark = pytest.mark.gpu


def _tiles(O, K, T):
    kind, bm, bn, _ = fb.faar_gemm_plan(fb.K_GEMM_FWD, O, K, T)
    return kind, -(-T // bm) * -(-O // bn)


# three slices and more, odd and even numbers of them; 528 to 585 tiles; the last two on the kernel of one tile a workgroup (a width that
# is not a multiple of 4, a contraction beyond 4096)
FORWARD = [(4092, 192, 8429), (4092, 256, 8429), (4100, 576, 8430), (2052, 320, 16389), (2051, 320, 16389), (2056, 4160, 16389)]
STEP = [(4104, 1088, 8384), (6152, 1024, 6208)]


@pytest.mark.parametrize("O,K,T", FORWARD)
def test_forward(O, K, T):
    assert _tiles(O, K, T)[0] == "L64" and _tiles(O, K, T)[1] >= 512
    assert (fb.faar_gemm_form(fb.K_GEMM_FWD, O, K, T) == fb.FORM_WALKS_TILES) == (O % 4 == 0 and K <= 4096)
    W, X, _, sg, scales, V, _ = _layer(O, K, T, torch.bfloat16)
    Wq = faar.faar_softquant_fwd_bwd(W, sg, scales, V, BETA)[0].double()
    got = faar.faar_linear_forward(W, sg, scales, V, BETA, X)
    for rows in torch.arange(T, device="cuda").split(4096):
        x = X[rows].double()
        want = _mm(x, Wq.T)
        assert bool(((got[rows].double() - want).abs() <= U8 * want.abs() + (K + 2) * EPS * _mm(x.abs(), Wq.abs().T)).all())


@pytest.mark.parametrize("O,K,T", STEP)
def test_residual_of_a_step(O, K, T):
    assert _tiles(O, K, T)[0] == "L64" and _tiles(O, K, T)[1] >= 512 and fb.faar_dw_token_major(O, K, T)
    assert fb.faar_gemm_form(fb.K_GEMM_RESIDUAL_H, O, K, T) == fb.FORM_WALKS_TILES
    W, X, Y, sg, scales, V, _ = _layer(O, K, T, torch.bfloat16)
    Xt, C, icodes, H, c_norm2 = faar.faar_layer_prepare(W, sg, scales, X, Y, gradient_constant=True)
    c = C.flatten()[:(T + 3) // 4 * 4 * O].view(-1, O, 4).permute(0, 2, 1).reshape(-1, O).double()[:T]
    delta = faar.faar_softquant_fwd_bwd(W, sg, scales, V, BETA, emit_delta=True)[0].double()
    alpha = 1.0 / (T * O)
    A = _mm(X.double(), delta.T)
    V1, m, u = V.clone(), torch.zeros_like(V), torch.zeros_like(V)
    losses = torch.zeros(3, dtype=torch.float32, device="cuda")
    faar.faar_layer_step(W, sg, scales, V1, m, u, X, Xt, C, icodes, BETA, LAMBDA, alpha, *ADAM, 1, losses,
                         faar.layer_step_workspace(O, K, T), H=H, c_norm2=c_norm2)
    assert float(losses[0]) == pytest.approx(alpha * float(((A - c) ** 2).sum()), rel=2e-5)
    _check_gradient(m, _mm(_bf16(2.0 * alpha * A).T, X.double()) - 2.0 * alpha * H.view(O, K).double(), W, sg, scales, V)
