"""Batched quantisation where its groups of chunks end, and where block scales leave the range of the quotient by reciprocals."""
import numpy as np
import pytest
import torch

import paper_2603_22370_amd as faar
from oracle import faar_oracle as fo

pytestmark = pytest.mark.gpu
GROUP = 4 * 256 * 8     # weights a workgroup takes at a time


def _quantise(Ws, given=None):
    sgs = [torch.full((1,), float("nan") if given is None else given, device="cuda") for _ in Ws]
    scs = [torch.zeros(w.numel() // 16, dtype=torch.uint8, device="cuda") for w in Ws]
    cds = [torch.zeros(w.numel() // 2, dtype=torch.uint8, device="cuda") for w in Ws]
    items, dt = faar.tensor_batch(Ws, sgs, scs, codes=cds)
    ws = torch.empty(faar.faar_workspace_bytes(faar.binding.OP_QUANT_RTN_BATCH, 16, 16), dtype=torch.uint8, device="cuda")
    faar.faar_quant_rtn_batch(items, dt, ws, s_global_given=given is not None)
    return [[t.cpu().numpy() for t in ts] for ts in zip(sgs, scs, cds)]


@pytest.mark.parametrize("dtype,large", [(torch.bfloat16, 700), (torch.float32, 700), (torch.bfloat16, 3), (torch.float32, 3)])
def test_largest_weight_at_the_ends_of_the_groups(dtype, large):
    """One tensor per case, the largest weight its last one, its group's first, or the last of a full group; 72 in one launch, so that
    large tensors beside small ones make a workgroup walk several groups; streamed (700) and within 64 MB (3)."""
    sizes = [16, GROUP - 16, GROUP, GROUP + 16, 2 * GROUP + 16, large * GROUP + 48] * 12
    gen = torch.Generator(device="cuda").manual_seed(5)
    Ws = []
    for k, n in enumerate(sizes):
        w = 0.02 * torch.randn(n, generator=gen, device="cuda")
        w[[n - 1, max(0, (n - 1) // GROUP * GROUP), min(n, GROUP) - 1][k % 3]] = -(7.0 + k)
        Ws.append(w.to(dtype).reshape(1, n))
    for k, (sg, sc, cd) in enumerate(_quantise(Ws)):
        assert sg[0] == np.float32(float(Ws[k].abs().max())) / np.float32(2688.0), k
        if k in (0, 1, 2, 3, 4, 16, 17):
            q = fo.quant_rtn(Ws[k].float().cpu().numpy(), dtype == torch.bfloat16)
            assert np.array_equal(cd, q["codes"].ravel()) and np.array_equal(sc, q["scales"].ravel()), k


@pytest.mark.parametrize("streamed", [False, True])
@pytest.mark.parametrize("scale", [1e-30, 1e-19, 1.0, 1e19, 1e30])
@pytest.mark.parametrize("sg", [1e-25, 3e-4, 1.0, 1e25])
def test_block_scale_bytes_at_any_size(scale, sg, streamed):
    """The block scale is E4M3((amax / 6) / s_global) by IEEE divisions: amax over 24 binades, zero blocks and exact ties among them.
    streamed: in a launch over more than 64 MB, whose kernel makes the quotients through reciprocals."""
    gen = torch.Generator(device="cuda").manual_seed(9)
    a = torch.randn((64, 16), generator=gen, device="cuda") * torch.exp2(torch.arange(64, device="cuda") * 24.0 / 64 - 12.0)[:, None]
    a[3] = 0.0
    W = a * scale
    W[4, :] = 6.0 * 1.0625 * float(np.float32(sg))     # a tie between two E4M3 values where nothing rounds
    W = W.reshape(1, -1).contiguous()
    _, sc, _ = _quantise([W] + [torch.zeros((1, 1 << 24), device="cuda")] * streamed, given=sg)[0]
    with np.errstate(over="ignore", under="ignore"):
        want = fo.block_scale_bytes(W.cpu().numpy(), np.float32(sg))
    assert np.array_equal(sc, np.asarray(want, dtype=np.uint8).ravel())
