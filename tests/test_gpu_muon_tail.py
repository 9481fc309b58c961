"""The weight step of large batches: one rule in all tiles of a matrix, and no
fewer bits of X_T than the output of the same call shows.  The comparisons are
with the same iteration's own X_T, exact but for the fused multiply-add, which is
redone in 64 bits."""
import numpy as np
import pytest

import synth
from tests.gpu_util import oracle_schedule

pytestmark = pytest.mark.gpu

LR = 0.03125  # exact in FP32; with wd = 0 and beta = 0 the iteration runs on G and W' = W - lr X_T


def _call(pe, count, shape, wdtype, out, seed, **kw):
    """W and W' of the first and last matrices, the call's output (out: its type) and
    X_T in FP32 of the same call without the weight step."""
    import torch
    abc = oracle_schedule(5)
    r = synth.rng(seed)
    G = torch.from_numpy(r.standard_normal(shape).astype(np.float32)).cuda().to(torch.bfloat16)
    W0 = torch.from_numpy(r.standard_normal(shape).astype(np.float32)).cuda().to(wdtype)
    Ms = [torch.zeros(shape, dtype=torch.float32, device="cuda") for _ in range(count)]
    Ws = [W0.clone() for _ in range(count)]
    outs = [torch.empty(shape, dtype=out, device="cuda") for _ in range(count)] if out is not None else None
    pe.muon_step([G] * count, Ms, Ws, lr=LR, beta=0.0, T=5, abc=abc, outs=outs, **kw)
    torch.cuda.synchronize()
    pick = (0, count - 1)
    return W0, [Ws[i] for i in pick], [outs[i] for i in pick] if outs is not None else None, G, abc


def _stepped(W0, X):
    """W - lr X in 64 bits, rounded to FP32 and to W's type."""
    import torch
    return (W0.double() - LR * X.double()).to(torch.float32).to(W0.dtype)


@pytest.mark.parametrize("wdtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("count,shape", [(17, (512, 2048)), (17, (2040, 500)), (20, (512, 2048))])
def test_bf16_output_and_weights_agree_in_every_tile(count, shape, wdtype):
    """16 tiles of 256 per matrix: the last matrix runs on 64 tiles (17), the last
    four on 128 tiles (20)."""
    import torch
    import paper_2505_16932_amd as pe
    W0, Ws, Xs, _, _ = _call(pe, count, shape, getattr(torch, wdtype), torch.bfloat16, 9900 + count, tile=2)
    for W, X in zip(Ws, Xs):
        assert int((W != _stepped(W0, X)).sum()) == 0


@pytest.mark.parametrize("count,shape,tile", [(17, (512, 2048), 2), (16, (1536, 1536), 0)])
def test_weights_alone_take_fp32_steps(count, shape, tile):
    """No output: W' comes from the FP32 X_T on the 256 tile too, which batches of
    576 update tiles take by size; 16 x 1536 x 1536 with little padding."""
    import torch
    import paper_2505_16932_amd as pe
    W0, Ws, _, G, abc = _call(pe, count, shape, torch.float32, None, 9950 + count, tile=tile)
    Ms = [torch.zeros(shape, dtype=torch.float32, device="cuda") for _ in range(count)]
    Xs = pe.polar_batched([G] * count, T=5, abc=abc, out_dtype=torch.float32, tile=tile, moms=Ms, muon=(0.0, 0.0, 0.0))
    torch.cuda.synchronize()
    for W, X in zip(Ws, (Xs[0], Xs[-1])):
        assert int((W != _stepped(W0, X)).sum()) == 0


def test_batch_of_two_rounds_with_bf16_output_keeps_fp32_steps():
    """The same batch with a bf16 output stays on the small tiles, whose weight step
    takes the FP32 X_T."""
    import torch
    import paper_2505_16932_amd as pe
    W0, Ws, Xs, G, abc = _call(pe, 16, (1536, 1536), torch.float32, torch.bfloat16, 9980)
    Ms = [torch.zeros((1536, 1536), dtype=torch.float32, device="cuda") for _ in range(16)]
    X32 = pe.polar_batched([G] * 16, T=5, abc=abc, out_dtype=torch.float32, tile=1, moms=Ms, muon=(0.0, 0.0, 0.0))
    torch.cuda.synchronize()
    for W, X, B in zip(Ws, (X32[0], X32[-1]), Xs):
        assert torch.equal(X.to(torch.bfloat16), B)
        assert int((W != _stepped(W0, X)).sum()) == 0
