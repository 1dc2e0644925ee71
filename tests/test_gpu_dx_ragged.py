"""Input gradient in registers of layers whose quantized part ends inside a group: the last half of a tile ends early and the weak channels begin behind it,
alone in their tile or beside a quantized half, up to two halves of them.  Rows enough that this kernel is the one taken, and few.  Tolerance: parity_util's
bar (weights rounded to fp16 once, 2^-11 relative each, over at least 64 terms; fp16 results)."""
import pytest
import torch

from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("oc,ic,k,bits,m", [(2048, 1024, 64, 4, 8200), (1088, 1024, 8, 4, 8200), (1024, 776, 256, 4, 9001), (64, 1400, 136, 4, 9000), (1024, 1160, 0, 4, 8200),
                                            (1024, 1128, 8, 4, 8193), (2048, 1024, 64, 3, 8200), (1024, 11008, 64, 4, 999), (1024, 8192, 64, 3, 777), (1024, 8192, 8, 3, 1000)])
def test_ragged_input_gradient(oc, ic, k, bits, m):
    layer = HostLayer(oc, ic, k, bits, 128, seed=oc + ic)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    dy = pad_cols(synth.make_grad_output(m, oc, m))[0]
    back = torch.full((m + 2, ic + 8), 7.0, dtype=torch.float16, device="cuda")
    dx = back[1:m + 1, :ic]
    B.qeft_linear_bwd_dx(layer.desc, w, dy, dx)
    first = dx.clone()
    B.qeft_linear_bwd_dx(layer.desc, w, dy, dx)
    ref = dy.double() @ w64
    torch.cuda.synchronize()
    assert torch.equal(first, dx), "repeats differ"
    assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, ic:] == 7).all()), "wrote outside"
    assert_close(dx.cpu().numpy(), ref.cpu().numpy(), "dX")
    if k > 0:   # with the weak gradient's strips behind the tiles (a 3-bit layer: its copy ahead of their partial sums)
        x = torch.randn((m, k), generator=torch.Generator().manual_seed(k)).half().cuda()
        n = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_BWD_DX, m) + B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_WEAK_GRAD, m)
        both, dw = B.qeft_linear_bwd(layer.desc, w, dy, x, ws=torch.empty(n, dtype=torch.uint8, device="cuda") if bits == 3 else None)
        want = B.qeft_weak_grad(layer.desc, dy, x)
        torch.cuda.synchronize()
        assert torch.equal(both, first) and torch.equal(dw, want), "one call"
