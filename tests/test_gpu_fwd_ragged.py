"""Forward with weights in registers of layers whose quantized part ends inside a stage of 64 columns: what is left of it (8 to 56 columns) goes with the
weak block, which may end in the same stage, in a later one, or not exist; one whole stage at least.  Channels and rows that end inside tiles, every panel
height, 3-bit layers through their copy.  Tolerance: parity_util's bar (weights rounded to fp16 once, 2^-11 relative each, over at least 64 terms; fp16 results)."""
import pytest
import torch

from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("oc,ic,k,bits,ms", [(16384, 600, 8, 4, (500, 1300)), (16392, 72, 0, 4, (900,)), (16384, 256, 136, 4, (520, 640)), (8200, 1160, 40, 4, (1000, 2048)),
                                             (16384, 184, 64, 4, (769,)), (28672, 512, 24, 4, (333,)), (8192, 1152, 16, 3, (1500,)), (24576, 320, 256, 4, (150, 3000))])
def test_ragged_forward(oc, ic, k, bits, ms):
    layer = HostLayer(oc, ic, k, bits, 128, seed=oc + ic)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    for m in ms:
        x = pad_cols(synth.make_activations(m, ic, k, m))[0]
        back = torch.full((m + 2, oc + 8), 7.0, dtype=torch.float16, device="cuda")
        y = back[1:m + 1, :oc]
        B.qeft_linear_fwd(layer.desc, w, x, y)
        first = y.clone()
        B.qeft_linear_fwd(layer.desc, w, x, y)
        ref = x.double() @ w64.t().contiguous()
        torch.cuda.synchronize()
        assert torch.equal(first, y), f"M={m}: repeats differ"
        assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, oc:] == 7).all()), f"M={m}: wrote outside"
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"M={m}")
