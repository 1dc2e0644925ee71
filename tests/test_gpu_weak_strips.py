"""Weak block's gradient in pieces of 64 and of 128 columns: pieces that end early, channels and tokens that end inside a strip and a stage,
more than one split, more pieces than CUs.  Tolerance per element: fp32 sums of M products that are exact in fp32, (M + 2) 2^-24 of the sum of their magnitudes."""
import pytest
import torch

from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import pad_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("oc,k", [(72, 8), (136, 64), (1000, 72), (264, 128), (520, 192), (64, 256), (4104, 40), (8256, 128), (16456, 72), (16448, 96), (26176, 72), (9032, 136)])
def test_weak_gradient_in_pieces(oc, k):
    d = B.make_desc(oc, k + 128, k, 4, 128)
    for m in (64, 65, 127, 128, 191, 449, 1000):
        dy = pad_cols(synth.make_grad_output(m, oc, m))[0]
        x = torch.randn((m, k + 8), generator=torch.Generator().manual_seed(m)).half().cuda()
        back = torch.full((oc + 2, k), 7.0, device="cuda")
        dw = back[1:oc + 1]
        B.qeft_weak_grad(d, dy, x[:, :k], dW=dw)
        first = dw.clone()
        B.qeft_weak_grad(d, dy, x[:, :k], dW=dw)
        torch.cuda.synchronize()
        assert torch.equal(first, dw), f"M={m}: repeats differ"
        assert bool((back[0] == 7).all()) and bool((back[oc + 1] == 7).all()), f"M={m}: wrote outside"
        a, b = dy.double().t().contiguous(), x[:, :k].double()
        assert bool(((dw.double() - a @ b).abs() <= (m + 2) * 2.0 ** -24 * (a.abs() @ b.abs())).all()), f"M={m}"
