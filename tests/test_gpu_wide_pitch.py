"""Rows so far apart that 32-bit offsets from a panel's first do not reach its last: 256 rows at a pitch of more than 2^24 elements, 64 tokens at more
than 2^25, and rows that are just within reach.  Layers of whole and of partial groups, 3-bit ones through their copies.  Tolerance: parity_util's bar."""
import pytest
import torch

from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close

pytestmark = pytest.mark.gpu

LAYERS = [(512, 512, 128, 4), (1024, 520, 8, 4), (512, 520, 40, 4), (264, 640, 0, 4), (1024, 1152, 128, 3), (1024, 1160, 64, 3)]
ROWS = [(256, (1 << 24) + 8), (120, (1 << 24) + 8), (120, (1 << 23) + 8)]


@pytest.fixture(autouse=True)
def give_back():
    yield
    torch.cuda.empty_cache()


def _far(a, pitch):
    out = torch.empty((a.shape[0], pitch), dtype=torch.float16, device="cuda")[:, : a.shape[1]]
    out.copy_(torch.as_tensor(a))
    return out


@pytest.mark.parametrize("m,pitch", ROWS)
@pytest.mark.parametrize("oc,ic,k,bits", LAYERS)
def test_forward_and_backward_of_far_rows(oc, ic, k, bits, m, pitch):
    layer = HostLayer(oc, ic, k, bits, 128, seed=oc + ic)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    x, dy = _far(synth.make_activations(m, ic, k, seed=m), pitch), _far(synth.make_grad_output(m, oc, m), pitch)
    want_y, want_dx = x.double() @ w64.t(), dy.double() @ w64
    for ws in (None, False):
        if bits == 3 and ws is False:
            continue                            # (the general kernels, a row at a time)
        y, dx = B.qeft_linear_fwd(layer.desc, w, x, ws=ws), B.qeft_linear_bwd_dx(layer.desc, w, dy, ws=ws)
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), want_y.cpu().numpy(), "y")
        assert_close(dx.cpu().numpy(), want_dx.cpu().numpy(), "dX")
    if k:
        n = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_BWD, m)
        dx, dw = B.qeft_linear_bwd(layer.desc, w, dy, x[:, ic - k:], ws=torch.empty(n, dtype=torch.uint8, device="cuda") if n else None)
        want_dw = dy.double().t().contiguous() @ x[:, ic - k:].double()
        torch.cuda.synchronize()
        assert_close(dx.cpu().numpy(), want_dx.cpu().numpy(), "dX, one call")
        assert_close(dw.cpu().numpy(), want_dw.cpu().numpy(), "dW, one call")


@pytest.mark.parametrize("far_dy,far_x", [(True, False), (False, True)])
def test_weak_gradient_of_far_tokens(far_dy, far_x):
    m, oc, k, pitch = 66, 72, 40, (1 << 25) + 8
    d = B.make_desc(oc, k + 128, k, 4, 128)
    dy, x = _far(synth.make_grad_output(m, oc, 1), pitch if far_dy else oc), _far(torch.randn((m, k), generator=torch.Generator().manual_seed(1)).half(), pitch if far_x else k)
    want = dy.double().t().contiguous() @ x.double()
    got = [B.qeft_weak_grad(d, dy, x)]
    got.append(B.qeft_weak_grad_noalloc(d, dy, x, torch.zeros((oc, k), device="cuda")))
    torch.cuda.synchronize()
    for g in got:
        assert_close(g.cpu().numpy(), want.cpu().numpy(), "dW")
