"""Forward and input gradient in tiles of 128 channels x 64 or 128 rows (calls without a split workspace), at their edges:
rows and channels that end inside a tile, a contraction shorter than the workgroup's shares, a ragged last group or stage,
weak blocks of none, less than a stage and more stages than shares.  Tolerance: parity_util's bar (weights rounded to fp16
once, 2^-11 relative each, over at least 64 terms; fp16 results)."""
import numpy as np
import pytest
import torch

from oracle import qeft_oracle as qo
from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu


def _run(call, m, cols, what, ref):
    back = torch.full((m + 2, (cols + 7) // 8 * 8 + 8), 7.0, dtype=torch.float16, device="cuda")
    out = back[1:m + 1, :cols]
    call(out)
    first = out.clone()
    call(out)
    torch.cuda.synchronize()
    assert torch.equal(first, out), f"{what}: repeats differ"
    assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, cols:] == 7).all()), f"{what}: wrote outside"
    assert_close(out.cpu().numpy(), ref, what)


# (oc, ic, k, rows)
FWD = [
    (200, 512 + 64, 64, (97, 193, 320)),          # 200 channels: the second tile mostly empty; one K group has no chunk in the second turn
    (264, 1352, 264, (257,)),                     # five weak stages for two shares, the last ragged; Kq = 1088 = 17 stages
    (392, 4080 + 16, 16, (130, 200, 400)),        # the last stage 48 columns wide (130 rows: the mid-row kernel)
    (136, 896, 0, (209,)),                        # nothing weak
    (4104, 1024 + 8, 8, (777,)),                  # 128-row tiles
    (2056, 1600, 128, (1000, 515)),
]
DX = [
    (64, 512 + 8, 8, (17, 64)),                   # (whole groups, one stage: the large tiles)
    (64, 504 + 16, 16, (17, 64)),                 # one stage of rows for eight shares of half-stages
    (320, 1024 + 136, 136, (65, 130)),            # two weak tiles, the second 8 wide; five stages
    (1088, 256, 0, (200,)),                       # nothing weak
    (1024, 3968 + 128, 128, (777, 129)),          # 128-row tiles
    (4160, 896 + 64, 64, (97,)),
    (192, 1000 + 24, 24, (97, 260)),              # a partial last group of 104 channels, then the weak ones
    (128, 8 + 200, 200, (33,)),                   # eight quantized channels, two weak tiles
]


@pytest.mark.parametrize("oc,ic,k,rows", FWD)
def test_forward(oc, ic, k, rows):
    layer = HostLayer(oc, ic, k, 4, 128, seed=oc + k)
    w = layer.to_device()
    for m in rows:
        x = synth.make_activations(m, ic, k, seed=m)
        xd, _ = pad_cols(x)
        _run(lambda out: B.qeft_linear_fwd(layer.desc, w, xd, out, ws=False), m, oc, f"M={m}", qo.linear_fwd(layer.w64, x))


@pytest.mark.parametrize("oc,ic,k,rows", DX)
def test_input_gradient(oc, ic, k, rows):
    layer = HostLayer(oc, ic, k, 4, 128, seed=oc + k)
    w = layer.to_device()
    for m in rows:
        dy = synth.make_grad_output(m, oc, seed=m)
        dyd, _ = pad_cols(dy)
        _run(lambda out: B.qeft_linear_bwd_dx(layer.desc, w, dyd, out, ws=False), m, ic, f"M={m}", qo.linear_bwd_dx(layer.w64, dy))


@pytest.mark.parametrize("bits,dense", [(4, False), (3, True)])
@pytest.mark.parametrize("oc,ic,k,rows", [
    (72, 384 + 128, 128, (17, 64)),               # the second stage has 8 rows of its own, the third weak stage of 32 too
    (200, 1000 + 136, 136, (65, 129)),            # four stages, the last of 8 rows, for eight shares; partial group, two weak tiles
    (120, 512, 0, (100,)),
    (1016, 2048 + 64, 64, (97, 300)),             # 15 whole stages and 56 rows
    (4104, 896 + 8, 8, (777,)),                   # 128-row tiles
])
def test_input_gradient_of_any_number_of_channels(oc, ic, k, rows, bits, dense):
    """OC no multiple of the stages of 64 (quantized) and 32 (weak) rows: the last begins before its own rows."""
    layer = HostLayer(oc, ic, k, bits, 128, seed=oc + k, dense=dense)
    w = layer.to_device()
    for m in rows:
        dy = synth.make_grad_output(m, oc, seed=m)
        dyd, _ = pad_cols(dy)
        n = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_BWD_DX, m)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda") if bits == 3 else False
        _run(lambda out: B.qeft_linear_bwd_dx(layer.desc, w, dyd, out, ws=ws), m, ic, f"M={m}", qo.linear_bwd_dx(layer.w64, dy))


def test_backward_call_equals_the_two_calls():
    """qeft_linear_bwd with the weak gradient's workspace alone: bit for bit qeft_linear_bwd_dx without one and qeft_weak_grad."""
    layer = HostLayer(512, 1024 + 128, 128, 4, 128, seed=4)
    w, m = layer.to_device(), 333
    x, dy = synth.make_activations(m, 1152, 128, seed=1), synth.make_grad_output(m, 512, seed=2)
    xd, dyd = pad_cols(x)[0], pad_cols(dy)[0]
    dx, dw = B.qeft_linear_bwd(layer.desc, w, dyd, xd[:, 1024:])
    dx2, dw2 = B.qeft_linear_bwd_dx(layer.desc, w, dyd, ws=False), B.qeft_weak_grad(layer.desc, dyd, xd[:, 1024:])
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2) and torch.equal(dw, dw2)


def test_fractional_zero_points():
    layer = HostLayer(256, 512 + 64, 64, 4, 128, seed=5)
    layer.zeros = (np.random.default_rng(9).integers(-40, 60, layer.zeros.shape) / 2).astype(np.float16)
    w, m = layer.to_device(), 150
    x, dy = synth.make_activations(m, 576, 64, seed=6), synth.make_grad_output(m, 256, seed=7)
    y, dx = B.qeft_linear_fwd(layer.desc, w, pad_cols(x)[0], ws=False), B.qeft_linear_bwd_dx(layer.desc, w, pad_cols(dy)[0], ws=False)
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), "forward")
    assert_close(dx.cpu().numpy(), qo.linear_bwd_dx(layer.w64, dy), "input gradient")


@pytest.mark.parametrize("oc,ic,k,bits", [(264, 1160, 72, 4), (4104, 712, 8, 4), (2048, 2048 + 128, 128, 4), (1024, 8192, 256, 4), (1024, 1152, 128, 3), (2560, 2048, 64, 3)])
@pytest.mark.parametrize("m", [64, 130, 520, 1000])
def test_backward_takes_the_weak_gradient_along(m, oc, ic, k, bits):
    """The weak gradient's strips behind the tiles of dX, or beside the sum of a split's partial tiles, with and without slabs of their own and
    room for them: bit for bit the two calls, nothing written past the workspace.  (The calls' own values are checked elsewhere.)"""
    layer = HostLayer(oc, ic, k, bits, 128, seed=oc + m)
    w, d = layer.to_device(), layer.desc
    dy, x = (pad_cols(a)[0] for a in (synth.make_grad_output(m, oc, m), synth.make_activations(m, ic, k, m)))
    xw = x[:, ic - k:].contiguous()
    sizes = [B.qeft_workspace_bytes(d, op, m) for op in (B.QEFT_OP_WEAK_GRAD, B.QEFT_OP_BWD, B.QEFT_OP_BWD_DX)]
    for n in sorted({sizes[0], sizes[1], sizes[1] + sizes[0] + 16}):
        if bits == 3 and n < sizes[2]:
            continue                               # (the general kernel)
        ws = torch.full((n + 64,), 171, dtype=torch.uint8, device="cuda")
        want_dx = B.qeft_linear_bwd_dx(d, w, dy, ws=torch.empty(sizes[2], dtype=torch.uint8, device="cuda") if n >= sizes[2] > 0 else False)
        for accumulate in (False, True):
            want = torch.full((oc, k), 0.5, dtype=torch.float32, device="cuda")
            got = want.clone()
            B.qeft_weak_grad(d, dy, xw, want, accumulate=accumulate)
            dx, _ = B.qeft_linear_bwd(d, w, dy, xw, dW=got, accumulate=accumulate, ws=ws[:n])
            torch.cuda.synchronize()
            assert torch.equal(got, want), f"dW, {n} bytes"
            assert torch.equal(dx, want_dx), f"dX, {n} bytes"
            assert bool((ws[n:] == 171).all())
