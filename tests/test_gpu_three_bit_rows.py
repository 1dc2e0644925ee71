"""3-bit layers of 17 rows and more with a workspace: the stored codes, or (forward from some hundred rows on, input gradient)
the codes rewritten in the 4-bit layout, then that layout's kernels.
Both 3-bit layouts; rows that end inside a word of either, weak blocks of 8 and 136, row counts of each kernel behind it,
workspaces of the stated size and of the fp16 copy alone.  Tolerance: parity_util's bar (fp16 weights, fp16 results)."""
import numpy as np
import pytest
import torch

from oracle import qeft_oracle as qo
from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("oc,ic,k", [(4096, 344, 8), (832, 1208 + 136, 136), (1024, 2048, 128), (16384, 72, 0), (128, 344, 8)])
def test_three_bit_rows(oc, ic, k, dense):
    h = HostLayer(oc, ic, k, 3, 128, seed=oc + ic, dense=dense)
    w = h.to_device()
    # 750 rows: the forward of layers from 2^20 weights on goes through a copy too.  Not with one group per row: weights rounded once to fp16,
    # all else in float64, already leave one of the 12 M outputs of 16384 x 72 3 % past the bar per element (a row of the largest scale).
    for m in (17, 96, 97, 300, 750) if ic > 128 else (17, 96, 97, 300):
        x, dy = synth.make_activations(m, ic, k, seed=m), synth.make_grad_output(m, oc, seed=m + 1)
        xd, dyd = pad_cols(x)[0], pad_cols(dy)[0]
        for op, call, ref in ((B.QEFT_OP_FWD, lambda ws: B.qeft_linear_fwd(h.desc, w, xd, ws=ws), qo.linear_fwd(h.w64, x)),
                              (B.QEFT_OP_BWD_DX, lambda ws: B.qeft_linear_bwd_dx(h.desc, w, dyd, ws=ws), qo.linear_bwd_dx(h.w64, dy))):
            n = B.qeft_workspace_bytes(h.desc, op, m)
            assert n >= 2 * oc * ic
            for size in {n, 2 * oc * ic}:
                back = torch.full((size + 64,), 0x5A, dtype=torch.uint8, device="cuda")
                out = call(back[:size])
                torch.cuda.synchronize()
                assert bool((back[size:] == 0x5A).all()), f"M={m}: wrote past the workspace"
                assert_close(out.cpu().numpy(), ref, f"op {op}, M={m}, workspace {size}")


# One rounding to fp16 is 2.1e-4 in norm over a uniform mantissa.  A call that keeps its sums in fp32 has two, independent of each
# other: the weights' and the result's, 2.9e-4; fp16 partial sums are a third, 3.6e-4; a fourth would make 4.2e-4.  The bounds
# lie half way.
TWO_ROUNDINGS, THREE_ROUNDINGS = 3.25e-4, 3.9e-4


def _error(out, ref):
    return float((out.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("dense", [False, True])
def test_sums_stay_in_fp32_without_room_for_a_split(dense):
    """The bytes of the fp16 copy alone: no fp16 partial tiles, also where they would fit behind the smaller copy."""
    oc = ic = 5120
    h = HostLayer(oc, ic, 128, 3, 128, seed=5, dense=dense)
    w, w64 = h.to_device(), torch.from_numpy(h.w64).cuda()
    for m in (40, 300, 1003):
        xd = torch.from_numpy(synth.make_activations(m, ic, 0, seed=m)).cuda()
        dyd = torch.from_numpy(synth.make_grad_output(m, oc, seed=m)).cuda()
        ws = torch.empty(2 * oc * ic, dtype=torch.uint8, device="cuda")
        for what, out, ref in (("forward", B.qeft_linear_fwd(h.desc, w, xd, ws=ws), xd.double() @ w64.t()),
                               ("dX", B.qeft_linear_bwd_dx(h.desc, w, dyd, ws=ws), dyd.double() @ w64)):
            err = _error(out, ref)
            assert err <= TWO_ROUNDINGS, f"{what}, M={m}: {err:.3e}"


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("oc,ic,k", [(5120, 5120, 128), (2048, 4096, 64), (5376, 4160, 64)])
def test_fractional_zero_points_are_rounded_once(oc, ic, k, dense):
    """Zero-points between 0 and 1: q - z is no fp16 number, and s (q - z) is still rounded once, in every kernel a row count
    leads to (panels of 128 to 256 rows, small tiles, both forms of the input gradient)."""
    h = HostLayer(oc, ic, k, 3, 128, seed=oc + k, dense=dense)
    h.zeros = np.random.default_rng(7).uniform(0.05, 0.95, h.zeros.shape).astype(np.float16)
    w, w64 = h.to_device(), torch.from_numpy(h.w64).cuda()
    for m in (40, 128, 200, 300, 333, 420, 1003, 1024):
        xd = torch.from_numpy(synth.make_activations(m, ic, 0, seed=m)).cuda()
        dyd = torch.from_numpy(synth.make_grad_output(m, oc, seed=m)).cuda()
        for what, op, call, ref in (("forward", B.QEFT_OP_FWD, lambda ws: B.qeft_linear_fwd(h.desc, w, xd, ws=ws), xd.double() @ w64.t()),
                                    ("dX", B.QEFT_OP_BWD_DX, lambda ws: B.qeft_linear_bwd_dx(h.desc, w, dyd, ws=ws), dyd.double() @ w64)):
            for size, bound in ((2 * oc * ic, TWO_ROUNDINGS), (B.qeft_workspace_bytes(h.desc, op, m), THREE_ROUNDINGS)):
                err = _error(call(torch.empty(size, dtype=torch.uint8, device="cuda")), ref)
                assert err <= bound, f"{what}, M={m}, workspace {size}: {err:.3e}"


@pytest.mark.gpu
@pytest.mark.parametrize("dense", [False, True])
def test_wide_layer_up_to_192_rows(dense):
    """97 to 192 rows of a wide layer: its stored codes, so the same bits with the copy's workspace as without."""
    k = 72
    layer = HostLayer(8200, 11 * 128 + k, k, 3, 128, seed=5, dense=dense)   # whole groups: dense rows that end inside one go through a copy
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    for m in (97, 144, 192):
        xd = pad_cols(synth.make_activations(m, layer.ic, k, seed=m))[0]
        room = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_FWD, m)
        y = B.qeft_linear_fwd(layer.desc, w, xd, ws=torch.empty(room, dtype=torch.uint8, device="cuda"))
        plain = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
        ref = xd.double() @ w64.t()
        torch.cuda.synchronize()
        assert torch.equal(y, plain), f"M={m}"
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"M={m}")


def test_more_workgroups_than_one_grid_counts():
    """Without a workspace any number of rows multiplies the stored codes: a product of rows and channels whose workgroups, counted in
    threads, pass 2^32 (103 GB of results) is still one call."""
    oc, ic, k, m = 51200, 7 * 128 + 8, 8, 1010000
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GB of device memory")
    h = HostLayer(oc, ic, k, 3, 128, seed=11)
    w = h.to_device()
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((m, ic), generator=gen, device="cuda", dtype=torch.float16)
    y = torch.empty((m, oc), dtype=torch.float16, device="cuda")
    looked = [0, 47, 48, 123456, 500000, m // 2 + 1, m - 49, m - 1]
    y[looked] = float("nan")
    B.qeft_linear_fwd(h.desc, w, x, y, ws=False)
    assert_close(y[looked].cpu().numpy(), qo.linear_fwd(h.w64, x[looked].cpu().numpy()), "rows of a large batch")
