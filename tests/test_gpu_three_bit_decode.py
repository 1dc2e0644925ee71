"""3-bit layers, both layouts, at 1 to 145 rows on their stored codes (no copy): rows at which the number of activation requests and
of 16-row tiles changes, a lane's 32 columns at every position within a ten-code word, channels that end inside a tile and inside a
quad of stores, ragged last groups, weak blocks of none and more than one step per wave, pitches beyond the 32-bit offsets, groups.
Tolerance: parity_util's bar; the weights are not rounded, so only the fp16 of the result is left (2.1e-4 in norm)."""
import numpy as np
import pytest
import torch

from oracle import qeft_oracle as qo
from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu

LAYERS = [(201, 1352, 264), (4106, 328, 8), (64, 1160, 0), (3, 136, 128), (16643, 320, 64), (520, 2688, 0)]


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("oc,ic,k", LAYERS)
def test_three_bit_rows(oc, ic, k, dense):
    layer = HostLayer(oc, ic, k, 3, 128, seed=oc + k, dense=dense)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    for m in (1, 2, 4, 5, 8, 9, 16, 17, 33, 48, 49, 145):
        x = synth.make_activations(m, ic, k, seed=m)
        xd, _ = pad_cols(x)
        ld = -(-oc // 8) * 8 + 8
        back = torch.full((m + 2, ld), 7.0, dtype=torch.float16, device="cuda")
        y = back[1:m + 1, :oc]
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=False)
        first = y.clone()
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=False)
        ref = xd.double() @ w64.t()
        torch.cuda.synchronize()
        assert torch.equal(first, y), f"M={m}: repeats differ"
        assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, oc:] == 7).all()), f"M={m}: wrote outside"
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"M={m}")


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("kq", [2048, 2560, 2568, 5120 + 640, 7680 + 384, 4 * 2560 + 72, 12288, 15360 - 8])
def test_three_bit_one_row_every_range_count(kq, dense):
    """One row of 1 to 6 kilobyte requests (ten codes a word: boundaries between groups inside lanes' pieces), rows that end early in one."""
    kq = kq // 32 * 32 if dense else kq        # (the dense kernel takes whole lane pieces)
    layer = HostLayer(77, kq + 72, 72, 3, 128, seed=kq, dense=dense)
    xd = pad_cols(synth.make_activations(1, layer.ic, 72, seed=kq))[0]
    y = B.qeft_linear_fwd(layer.desc, layer.to_device(), xd, ws=False)
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, xd.cpu().numpy()), f"{kq} columns")


@pytest.mark.parametrize("dense", [False, True])
def test_three_bit_rows_many_groups_per_wave(dense):
    """Ten-code words start at every shift as a wave's groups go by; both register sets of codes; all tile widths."""
    for oc, kq in ((2056, 25 * 128 + 64), (4104, 21 * 128), (8200, 13 * 128 + 96)):
        layer = HostLayer(oc, kq + 128, 128, 3, 128, seed=oc, dense=dense)
        w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
        for m in (2, 7, 16, 40, 96):
            xd = pad_cols(synth.make_activations(m, layer.ic, 128, seed=m))[0]
            y = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
            ref = xd.double() @ w64.t()
            torch.cuda.synchronize()
            assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"{oc} channels, M={m}")


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("m", [1, 3, 8, 40])
def test_three_bit_group(m, dense):
    layers = [HostLayer(oc, 640, 128, 3, 128, seed=oc, dense=dense) for oc in (264, 4096, 72)]
    xd, _ = pad_cols(synth.make_activations(m, 640, 128, seed=3))
    ys = B.qeft_linear_fwd_group([l.desc for l in layers], [l.to_device() for l in layers], xd)
    torch.cuda.synchronize()
    for l, y in zip(layers, ys):
        assert_close(y.cpu().numpy(), qo.linear_fwd(l.w64, xd.cpu().numpy()), f"{l.oc} channels")


@pytest.mark.parametrize("m", [2, 3])
def test_three_bit_rows_far_apart(m):
    """A pitch past the kernel's 32-bit offsets (2^24 elements): a row at a time."""
    layer = HostLayer(40, 264, 8, 3, 128, seed=1)
    w, pitch = layer.to_device(), (1 << 24) + 8
    x = synth.make_activations(m, 264, 8, seed=m)
    xd = torch.empty((m, pitch), dtype=torch.float16, device="cuda")[:, :264]
    xd.copy_(torch.from_numpy(x))
    y = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), "far rows")


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("m", [16, 48])
def test_three_bit_infinite_activations(m, dense):
    """Infinities as the sum itself treats them: x w where that is infinite, no number from inf x 0 and inf - inf."""
    layer = HostLayer(200, 1352, 72, 3, 128, seed=7, dense=dense)
    layer.codes[3, :] = 5
    layer.zeros[3, :] = 5                       # a whole row of zeros: inf x 0
    layer.qweight = (qo.pack_codes_dense3(layer.codes, layer.lay["row_stride_words"]) if dense
                     else qo.pack_codes(layer.codes, 3, layer.lay["row_stride_words"]))
    w = layer.to_device()
    x = synth.make_activations(m, 1352, 72, seed=m)
    inf = np.float16(np.inf)
    x[0, 5], x[3, 1351], x[m - 1, layer.kq - 1] = inf, -inf, inf
    x[7, [2, 300]] = inf, -inf
    x[11, 130] = np.nan
    with np.errstate(invalid="ignore"):
        want = np.stack([(row * layer.w64).sum(axis=1) for row in x.astype(np.float64)])
    y = B.qeft_linear_fwd(layer.desc, w, pad_cols(x)[0], ws=False)
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    fine = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fine) and np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.sign(got[np.isinf(want)]), np.sign(want[np.isinf(want)]))
    rows = fine.all(axis=1)
    assert_close(y.cpu().numpy()[rows], want[rows], "finite rows")
