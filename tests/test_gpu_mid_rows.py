"""The forward between the decode sizes and the large GEMM (17 rows to a few hundred), at the edges of its tiles: rows around the
panels of 32 and 48, channels that end inside a tile of 16 ... 64, rows of fewer groups than waves, a ragged last group,
weak blocks of none, one and more than eight 32-column steps, a layer without quantized columns, and the group call.
Tolerance: parity_util's bar (2e-3 in norm and per element); this kernel does not round the weights, so only the fp16 of the
result is left (2.1e-4 in norm: half an ulp, 2^-12 at most per value, over a uniform mantissa)."""
import numpy as np
import pytest
import torch

from oracle import qeft_oracle as qo
from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu

LAYERS = [
    (200, 512, 128),            # three groups for eight waves; 200 channels: the last tile ends after 8 of 16
    (4104, 256 + 8, 8),         # 257 tiles of 16: wider ones, the last mostly empty
    (1032, 1352, 264),          # nine 32-column weak steps for eight waves; a ragged last group (1088 = 8 x 128 + 64)
    (264, 1160, 0),             # nothing weak; 9 x 128 + 8 columns
    (96, 320, 320),             # nothing quantized
    (16648, 384, 64),           # more tiles than CUs; three waves of one group each
    (520, 128 + 256, 256),      # one group: seven waves of eight have weak columns alone
    (8200, 256 + 264, 264),     # wider tiles, four waves for one pair and nine weak steps
]


@pytest.mark.parametrize("oc,ic,k", LAYERS)
def test_mid_rows(oc, ic, k):
    layer = HostLayer(oc, ic, k, 4, 128, seed=oc + k)
    w = layer.to_device()
    for m in (17, 32, 33, 48, 49, 96, 97, 145):
        x = synth.make_activations(m, ic, k, seed=m)
        xd, _ = pad_cols(x)
        back = torch.full((m + 2, oc + 8), 7.0, dtype=torch.float16, device="cuda")
        y = back[1:m + 1, :oc]
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=False)
        first = y.clone()
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=False)
        torch.cuda.synchronize()
        assert torch.equal(first, y), f"M={m}: repeats differ"
        assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, oc:] == 7).all()), f"M={m}: wrote outside"
        assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), f"M={m}")


@pytest.mark.parametrize("oc,kq", [
    (2056, 25 * 128 + 64),      # tiles of 32 channels, eight waves: four groups each or three, the last ragged
    (4104, 25 * 128 + 64),      # ... of 48
    (6152, 25 * 128 + 64),      # ... of 64
    (8200, 10 * 128 + 64),      # four waves: three groups each or two; tiles of 48
    (12296, 10 * 128 + 64),     # ... of 64; at 96 rows of 32, two waves
    (12296, 17 * 128 + 64),     # ... of 64; at 96 rows three waves, as many as LDS holds twice
    (16392, 5 * 128 + 64),      # ... of 64; at 96 rows two waves and tiles of 48
])
def test_mid_rows_many_groups_per_wave(oc, kq):
    """What one turn of a wave's loop fetches for the next: two and three 16-row tiles, every tile width."""
    layer = HostLayer(oc, kq + 128, 128, 4, 128, seed=oc)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    for m in (64, 96):
        x = synth.make_activations(m, layer.ic, 128, seed=m)
        xd = pad_cols(x)[0]
        y = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
        again = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
        ref = xd.double() @ w64.t()
        torch.cuda.synchronize()
        assert torch.equal(y, again), f"M={m}: repeats differ"
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"M={m}")


@pytest.mark.parametrize("bits,dense", [(3, False), (3, True)])
@pytest.mark.parametrize("oc,kq,k", [(520, 128, 256), (264, 200, 264), (8200, 256, 128), (1000, 64, 96)])
def test_few_groups_and_a_wide_weak_block_of_three_bit_layers(oc, kq, k, bits, dense):
    layer = HostLayer(oc, kq + k, k, bits, 128, seed=oc, dense=dense)
    w = layer.to_device()
    for m in (2, 7, 17, 48, 97):
        x = synth.make_activations(m, layer.ic, k, seed=m)
        y = B.qeft_linear_fwd(layer.desc, w, pad_cols(x)[0], ws=False)
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), f"M={m}")


@pytest.mark.parametrize("oc,kq,k", [(28680, 200, 128), (32768, 512, 64)])
def test_short_rows_of_more_workgroups_than_fit_in_twos(oc, kq, k):
    """One wave per workgroup of 32 channels."""
    layer = HostLayer(oc, kq + k, k, 4, 128, seed=oc)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    x = synth.make_activations(96, layer.ic, k, seed=3)
    xd = pad_cols(x)[0]
    y = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
    ref = xd.double() @ w64.t()
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"{oc} channels")


@pytest.mark.parametrize("m", [20, 40, 96])
def test_mid_rows_group_of_many_tiles(m):
    """More tiles than CUs over three layers: four waves, three groups each or two."""
    layers = [HostLayer(oc, 10 * 128 + 64 + 72, 72, 4, 128, seed=oc) for oc in (8200, 8264, 136)]
    ws = [l.to_device() for l in layers]
    x = synth.make_activations(m, layers[0].ic, 72, seed=4)
    xd, _ = pad_cols(x)
    ys = B.qeft_linear_fwd_group([l.desc for l in layers], ws, xd)
    for l, y in zip(layers, ys):
        ref = xd.double() @ torch.from_numpy(l.w64).cuda().t()
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"{l.oc} channels")


@pytest.mark.parametrize("m", [17, 40, 96])
def test_mid_rows_group(m):
    layers = [HostLayer(oc, 640, 128, 4, 128, seed=oc) for oc in (264, 4096, 72)]
    ws = [l.to_device() for l in layers]
    x = synth.make_activations(m, 640, 128, seed=3)
    xd, _ = pad_cols(x)
    ys = B.qeft_linear_fwd_group([l.desc for l in layers], ws, xd)
    torch.cuda.synchronize()
    for l, y in zip(layers, ys):
        assert_close(y.cpu().numpy(), qo.linear_fwd(l.w64, x), f"{l.oc} channels")


def test_mid_rows_fractional_zero_points():
    """Any fp16 zero-point: halves and values outside the code range."""
    layer = HostLayer(80, 768, 64, 4, 128, seed=5)
    rng = np.random.default_rng(9)
    layer.zeros = (rng.integers(-40, 60, layer.zeros.shape) / 2).astype(np.float16)
    w = layer.to_device()
    x = synth.make_activations(37, 768, 64, seed=6)
    y = B.qeft_linear_fwd(layer.desc, w, pad_cols(x)[0], ws=False)
    torch.cuda.synchronize()
    assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), "fractional zero-points")


@pytest.mark.parametrize("oc,ic,k", [(200, 512, 128), (1032, 1352, 264), (264, 1160, 0)])
def test_mid_rows_infinite_activations(oc, ic, k):
    """Infinities as the sum itself treats them: x w where that is infinite, no number from inf x 0 and inf - inf."""
    layer = HostLayer(oc, ic, k, 4, 128, seed=oc)
    layer.codes[3, :] = 5                       # a whole row of zeros: inf x 0
    layer.zeros[3, :] = 5
    layer.qweight = qo.pack_codes(layer.codes, 4, layer.lay["row_stride_words"])
    w = layer.to_device()
    for m in (17, 40, 96):
        x = synth.make_activations(m, ic, k, seed=m)
        inf = np.float16(np.inf)
        x[0, 5], x[3, ic - 1], x[m - 1, layer.kq - 1] = inf, -inf, inf
        x[7, [2, 300]] = inf, -inf
        x[11, 130] = np.nan
        with np.errstate(invalid="ignore"):
            want = np.stack([(row * layer.w64).sum(axis=1) for row in x.astype(np.float64)])
        y = B.qeft_linear_fwd(layer.desc, w, pad_cols(x)[0], ws=False)
        torch.cuda.synchronize()
        got = y.cpu().numpy().astype(np.float64)
        fine = np.isfinite(want)
        assert np.array_equal(np.isfinite(got), fine) and np.array_equal(np.isnan(got), np.isnan(want)), f"M={m}"
        assert np.array_equal(np.sign(got[np.isinf(want)]), np.sign(want[np.isinf(want)])), f"M={m}"
        rows = fine.all(axis=1)
        assert_close(y.cpu().numpy()[rows], want[rows], f"M={m}, finite rows")


def test_mid_rows_infinite_activations_of_long_rows():
    """The columns are looked through 1024 at a time: infinities in each part of a row, in its last group (64 columns) and beside
    the weak block's, alone and against each other; whole rows of them."""
    layer = HostLayer(520, 4256, 32, 4, 128, seed=11)
    layer.codes[3, :] = 5
    layer.zeros[3, :] = 5
    layer.qweight = qo.pack_codes(layer.codes, 4, layer.lay["row_stride_words"])
    w = layer.to_device()
    inf = np.float16(np.inf)
    for m in (17, 48, 96):
        x = synth.make_activations(m, layer.ic, 32, seed=m)
        for r, cols in enumerate(([0], [1023], [1024], [2047, 2048], [3071, 4222], [4160], [4223], [4224], [4255, 7], [4096, 4223])):
            x[r, cols] = inf
        x[9, 4223] = -inf
        x[10, [1, 4000]] = inf, np.nan
        x[11, :] = inf
        x[m - 1, 4100] = -inf
        with np.errstate(invalid="ignore"):
            want = np.stack([(row * layer.w64).sum(axis=1) for row in x.astype(np.float64)])
        y = B.qeft_linear_fwd(layer.desc, w, pad_cols(x)[0], ws=False)
        torch.cuda.synchronize()
        got = y.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isfinite(got), np.isfinite(want)) and np.array_equal(np.isnan(got), np.isnan(want)), f"M={m}"
        assert np.array_equal(np.sign(got[np.isinf(want)]), np.sign(want[np.isinf(want)])), f"M={m}"
        rows = np.isfinite(want).all(axis=1)
        assert_close(y.cpu().numpy()[rows], want[rows], f"M={m}, finite rows")


@pytest.mark.parametrize("m", [97, 144, 192])
def test_mid_rows_with_a_split_workspace(m):
    """Few channels: this kernel rather than the K split, so the same bits with the workspace as without."""
    layer = HostLayer(1032, 2056, 136, 4, 128, seed=m)
    w = layer.to_device()
    x = synth.make_activations(m, 2056, 136, seed=m)
    xd = pad_cols(x)[0]
    room = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_FWD, m)
    assert room > 0
    y = B.qeft_linear_fwd(layer.desc, w, xd, ws=torch.empty(room, dtype=torch.uint8, device="cuda"))
    plain = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
    torch.cuda.synchronize()
    assert torch.equal(y, plain)
    assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), f"M={m}")


@pytest.mark.parametrize("oc,groups,tail", [
    (200, 3, 0),        # one tile per workgroup, fewer pairs of groups than waves
    (1032, 34, 64),     # long rows, an odd number of groups, the last ragged
    (5128, 33, 0),      # tiles of 32 channels; the last pair is half one
    (8200, 34, 0),      # ... of 48
    (12296, 33, 8),     # ... of 64; at 33 rows and more seven waves
])
def test_few_rows_of_four_bits(oc, groups, tail):
    """2 to 16 rows where they take this kernel: one, two and four requests of rows, every tile width, guard rows around Y."""
    k = 72
    layer = HostLayer(oc, groups * 128 + tail + k, k, 4, 128, seed=oc)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    for m in (2, 3, 4, 5, 8, 9, 16, 40):
        xd = pad_cols(synth.make_activations(m, layer.ic, k, seed=m))[0]
        back = torch.full((m + 2, oc + 8), 7.0, dtype=torch.float16, device="cuda")
        y = back[1:m + 1, :oc]
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=False)
        first = y.clone()
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=False)
        ref = xd.double() @ w64.t()
        torch.cuda.synchronize()
        assert torch.equal(first, y), f"M={m}: repeats differ"
        assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, oc:] == 7).all()), f"M={m}: wrote outside"
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"M={m}")


@pytest.mark.parametrize("m", [2, 7, 16])
def test_few_rows_group(m):
    """Long rows of three layers in one launch, with and without a layer whose channels end inside an eight (other kernels)."""
    for ocs in ((264, 520, 72), (264, 515, 72)):
        layers = [HostLayer(oc, 33 * 128 + 40, 40, 4, 128, seed=oc) for oc in ocs]
        x = synth.make_activations(m, layers[0].ic, 40, seed=m)
        xd = pad_cols(x)[0]
        ys = B.qeft_linear_fwd_group([l.desc for l in layers], [l.to_device() for l in layers], xd)
        torch.cuda.synchronize()
        for l, y in zip(layers, ys):
            assert_close(y.cpu().numpy(), qo.linear_fwd(l.w64, x), f"{l.oc} channels")


@pytest.mark.parametrize("m", [193, 241, 433, 672])
@pytest.mark.parametrize("oc,ic,k", [(520, 512, 8), (1032, 2056, 136), (2048, 1352, 72)])
def test_hundreds_of_rows_of_small_layers(oc, ic, k, m):
    """Up to 14 panels of 48 rows: the same bits with a split's workspace as without, and every row at its place."""
    layer = HostLayer(oc, ic, k, 4, 128, seed=m)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    xd = pad_cols(synth.make_activations(m, ic, k, seed=m))[0]
    room = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_FWD, m)
    back = torch.full((m + 2, oc + 8), 7.0, dtype=torch.float16, device="cuda")
    y = back[1:m + 1, :oc]
    B.qeft_linear_fwd(layer.desc, w, xd, y, ws=torch.empty(room, dtype=torch.uint8, device="cuda") if room else False)
    plain = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
    ref = xd.double() @ w64.t()
    torch.cuda.synchronize()
    panels = -(-m // 48)
    if panels * -(-oc // 16) <= 5 * 256:
        assert torch.equal(y, plain)
    assert bool((back[0] == 7).all()) and bool((back[m + 1] == 7).all()) and bool((back[:, oc:] == 7).all())
    assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"M={m}")


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("oc,kq,k", [(72, 64 * 128, 8), (4096, 75 * 128 + 72, 72), (264, 64 * 128 - 8, 0)])
def test_few_rows_of_many_groups(oc, kq, k, bits):
    """Twelve waves, of which the last have a pair of groups less, one group of a pair or none in the last turn."""
    layer = HostLayer(oc, kq + k, k, bits, 128, seed=oc)
    w, w64 = layer.to_device(), torch.from_numpy(layer.w64).cuda()
    for m in (2, 4, 5, 8, 9):
        xd = pad_cols(synth.make_activations(m, layer.ic, k, seed=m))[0]
        y = B.qeft_linear_fwd(layer.desc, w, xd, ws=False)
        ref = xd.double() @ w64.t()
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), ref.cpu().numpy(), f"{oc} channels, M={m}")
