"""The grid-search quantizer on values where its division-free scores and its skipped candidates could go wrong: quotients
exactly half way between codes, fp16 subnormals, one huge column among small ones, one-sided ranges.  As in the parity
tests the criterion is checked: parameters of a candidate of the grid, round-to-nearest codes under them, a float64 error
within 1e-5 of the minimum over the grid (128 fp32 terms: 128 x 2^-24 = 7.6e-6)."""
import numpy as np
import pytest
import torch

from oracle import qeft_oracle as qo
from paper_2410_08661_amd import binding as B
from parity_util import pad_cols

pytestmark = pytest.mark.gpu


def _values(kind, oc, ic):
    r = np.random.default_rng(17)
    if kind == "ties":        # multiples of half a step of many candidates
        return (r.integers(-15, 16, (oc, ic)) * 2.0 ** -6).astype(np.float16)
    if kind == "subnormal":
        return (r.integers(-700, 700, (oc, ic)) * 2.0 ** -24).astype(np.float16)
    if kind == "outlier":
        w = (r.standard_normal((oc, ic)) * 1e-3).astype(np.float16)
        w[:, ::61] = np.float16(2.0)
        return w
    return np.abs(r.standard_normal((oc, ic)) * 0.02).astype(np.float16)   # one-sided


@pytest.mark.parametrize("kind", ["ties", "subnormal", "outlier", "one-sided"])
@pytest.mark.parametrize("bits,g,k,n_grid,step", [(4, 128, 24, 80, 0.01), (4, 128, 0, 17, 0.05), (3, 64, 8, 33, 0.03)])
def test_search_criterion(kind, bits, g, k, n_grid, step):
    oc, ic = 37, 600 + k
    w = _values(kind, oc, ic)
    d = B.make_desc(oc, ic, k, bits, g)
    out = B.Weight(d)
    out.qweight.fill_(-1)
    B.qeft_pack_search(d, pad_cols(w)[1][:, :ic], n_grid, step, out)
    torch.cuda.synchronize()
    lay = qo.layout(oc, ic, k, bits, g)
    ng, kq = lay["n_groups"], lay["kq"]
    s, z = out.scales[:, :ng].cpu().numpy(), out.zeros[:, :ng].cpu().numpy()
    words = out.qweight.cpu().numpy().view(np.uint32)
    codes = qo.unpack_codes(words, kq, bits)
    assert np.array_equal(qo.pack_codes(codes, bits, lay["row_stride_words"]), words)     # padding zero
    s_all, z_all, e_all = qo.search_candidates(w, k, bits, g, n_grid, step)
    assert np.all(np.any((s_all.view(np.uint16) == s.view(np.uint16)[None]) & (z_all == z.astype(np.float32)[None]), axis=0))
    assert np.array_equal(codes, qo.codes_for_params(w, k, bits, g, s, z))
    wq = qo.dequantize(codes, s, z, np.zeros((oc, 0), dtype=np.float16), g)
    sq = (w[:, :kq].astype(np.float64) - wq) ** 2
    err = np.stack([sq[:, i * g:min((i + 1) * g, kq)].sum(axis=1) for i in range(ng)], axis=1)
    assert np.all(err <= e_all.min(axis=0) * (1 + 1e-5) + 1e-30)


@pytest.mark.parametrize("oc,kq,k,n_grid,step", [(37, 600, 24, 80, 0.01), (5, 1032, 13, 7, 0.1), (9, 2048, 0, 33, 0.03), (130, 8, 128, 16, 0.05)])
def test_dense_three_bit_words(oc, kq, k, n_grid, step):
    """The dense layout in groups of 128 is packed by the searching lanes, 3 words from 4 of them: rows that end inside those, padding,
    grids that are no whole rounds of 16, weak blocks copied by the same launch and (13 columns) by another."""
    ic = kq + k
    w = (np.random.default_rng(oc).standard_normal((oc, ic)) * 0.02).astype(np.float16)
    d = B.make_desc(oc, ic, k, 3, 128, B.QEFT_LAYOUT_DENSE3)
    out = B.Weight(d)
    for a in (out.qweight, out.scales, out.zeros):
        a.fill_(-1)
    B.qeft_pack_search(d, pad_cols(w)[1][:, :ic], n_grid, step, out)
    torch.cuda.synchronize()
    lay = qo.layout(oc, ic, k, 3, 128, dense=True)
    ng = lay["n_groups"]
    s, z = out.scales.cpu().numpy(), out.zeros.cpu().numpy()
    assert not s[:, ng:].any() and not z[:, ng:].any()
    s, z = s[:, :ng], z[:, :ng]
    codes = qo.codes_for_params(w, k, 3, 128, s, z)
    assert np.array_equal(qo.pack_codes_dense3(codes, lay["row_stride_words"]), out.qweight.cpu().numpy().view(np.uint32))
    s_all, z_all, e_all = qo.search_candidates(w, k, 3, 128, n_grid, step)
    assert np.all(np.any((s_all.view(np.uint16) == s.view(np.uint16)[None]) & (z_all == z.astype(np.float32)[None]), axis=0))
    wq = qo.dequantize(codes, s, z, np.zeros((oc, 0), dtype=np.float16), 128)
    sq = (w[:, :kq].astype(np.float64) - wq) ** 2
    err = np.stack([sq[:, i * 128:min((i + 1) * 128, kq)].sum(axis=1) for i in range(ng)], axis=1)
    assert np.all(err <= e_all.min(axis=0) * (1 + 1e-5) + 1e-30)
    if k:
        assert np.array_equal(out.weak.cpu().numpy(), w[:, kq:])


def _choice(w, bits, g, n_grid, step):
    """Scale and zero-point of the candidate with the least score, the first of equals, all in fp32: a
    lane's 8 columns left to right, square and sum in one rounding, then neighbouring lanes, pairs, quads and halves of the 16."""
    f32 = np.float32
    s_all, z_all, _ = qo.search_candidates(w, 0, bits, g, n_grid, step)
    oc, ng = s_all.shape[1:]
    v = np.zeros((oc, ng, 16, 8), dtype=f32)
    v.reshape(oc, ng, 128)[:, :, :g] = w.astype(f32).reshape(oc, ng, g)
    qmax = f32(2 ** bits - 1)
    scores = []
    for s16, z in zip(s_all, z_all):
        s, z = s16.astype(f32)[..., None, None], z.astype(f32)[..., None, None]
        d = v - s * np.clip(np.rint(v * (f32(1) / s)), -z, qmax - z)     # (s times a code is exact: one rounding)
        sq = d.astype(np.float64) ** 2
        a = sq[..., 0].astype(f32)
        for e in range(1, 8):
            a = (sq[..., e] + a).astype(f32)
        while a.shape[-1] > 1:
            a = a[..., 0::2] + a[..., 1::2]
        scores.append(a[..., 0])
    best = np.argmin(np.stack(scores), axis=0)[None]
    return np.take_along_axis(s_all, best, axis=0)[0], np.take_along_axis(z_all, best, axis=0)[0]


def _mirrored(oc, ng, g):
    """Every value with its negative, at random places: with a small step several candidates share a scale under zero-points whose
    errors are one another's mirror images, equal but for the order in which they are summed."""
    r = np.random.default_rng(5)
    h = (r.standard_normal((oc, ng, g // 2)) * 0.02).astype(np.float16)
    return r.permuted(np.concatenate([h, -h], axis=2), axis=2).reshape(oc, ng * g)


def _skewed(oc, ng, g, amp):
    """One-sided groups of a few units of the least subnormal, four alike in a row: the scales of narrow ranges are rounded by as
    much as they are large."""
    r = np.random.default_rng(7)
    u = np.rint(r.exponential(amp, (oc, ng // 4, 1, g)) * np.where(r.random((oc, ng // 4, 1, g)) < 0.1, -1, 1))
    return np.repeat((u * 2.0 ** -24).astype(np.float16), 4, axis=2).reshape(oc, ng * g)


@pytest.mark.parametrize("kind", ["mirrored", "skewed 1.5", "skewed 4"])
@pytest.mark.parametrize("bits,g,dense", [(4, 128, False), (3, 128, True), (3, 128, False), (4, 64, False)])
def test_search_choice(kind, bits, g, dense):
    """One candidate per group, the one that scores least over the whole grid, and codes, scale and zero-point all of it."""
    oc, ng = 256, 8
    n_grid, step = (33, 2.0 ** -12) if kind == "mirrored" else (80, 0.01)
    w = _mirrored(oc, ng, g) if kind == "mirrored" else _skewed(oc, ng, g, float(kind.split()[1]))
    d = B.make_desc(oc, ng * g, 0, bits, g, B.QEFT_LAYOUT_DENSE3 if dense else B.QEFT_LAYOUT_CANONICAL)
    out = B.Weight(d)
    B.qeft_pack_search(d, torch.from_numpy(w).cuda(), n_grid, step, out)
    torch.cuda.synchronize()
    lay = qo.layout(oc, ng * g, 0, bits, g, dense=dense)
    s, z = out.scales[:, :ng].cpu().numpy(), out.zeros[:, :ng].cpu().numpy()
    codes = qo.codes_for_params(w, 0, bits, g, s, z)
    packed = qo.pack_codes_dense3(codes, lay["row_stride_words"]) if dense else qo.pack_codes(codes, bits, lay["row_stride_words"])
    assert np.array_equal(packed, out.qweight.cpu().numpy().view(np.uint32))
    s_ref, z_ref = _choice(w, bits, g, n_grid, step)
    assert np.array_equal(s, s_ref) and np.array_equal(z.astype(np.float32), z_ref)


@pytest.mark.parametrize("bits,dense", [(4, False), (3, True)])
def test_divisions_by_short_numbers(bits, dense):
    """Scales, zero-points and codes come from quotients by numbers of 11 bits, corrected by their remainder instead of divided: the same
    bits as the division rules give over the whole range of scales (single candidate), and infinities end at the outermost codes."""
    r = np.random.default_rng(5)
    oc, ic = 64, 1024
    w = (r.standard_normal((oc, ic)) * 2.0 ** r.integers(-24, 14, (oc, 1))).clip(-65504, 65504).astype(np.float16)
    w[::3] = (r.integers(-15, 16, (len(w[::3]), ic)) * 2.0 ** r.integers(-24, 10, (len(w[::3]), 1))).astype(np.float16)
    w[5, 40], w[6, 50], w[7, 60] = np.inf, -np.inf, np.nan
    d = B.make_desc(oc, ic, 0, bits, 128, B.QEFT_LAYOUT_DENSE3 if dense else B.QEFT_LAYOUT_CANONICAL)
    out, ref = B.qeft_pack_search(d, pad_cols(w)[1][:, :ic], 1, 0.5), B.qeft_pack(d, pad_cols(w)[1][:, :ic])
    torch.cuda.synchronize()
    whole = [i for i in range(oc) if i not in (5, 6, 7)]
    assert torch.equal(out.scales[whole], ref.scales[whole]) and torch.equal(out.zeros[whole], ref.zeros[whole])
    assert torch.equal(out.qweight[whole], ref.qweight[whole])
    # a group with a value that is no finite number has scale 1 and zero-point 0
    assert bool((out.scales[5:8, 0] == 1).all()) and bool((out.zeros[5:8, 0] == 0).all())
    codes = B.qeft_unpack(d, out)[0].cpu()
    assert [int(codes[5, 40]), int(codes[6, 50]), int(codes[7, 60])] == [2 ** bits - 1, 0, 0]
