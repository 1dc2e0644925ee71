"""Perf-informational: the host-side choices between kernels, on shapes OFF the Llama-2 grid.

The choices are made from row counts and time models fitted to the Llama-2 shapes: which forward kernel serves the rows between the
decode sizes and the large GEMM, whether the contraction of some or all tiles is split over the optional workspace, which copy of
a 3-bit layer is multiplied, how many ways the weak gradient splits its tokens.  These tests time the library's
choice and an alternative that the boundary lets a caller force (calls on 16-row slices; the call without the workspace; the
product of an fp16 copy; a wider weak block) with HIP events and require the choice to be at most 10 % slower than that alternative.
No numerics here (the parity tests cover every path); a failure means a heuristic needs refitting, not a wrong
result.  Timings on a shared machine wobble, so a miss is measured a second time, and only a miss of more than 25 %
fails the test; one between 10 % and 25 % is reported as an expected-failure note with the figures.  The file is named
to be collected after the parity tests: a run that stops at the first failure has then compared every result first.
"""
import pytest
import torch

from paper_2410_08661_amd import binding as B

pytestmark = pytest.mark.gpu

SLACK, HARD = 1.10, 1.25


def _judge(measure, what):
    """measure() -> (library's time, alternative's time); informational between SLACK and HARD, failing beyond."""
    t_lib, t_alt = measure()
    if t_lib > SLACK * t_alt:
        t_lib, t_alt = measure()          # once more before believing it
    print(f"\n{what}: library {t_lib:.1f} us, alternative {t_alt:.1f} us")
    assert t_lib <= HARD * t_alt, f"{what}: {t_lib:.1f} us against {t_alt:.1f} us"
    if t_lib > SLACK * t_alt:
        pytest.xfail(f"{what}: {t_lib:.1f} us against {t_alt:.1f} us (more than 10 % slower than the alternative)")


def _layer(oc, ic, k, seed, bits=4):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d = B.make_desc(oc, ic, k, bits, 128)
    w = B.Weight(d)
    w.qweight.random_(-2**31, 2**31 - 1, generator=gen)
    w.scales.copy_((torch.rand(w.scales.shape, generator=gen, device="cuda") * 0.008 + 0.004).half())
    w.zeros.copy_(torch.randint(0, 2 ** bits, w.zeros.shape, generator=gen, device="cuda").half())
    w.weak.copy_((torch.randn(w.weak.shape, generator=gen, device="cuda") * 0.02).half())
    return d, w, gen


def _us(fn, n=20, repeats=3):
    """Best of `repeats` event timings of n back-to-back calls, in microseconds per call."""
    for _ in range(3):
        fn()
    best = float("inf")
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            fn()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3 / n)
    return best


@pytest.mark.parametrize("oc,ic", [(6144, 6144), (2560, 7168)])
@pytest.mark.parametrize("m", [48, 96, 320])
def test_passes_or_gemm_without_workspace(oc, ic, m):
    d, w, gen = _layer(oc, ic, 128, oc + m)
    x = torch.randn((m, ic), generator=gen, device="cuda").half()
    y = torch.empty((m, oc), dtype=torch.float16, device="cuda")
    def passes():
        for r in range(0, m, 16):
            B.qeft_linear_fwd(d, w, x[r:r + 16], y[r:r + 16], ws=False)
    _judge(lambda: (_us(lambda: B.qeft_linear_fwd(d, w, x, y, ws=False)), _us(passes)),
           f"forward {oc}x{ic} M={m} without workspace against {(m + 15) // 16} passes of 16 rows")


@pytest.mark.parametrize("oc,ic,m", [(6144, 6144, 48), (6144, 6144, 320), (6144, 6144, 2816), (2560, 7168, 320), (7168, 2560, 1536)])
def test_workspace_never_costs_more_than_ten_percent(oc, ic, m):
    """With the optional workspace the library may split tiles (all of them when they are few, the last round's when
    it is sparse); a caller who passes one must not lose by it."""
    d, w, gen = _layer(oc, ic, 128, oc + ic + m)
    x = torch.randn((m, ic), generator=gen, device="cuda").half()
    dy = (torch.randn((m, oc), generator=gen, device="cuda") * 0.01).half()
    y = torch.empty((m, oc), dtype=torch.float16, device="cuda")
    dx = torch.empty((m, ic), dtype=torch.float16, device="cuda")
    for name, op, call in (("forward", B.QEFT_OP_FWD, lambda ws: B.qeft_linear_fwd(d, w, x, y, ws=ws)),
                           ("dX", B.QEFT_OP_BWD_DX, lambda ws: B.qeft_linear_bwd_dx(d, w, dy, dx, ws=ws))):
        n = B.qeft_workspace_bytes(d, op, m)
        if n == 0:
            continue                     # no split planned for this launch: both calls are the same
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        _judge(lambda: (_us(lambda: call(ws)), _us(lambda: call(False))), f"{name} {oc}x{ic} M={m} with the workspace against without")


def _group_call(ocs, ic, m):
    layers = [_layer(oc, ic, 128, oc + i) for i, oc in enumerate(ocs)]
    x = torch.randn((m, ic), generator=layers[0][2], device="cuda").half()
    ys = [torch.empty((m, oc), dtype=torch.float16, device="cuda") for oc in ocs]
    group = B.Group([d for d, _, _ in layers], [w for _, w, _ in layers], ys)
    return lambda: B.qeft_linear_fwd_group(None, None, x, group=group)


def _single_call(oc, ic, m):
    d, w, gen = _layer(oc, ic, 128, oc)
    x = torch.randn((m, ic), generator=gen, device="cuda").half()
    y = torch.empty((m, oc), dtype=torch.float16, device="cuda")
    return lambda: B.qeft_linear_fwd(d, w, x, y, ws=False)


@pytest.mark.parametrize("oc,ic,m", [(7680, 8192, 97), (7680, 8192, 128), (12288, 640, 144), (16384, 1408, 144)])
def test_layer_no_slower_than_its_halves_in_one_call(oc, ic, m):
    single, halves = _single_call(oc, ic, m), _group_call((oc // 2, oc // 2), ic, m)
    _judge(lambda: (_us(single), _us(halves)), f"forward {oc}x{ic} M={m} without workspace against a group of its halves")


@pytest.mark.parametrize("oc", [512, 4096])
def test_short_row_no_slower_than_a_longer_one(oc):
    """A wide weak block is divided among a workgroup's waves however few groups stand before it: with two groups no slower than with
    six.  (Calls of 5 us: replayed from a graph.)"""
    def replayed(ic):
        d, w, gen = _layer(oc, ic, 256, oc + ic)
        x = torch.randn((48, ic), generator=gen, device="cuda").half()
        y = torch.empty((48, oc), dtype=torch.float16, device="cuda")
        graph = torch.cuda.CUDAGraph()
        B.qeft_linear_fwd(d, w, x, y, ws=False)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            for _ in range(50):
                B.qeft_linear_fwd(d, w, x, y, ws=False)
        return lambda: graph.replay(), (graph, w, x, y)
    short, _keep = replayed(512)
    long, _keep2 = replayed(1024)
    for attempt in range(2):
        t_short, t_long = _us(short, n=5) / 50, _us(long, n=5) / 50
        if t_short <= 1.02 * t_long:
            return
    pytest.fail(f"forward of {oc} channels, M=48, 256 weak columns: two groups {t_short:.2f} us, six {t_long:.2f} us")


@pytest.mark.parametrize("ocs,ic", [((8192, 1024, 1024), 8192), ((7168, 7168), 7168)])
def test_group_of_fewer_rows_no_slower(ocs, ic):
    """Three panels of 48 rows hold 97 rows and 144."""
    few, more = _group_call(ocs, ic, 97), _group_call(ocs, ic, 144)
    _judge(lambda: (_us(few), _us(more)), f"group {ocs} x {ic} M=97 against M=144")


@pytest.mark.parametrize("oc,ic,k,m", [(8192, 8192, 64, 2048), (4096, 4096, 64, 1003), (11008, 4096, 8, 512), (13824, 5120, 16, 1003)])
def test_three_bit_rows_no_slower_than_an_fp16_copy(oc, ic, k, m):
    """3-bit layers whose last group is partial: the call with its workspace against the dense product that the boundary offers
    (a layer whose columns are all weak, with its workspace) after one pass that writes those fp16 weights."""
    d, w, gen = _layer(oc, ic, k, oc + m, bits=3)
    dense, wd, _ = _layer(oc, ic, ic, 1)
    src = wd.weak.clone()
    x = torch.randn((m, ic), generator=gen, device="cuda").half()
    dy = (torch.randn((m, oc), generator=gen, device="cuda") * 0.01).half()
    y = torch.empty((m, oc), dtype=torch.float16, device="cuda")
    dx = torch.empty((m, ic), dtype=torch.float16, device="cuda")
    for name, op, call in (("forward", B.QEFT_OP_FWD, lambda d, w, ws: B.qeft_linear_fwd(d, w, x, y, ws=ws)),
                           ("dX", B.QEFT_OP_BWD_DX, lambda d, w, ws: B.qeft_linear_bwd_dx(d, w, dy, dx, ws=ws))):
        ws = torch.empty(B.qeft_workspace_bytes(d, op, m), dtype=torch.uint8, device="cuda")
        n = B.qeft_workspace_bytes(dense, op, m)
        wsd = torch.empty(n, dtype=torch.uint8, device="cuda") if n else False
        def through_copy():
            wd.weak.copy_(src)
            call(dense, wd, wsd)
        _judge(lambda: (_us(lambda: call(d, w, ws)), _us(through_copy)), f"3-bit {name} {oc}x{ic} k={k} M={m} against the product of an fp16 copy")


@pytest.mark.parametrize("oc,k,m", [(13824, 64, 3000), (13824, 16, 2048), (4096, 96, 777)])
def test_weak_gradient_of_a_narrow_block(oc, k, m):
    """How the tokens are split: a weak block narrower than 128 reads the same gradients as one of 128 and forms fewer products
    (its partly filled strips cost a stage more than full ones, which leaves it up to 1.2 times as long)."""
    gen = torch.Generator(device="cuda").manual_seed(k)
    dy = (torch.randn((m, oc), generator=gen, device="cuda") * 0.01).half()
    x = torch.randn((m, 1024), generator=gen, device="cuda").half()
    def run(k):
        d = B.make_desc(oc, 1024, k)
        dw = torch.empty((oc, k), dtype=torch.float32, device="cuda")
        n = B.qeft_workspace_bytes(d, B.QEFT_OP_WEAK_GRAD, m)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
        return lambda: B.qeft_weak_grad(d, dy, x[:, 1024 - k:], dw, ws=ws)
    narrow, full = run(k), run(128)
    for attempt in range(2):
        t, t_full = _us(narrow), _us(full)
        if t <= 1.3 * t_full:
            return
    pytest.fail(f"weak gradient {oc} channels, M={m}: k={k} {t:.1f} us, k=128 {t_full:.1f} us")


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_row_that_is_not_finite_costs_no_more_than_a_few_calls(value):
    """One such activation, late in one row of 40: outputs that are no number are taken again, which must stay small beside the call."""
    d, w, gen = _layer(4096, 11008, 128, 3)
    x = torch.randn((40, 11008), generator=gen, device="cuda").half()
    y = torch.empty((40, 4096), dtype=torch.float16, device="cuda")
    t = _us(lambda: B.qeft_linear_fwd(d, w, x, y, ws=False))
    x[7, 10800] = value
    t_bad = _us(lambda: B.qeft_linear_fwd(d, w, x, y, ws=False))
    print(f"\nfinite {t:.1f} us, one value {value}: {t_bad:.1f} us")
    assert t_bad <= 3 * t
