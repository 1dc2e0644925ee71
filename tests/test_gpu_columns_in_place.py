"""Gather and scatter of rows through a table, at the widths and rows where the kernels' shares change: whole values, so equality."""
import pytest
import torch

from paper_2410_08661_amd import binding as B

pytestmark = pytest.mark.gpu

WIDTHS = [8, 16, 1016, 1024, 1032, 2048, 2056, 4096, 4104, 8192, 8200]


def _table(ic, seed):
    return torch.randperm(ic, generator=torch.Generator().manual_seed(seed)).int().cuda()


@pytest.mark.parametrize("ic", WIDTHS)
def test_gathered_columns(ic):
    perm = _table(ic, ic)
    for m in (1, 3, 1025, 4099):
        back = torch.randn((m + 2, ic + 8), device="cuda").half()
        a = back[1:m + 1, :ic]
        assert torch.equal(B.qeft_reorder(a, perm, 1), a[:, perm.long()]), f"{m} rows"


@pytest.mark.parametrize("ic", [w for w in WIDTHS if w <= 8192])
def test_gathered_columns_by_a_table_on_four_bytes(ic):
    perm = torch.zeros(ic + 1, dtype=torch.int32, device="cuda")[1:]
    perm.copy_(_table(ic, ic))
    assert perm.data_ptr() % 8 == 4
    for m in (1, 1025, 4099):
        back = torch.randn((m + 2, ic + 8), device="cuda").half()
        a = back[1:m + 1, :ic]
        assert torch.equal(B.qeft_reorder(a, perm, 1), a[:, perm.long()]), f"{m} rows"


@pytest.mark.parametrize("ic", [w for w in WIDTHS if w >= 128] + [129, 1023, 1026, 2047, 2049, 4092, 4097, 8190, 8191, 8193])
def test_scattered_columns(ic):
    oc, k = 64, 8
    d = B.make_desc(oc, ic, k, 4, 128)
    w = B.qeft_pack(d, torch.randn((oc, (ic + 7) // 8 * 8), device="cuda").half()[:, :ic])
    perm = _table(ic, ic)
    for m in (3, 17, 1025, 4099):
        dy = torch.randn((m, oc), device="cuda").half()
        back = torch.full((m + 2, (ic + 7) // 8 * 8 + 8), 7.0, dtype=torch.float16, device="cuda")
        B.qeft_linear_bwd_dx_irregular(d, w, perm, dy, back[1:m + 1, :ic])
        want = torch.full_like(back, 7.0)
        want[1:m + 1, perm.long()] = B.qeft_linear_bwd_dx(d, w, dy, ws=False)
        assert torch.equal(back, want), f"{m} rows"
