"""The forward GEMM's panels of 128 to 256 rows: row counts of every panel height in one and two panels, with a K split
(workspace) and without, weak blocks of whole stages, ragged and none.  Tolerance: parity_util's bar (fp16 weights, fp16
partial tiles under a split, fp16 results)."""
import pytest
import torch

from oracle import qeft_oracle as qo
from paper_2410_08661_amd import binding as B
from paper_2410_08661_amd import synth
from parity_util import HostLayer, assert_close, pad_cols

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("oc,ic,k,rows", [
    (520, 4096 + 64, 64, (100, 150, 180, 220, 256, 300, 333, 430)),    # split; direct weak stages
    (328, 4096 + 72, 72, (131, 192, 385, 512)),                        # split; ragged weak block
    (328, 4096 + 72, 72, (300, 333)),                                  # ... at 160 and 192 rows per panel
    (5384, 4096 + 72, 72, (100, 128, 150, 180)),                       # one panel (layers of few channels run the mid-row kernel there)
    (5384, 4096 + 64, 64, (97, 110)),
    (16648, 256, 0, (140, 333)),                                       # more tiles than a split is planned for
    (16648, 192 + 64, 64, (165, 222)),
])
def test_row_panels(oc, ic, k, rows):
    layer = HostLayer(oc, ic, k, 4, 128, seed=oc + k)
    w = layer.to_device()
    for m in rows:
        x = synth.make_activations(m, ic, k, seed=m)
        xd, _ = pad_cols(x)
        n = B.qeft_workspace_bytes(layer.desc, B.QEFT_OP_FWD, m)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else False
        back = torch.full((m + 1, oc + 8), 7.0, dtype=torch.float16, device="cuda")
        y = back[:m, :oc]
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=ws)
        first = y.clone()
        B.qeft_linear_fwd(layer.desc, w, xd, y, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(first, y), f"M={m}: repeats differ"
        assert bool((back[m] == 7).all()) and bool((back[:, oc:] == 7).all()), f"M={m}: wrote outside"
        assert_close(y.cpu().numpy(), qo.linear_fwd(layer.w64, x), f"M={m}")
