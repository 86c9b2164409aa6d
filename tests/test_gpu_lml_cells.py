"""GPU parity of llc_lml_bound where cells of ln(q/p) decide (needs an MI355X): large masses that share cells, few
enough to be resolved one by one or so many that the row is sorted, and the shortest rows that go by cells.
Bound on the error: what cells leave open is at most 2^-23 of a result, sorted masses are rounded to fp32 (2^-24)."""
import numpy as np
import pytest
import torch

import paper_2506_05632_amd as llc
from oracle import lml
from test_gpu_lml_buckets import _left_to_sorting

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KS = [1, 4, 5, 9, 16]


def _check(draft, target, ws, kind="logits"):
    gpu = llc.llc_lml_bound(draft, target, KS, kind=kind, workspace=ws)
    torch.cuda.synchronize()
    ref = lml.lml_rows(draft.float().cpu().numpy(), target.float().cpu().numpy(), KS, kind=kind)
    for name in ("bound", "relaxed", "tv"):
        np.testing.assert_allclose(gpu[name].cpu().numpy(), ref[name], rtol=2.0 ** -22, err_msg=name)
    again = llc.llc_lml_bound(draft, target, KS, kind=kind, workspace=torch.zeros_like(ws))
    for name in ("bound", "relaxed", "tv"):
        assert torch.equal(again[name], gpu[name]), name


@pytest.mark.parametrize("heavy,left", [(2, False), (60, False), (250, True)])
@pytest.mark.parametrize("swap", [False, True])
def test_large_masses_that_share_cells(heavy, left, swap):
    # all of them are entries of the same two threads, which report one of them to the sample: the others lie between
    # splitters far apart
    g = torch.Generator(device=DEV).manual_seed(heavy)
    B, V = 3, 131072
    td = torch.randn(B, V, generator=g, device=DEV)
    tq = td + 0.01 * torch.randn(B, V, generator=g, device=DEV)
    at = (torch.arange(32, device=DEV)[:, None] * 4096 + torch.arange(8, device=DEV)).flatten()[:heavy]
    td[:, at] = 16.0 + 0.3 * torch.randn(B, heavy, generator=g, device=DEV)
    tq[:, at] = td[:, at] + 5.0 + torch.rand(B, heavy, generator=g, device=DEV)
    if swap:
        td, tq = tq, td
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    _check(td, tq, ws)
    assert _left_to_sorting(ws, B, V) == (list(range(B)) if left else [])


@pytest.mark.parametrize("V,dtype", [(6143, torch.float32), (6144, torch.float32), (6145, torch.float32),
                                     (8191, torch.bfloat16), (8192, torch.bfloat16), (8193, torch.bfloat16)])
@pytest.mark.parametrize("kind", ["logits", "probs"])
def test_the_shortest_rows(V, dtype, kind):
    g = torch.Generator(device=DEV).manual_seed(V)
    B = 6
    tq = 2.0 * torch.randn(B, V + 1, generator=g, device=DEV)[:, 1:]
    td = tq + torch.randn(B, V, generator=g, device=DEV)
    td[1] = tq[1]
    td[2, ::3], tq[2, 1::3] = float("-inf"), float("-inf")
    tq[3, 40:] = -1e9
    td[4, :], td[4, 7] = float("-inf"), 0.0      # one entry with mass
    if kind == "probs":
        td, tq = (torch.exp(t.double() - t.double().amax(dim=1, keepdim=True)).float() for t in (td, tq))
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    _check(td.to(dtype), tq.to(dtype), ws, kind)
