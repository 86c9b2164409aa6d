"""GPU parity of llc_lml_bound where cells of ln(q/p) decide (needs an MI355X): large masses that share cells, few
enough to be resolved one by one or so many that the row is sorted, and the shortest rows that go by cells.
Bound on the error: what cells leave open is at most 1.5 x 2^-23 of a result, sorted masses are rounded to fp32 (2^-24)."""
import numpy as np
import pytest
import torch

import paper_2506_05632_amd as llc
from oracle import lml
from test_gpu_lml_buckets import _left_to_sorting

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KS = [1, 4, 5, 9, 16]


def _check(draft, target, ws, kind="logits", ks=KS):
    gpu = llc.llc_lml_bound(draft, target, ks, kind=kind, workspace=ws)
    torch.cuda.synchronize()
    ref = lml.lml_rows(draft.float().cpu().numpy(), target.float().cpu().numpy(), ks, kind=kind)
    for name in ("bound", "relaxed", "tv"):
        np.testing.assert_allclose(gpu[name].cpu().numpy(), ref[name], rtol=2.0 ** -22, err_msg=name)
    again = llc.llc_lml_bound(draft, target, ks, kind=kind, workspace=torch.zeros_like(ws))
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


def _uncertain_row(V, width, mass, g, heavy=200):
    """Half of the entries have next to no mass and lie far to the right in ln(q/p); between them and the others, `heavy`
    entries of a few threads (so that the sample holds few of them) with one ratio and together `mass` of the
    draft's and half of the target's, and at 0.5 `width` on either side of it in ln(q/p) one of them each: one cell whose order
    is not known, and in which the entries do not lie evenly."""
    p = torch.randn(V, generator=g, device=DEV, dtype=torch.float64)
    q = p + torch.randn(V, generator=g, device=DEV, dtype=torch.float64)
    far = torch.rand(V, generator=g, device=DEV) < 0.5
    p[far] -= 70.0
    q[far] -= 40.0
    at = (torch.arange(13, device=DEV)[:, None] * 4096 + torch.arange((heavy + 12) // 13, device=DEV)).flatten()[:heavy]
    p_ln, q_ln = torch.log(p.exp().sum() * mass / heavy), torch.log(q.exp().sum() / heavy)
    p[at] = p_ln
    q[at] = q_ln + 1e-6 * torch.randn(heavy, generator=g, device=DEV, dtype=torch.float64)
    q[at[0]] += 0.5 * width
    q[at[1]] -= 0.5 * width
    return p.float(), q.float()


@pytest.mark.parametrize("ks", [[1, 4, 8, 16, 64], [64, 1], [1024, 64, 16, 8, 4, 2, 1], [1 << 20]])
@pytest.mark.parametrize("swap", [False, True])
def test_what_cells_leave_open_is_bounded_for_every_list_size(ks, swap):
    # an error of a denominator counts up to K times as much for the sum of K as for that of 1, so rows that are certain
    # enough for one list size are not for another, in whatever order they are asked for
    g = torch.Generator(device=DEV).manual_seed(9)
    V = 131072
    rows = [_uncertain_row(V, width, mass, g) for width in (0.005, 0.02, 0.05) for mass in (0.0005, 0.002, 0.005)]
    draft, target = (torch.stack(side) for side in zip(*rows))
    if swap:
        draft, target = target, draft
    _check(draft, target, torch.zeros(24 * V * len(rows) + 256, dtype=torch.uint8, device=DEV), ks=ks)


def test_masses_that_cells_do_not_see():
    # all that the two sides share has less than 2^-46 of either row's largest: the cells' sums are 0 there
    g = torch.Generator(device=DEV).manual_seed(10)
    B, V = 3, 40000
    draft = -40.0 + torch.randn(B, V, generator=g, device=DEV)
    target = -40.0 + torch.randn(B, V, generator=g, device=DEV)
    draft[:, 5], target[:, 5] = 0.0, -90.0
    draft[:, 9], target[:, 9] = -90.0, 0.0
    draft[1, 100:200], target[1, 100:200] = -0.5, -85.0
    target[2, 300:900] = -20.0
    _check(draft, target, torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV), ks=[1, 16, 1000])


@pytest.mark.parametrize("V", [60000, 131072])
def test_a_row_uncertain_in_no_one_entry_is_sorted(V):
    # (416 masses of one ratio, which a second attempt on the longer row cannot tell from the two beside them either)
    g = torch.Generator(device=DEV).manual_seed(9)
    draft, target = (x[None] for x in _uncertain_row(V, 0.03, 0.002, g, 416))
    ws = torch.zeros(24 * V + 256, dtype=torch.uint8, device=DEV)
    _check(draft, target, ws, ks=[1, 2, 4, 8])
    assert _left_to_sorting(ws, 1, V) == [0]


@pytest.mark.parametrize("V", [65535, 65536, 128256, 152064, 200003, 1 << 18])
@pytest.mark.parametrize("kind,dtype", [("logits", torch.float32), ("probs", torch.float32), ("logits", torch.bfloat16)])
def test_wide_rows_are_not_sorted(V, kind, dtype):
    # one side flat and the other spread over many e-folds, or two slopes: many entries of middling mass, dozens to a cell
    g = torch.Generator(device=DEV).manual_seed(V)
    B = 6
    wide, flat = 3.0 * torch.randn(B, V, generator=g, device=DEV), torch.zeros(B, V, device=DEV)
    wide[4:], flat[4:] = torch.linspace(-30, 0, V, device=DEV), torch.linspace(-25, 0, V, device=DEV)
    wide[5] += 1e-3 * torch.randn(V, generator=g, device=DEV)
    if kind == "probs":
        wide, flat = torch.exp(wide), torch.exp(flat)
    wide, flat = wide.to(dtype), flat.to(dtype)
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    for draft, target in ((wide, flat), (flat, wide)):
        _check(draft, target, ws, kind, ks=[1, 8])
        assert _left_to_sorting(ws, B, V) == []
