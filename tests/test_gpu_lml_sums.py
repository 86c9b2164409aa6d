"""GPU parity of llc_lml_bound's form by cells' sums where it can go wrong (needs an MI355X): references that do not serve, heavy
entries that share threads, cells shared out again, any number of list sizes, rows that it has to leave to the other forms.
Bound on the error: cells leave at most 0.75 x 2^-23 of a result open, in rows of 131 072 entries or more 0.75 x 2^-22, the other forms 2^-22; tv and the
relaxed sums are 64-bit sums."""
import numpy as np
import pytest
import torch

import paper_2506_05632_amd as llc
from oracle import lml
from test_gpu_lml_buckets import _left_to_sorting

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(draft, target, ks, kind="logits", rtol=2.0 ** -22, **kw):
    B, V = draft.shape
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    gpu = llc.llc_lml_bound(draft, target, ks, kind=kind, workspace=ws, **kw)
    torch.cuda.synchronize()
    ref = lml.lml_rows(draft.float().cpu().numpy(), target.float().cpu().numpy(), ks, kind=kind, **kw)
    np.testing.assert_allclose(gpu["bound"].cpu().numpy(), ref["bound"], rtol=rtol, err_msg="bound")
    for name in ("relaxed", "tv"):
        np.testing.assert_allclose(gpu[name].cpu().numpy(), ref[name], rtol=1e-12, atol=1e-15, err_msg=name)
    again = llc.llc_lml_bound(draft, target, ks, kind=kind, workspace=torch.ones_like(ws), **kw)
    for name in ("bound", "relaxed", "tv"):
        assert torch.equal(again[name], gpu[name]), name
    return ws


def _by_cells(ws, B, V):
    """Rows that the form behind did, in a workspace of B slots that held zeros: it writes the entries' cells there, the form by sums nothing."""
    return ws[:24 * V * B].view(B, 24 * V)[:, :2 * V].amax(dim=1).nonzero().flatten().tolist()


def _rows(B, V, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    tq = -1.1 * torch.log(torch.rand(B, V, generator=g, device=DEV).argsort(dim=1) + 1.0)
    tq += 0.5 * torch.randn(B, V, generator=g, device=DEV)
    return tq + 0.5 * torch.randn(B, V, generator=g, device=DEV), tq, g


@pytest.mark.parametrize("V", [6144, 8191, 8192, 8193, 12287, 32003, 65537])
@pytest.mark.parametrize("ks", [[3], [1, 2], [7, 1, 2], [1, 2, 4, 8], [5, 4, 3, 2, 1], [1, 2, 3, 4, 5, 6, 7, 65535]])
def test_any_number_of_list_sizes(V, ks):
    # (by sums: an ordinary row's cells leave some 1e-8 open, of which the tenth part is missed at most; by sorting masses are
    # rounded to fp32)
    draft, target, _ = _rows(3, V, V)
    ws = _check(draft, target, ks, rtol=5e-9, temp_draft=0.7, temp_target=0.9)
    assert _by_cells(ws, 3, V) == []
    ws = _check(draft.bfloat16(), target.bfloat16(), ks, rtol=5e-9 if V >= 8192 else 2.0 ** -22)
    assert _by_cells(ws, 3, V) == []


@pytest.mark.parametrize("first", [float("-inf"), float("nan"), -1e4, -1e9, -3e38, 90.0])
def test_the_first_entries_are_no_measure_of_the_others(first):
    # masses are summed relative to the largest of the first 64 entries, then to the row's largest if that overflows
    draft, target, _ = _rows(4, 20000, 1)
    draft[0, :64] = first
    target[1, :64] = first
    draft[2, :5000], target[2, :64] = first, first
    ws = _check(draft + 1000.0, target, [1, 4])
    # (90: all of the draft's mass is on entries that the target has next to none of)
    assert _by_cells(ws, 4, 20000) == ([0] if first == 90.0 else [])


def test_rows_that_are_left_to_the_other_forms():
    draft, target, _ = _rows(6, 9001, 2)
    draft[0, 7], target[1, 8999] = float("inf"), float("inf")   # carry no mass
    draft[2, 1:] = float("-inf")                                # one entry
    draft[3, :9000], target[3, 9000] = float("-inf"), float("-inf")  # disjoint: 0
    draft[4, ::2] -= 45.0                                       # sides that share little, where rounding may count
    target[4, 1::2] -= 45.0
    ws = torch.zeros(24 * 9001 * 6 + 256, dtype=torch.uint8, device=DEV)
    gpu = llc.llc_lml_bound(draft, target, [1, 16], workspace=ws)
    ref = lml.lml_rows(draft.cpu().numpy(), target.cpu().numpy(), [1, 16])
    for name in ("bound", "relaxed", "tv"):
        np.testing.assert_allclose(gpu[name].cpu().numpy(), ref[name], rtol=2.0 ** -22, atol=1e-30, err_msg=name)
    assert (gpu["bound"][3] == 0.0).all()
    assert _by_cells(ws, 6, 9001) == [0, 1, 3, 4]               # (a row of one entry has one cell, for which nothing is open)
    draft[2] = float("-inf")                                    # no mass on a side
    gpu = llc.llc_lml_bound(draft[2:3], target[2:3], [1, 16])
    assert (gpu["bound"] == 0.0).all() and (gpu["relaxed"] == 0.0).all()


@pytest.mark.parametrize("V,dtype", [(20000, torch.float32), (128256, torch.float32), (70001, torch.bfloat16)])
@pytest.mark.parametrize("heavy", [1, 8, 64, 300])
def test_heavy_entries_of_the_same_threads(V, dtype, heavy):
    # half of either side's mass on `heavy` entries that four threads meet, close to each other in ln r and among the light
    # ones, so that most of them have no cell of their own
    draft, target, g = _rows(4, V, heavy)
    at = (torch.arange(64, device=DEV)[:, None] * 4096 + torch.arange(16, device=DEV)).flatten()
    at = at[at < V][:heavy]
    heavy = at.numel()
    top = torch.logsumexp(target, dim=1, keepdim=True) - np.log(heavy)
    target[:, at] = top + 0.3 * torch.randn(4, heavy, generator=g, device=DEV)
    draft[:, at] = target[:, at] + 0.05 * torch.randn(4, heavy, generator=g, device=DEV)
    _check(draft.to(dtype), target.to(dtype), [1, 8])
    _check(target.to(dtype), draft.to(dtype), [1, 8])


@pytest.mark.parametrize("V", [65536, 200003, 1 << 18])
@pytest.mark.parametrize("kind", ["logits", "probs"])
def test_cells_are_shared_out_again(V, kind):
    # many entries of middling mass over a wide range: most rows leave more open than they may before that
    g = torch.Generator(device=DEV).manual_seed(V)
    wide, flat = 4.0 * torch.randn(4, V, generator=g, device=DEV), 0.1 * torch.randn(4, V, generator=g, device=DEV)
    if kind == "probs":
        wide, flat = torch.exp(wide), torch.exp(flat)
    for draft, target in ((wide, flat), (flat, wide)):
        ws = _check(draft, target, [1, 8], kind)
        assert _left_to_sorting(ws, 4, V) == []
        assert len(_by_cells(ws, 4, V)) <= 1


@pytest.mark.parametrize("ratios", [1, 5, 40, 130, 300])
@pytest.mark.parametrize("V", [8192, 40001])
def test_ratios_shared_by_many_entries(ratios, V):
    # whole cells of one ratio, which have one cell each or up to eight (sums are exact but for the masses' rounding), beside
    # entries spread between them
    g = torch.Generator(device=DEV).manual_seed(ratios)
    tq = torch.randn(3, V, generator=g, device=DEV)
    td = tq + 0.125 * torch.randint(-ratios // 2, ratios - ratios // 2, (3, V), generator=g, device=DEV)
    td[1, ::3] += 0.01 * torch.randn(td[1, ::3].numel(), generator=g, device=DEV)
    td[2, :40] = tq[2, :40] + 3.0   # heavy ones among them
    tq[2, :40] += 8.0
    _check(td, tq, [1, 4])
    _check(td.bfloat16(), tq.bfloat16(), [1, 4])


@pytest.mark.parametrize("V,heavy,light,spread", [(50257, 300, 7e-10, "flat"), (128256, 3000, 1e-10, "flat"), (128256, 3000, 7e-10, "normal"),
                                                  (262136, 3000, 1e-5, "normal"), (262136, 300, 7e-10, "flat")])
@pytest.mark.parametrize("kind", ["logits", "probs"])
def test_sides_that_share_light_entries_only(V, heavy, light, spread, kind):
    # either side's mass is on entries that the other has none of; the rest differ by up to e^20 or so
    g = torch.Generator(device=DEV).manual_seed(7)
    s = 20.0 * (torch.randn(2, V, generator=g, device=DEV) if spread == "normal" else 2.0 * torch.rand(2, V, generator=g, device=DEV) - 1.0)
    draft, target = np.log(light) - s.clamp(min=0.0), np.log(light) + s.clamp(max=0.0)
    at = torch.rand(2, V, generator=g, device=DEV).argsort(dim=1)
    for mine, other, where in ((draft, target, at[:, :heavy]), (target, draft, at[:, heavy:2 * heavy])):
        mine.scatter_(1, where, -np.log(heavy))
        other.scatter_(1, where, float("-inf"))
    if kind == "probs":
        draft, target = draft.exp(), target.exp()
    _check(draft, target, [1, 4, 64, 4096], kind)
    _check(target, draft, [1, 4, 64, 4096], kind)


@pytest.mark.parametrize("low", [-1e9, -1e10, -1e30, None])
@pytest.mark.parametrize("temp", [0.6, 0.7, 0.8, 0.9, 1.0, 1.2])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_masked_at_their_beginning_are_like_others(low, temp, dtype):
    # the first entries are as far below the others as the type allows (None: its lowest), on either side or both
    low = torch.finfo(dtype).min if low is None else low
    draft, target, _ = _rows(4, 10001, 3)
    draft[0, :64] = low
    target[1, :64] = low
    draft[2, :6000], target[2, :6000] = low, low
    ws = _check(draft.to(dtype), target.to(dtype), [1, 4], temp_draft=temp, temp_target=temp)
    assert _by_cells(ws, 4, 10001) == []
