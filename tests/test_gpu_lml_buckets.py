"""GPU parity of llc_lml_bound on rows long enough to go by cells of ln(q/p), which a sample shares out (needs an
MI355X).

Same oracle and same bound on the error as in test_gpu_lml.py: what cells leave open, or the order among
ratios that agree to fp32 precision and masses rounded to fp32, everything else is fp64 on both sides; rtol
1e-6."""
import numpy as np
import pytest
import torch

import paper_2506_05632_amd as llc
from oracle import lml
from test_gpu_lml import KS, check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (the ends of the range of either type, a walk's 4096 entries and one more, ragged tails, the first length with a
# second attempt; test_gpu_lml_cells.py has the ends more closely)
@pytest.mark.parametrize("V", [6143, 6144, 8191, 8192, 8193, 16384, 16385, 40961, 65536, 70003])
@pytest.mark.parametrize("kind", ["logits", "logw", "probs"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_lengths_kinds_and_types(V, kind, dtype):
    g = torch.Generator(device=DEV).manual_seed(V)
    B = 5
    tq = 2.0 * torch.randn(B, V + 1, generator=g, device=DEV)[:, 1:] + 30.0   # (odd strides, far from zero)
    td = tq + torch.randn(B, V, generator=g, device=DEV)
    td[1, V // 2:] = tq[1, V // 2:]          # half a row of equal logits
    td[2] = tq[2]                            # equal distributions up to the temperatures
    td[3, : V // 3] = float("-inf")          # no mass on one side, and on both
    tq[3, V // 4: V // 2] = float("-inf")
    td[4] = 8.0 * td[4]                      # widely spread ratios
    if kind == "probs":
        td, tq = (torch.exp(t.double() - t.double().amax(dim=1, keepdim=True)).float() for t in (td, tq))
    td, tq = td.to(dtype), tq.to(dtype)
    temp = 1.0 if V % 2 else 0.9
    check(td, tq, KS if V % 3 else KS[:2], kind=kind, temp_draft=temp, temp_target=1.0)


def _sampled(V):
    """The positions of the half of the kernel's sample that is spread over a row."""
    j = np.arange(1024, dtype=np.uint64)
    jitter = (j * np.uint64(0x9E3779B9)) & np.uint64(0xFFFFFFFF)
    return ((j * np.uint64(V) + ((jitter * np.uint64(V)) >> np.uint64(32))) >> np.uint64(10)).astype(np.int64)


def _pair_of(V):
    """Which two of the kernel's threads meet an entry; the other half of the sample is the largest entry of every pair."""
    return torch.arange(V, device=DEV) // 8 % 512


def test_a_row_whose_sample_misleads_is_sorted():
    # everywhere but at the sample's positions the ratios lie within 2e-5 of each other, beside all that the sample
    # holds, so one cell takes most of the row: no entry leaves as much as 1e-9 of a result open, all together some
    # 4e-6; the rows beside it are ordinary
    g = torch.Generator(device=DEV).manual_seed(1)
    B, V = 4, 20011
    tq = torch.randn(B, V, generator=g, device=DEV)
    td = tq + torch.randn(B, V, generator=g, device=DEV)
    crowd = torch.full((V,), 0.1, device=DEV) + 2e-5 * torch.rand(V, generator=g, device=DEV)
    # the draft's largest of every pair of threads, and the target's, all of which are as large: the pair's first entry
    at = torch.cat([torch.from_numpy(_sampled(V)).to(DEV), 8 * torch.arange(512, device=DEV)])
    crowd[at] = 0.2 + torch.randn(at.numel(), generator=g, device=DEV).abs()
    tq[2] = 0.0
    td[2] = crowd
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    check(td, tq, [1, 4], workspace=ws)
    assert _left_to_sorting(ws, B, V) == [2]


def test_results_do_not_depend_on_the_workspace_or_the_run():
    g = torch.Generator(device=DEV).manual_seed(2)
    B, V = 9, 33001
    tq = (2.0 * torch.randn(B, V, generator=g, device=DEV)).bfloat16().float()   # many ties
    td = (tq + torch.randn(B, V, generator=g, device=DEV)).bfloat16().float()
    first = llc.llc_lml_bound(td, tq, KS)
    for rows in (1, 4, 9, 9):
        ws = torch.randint(0, 255, (24 * V * rows + 256,), dtype=torch.uint8, device=DEV)
        other = llc.llc_lml_bound(td, tq, KS, workspace=ws)
        torch.cuda.synchronize()
        for name in ("bound", "relaxed", "tv"):
            assert torch.equal(other[name], first[name]), (rows, name)


def _keep(x, kept, low, g):
    """x with all but `kept` random entries of every row at `low`."""
    at = torch.rand(x.shape, generator=g, device=DEV).argsort(dim=1)[:, :kept]
    return torch.full_like(x, low).scatter(1, at, x.gather(1, at))


@pytest.mark.parametrize("V,dtype", [(32000, torch.float32), (50001, torch.bfloat16)])
@pytest.mark.parametrize("temp_draft,temp_target", [(0.7, 0.7), (0.7, 1.0), (1.0, 0.01), (0.02, 1.0)])
def test_rows_masked_by_a_finite_value_and_very_sharp_rows(V, dtype, temp_draft, temp_target):
    # most of a row far away in ln r from the entries that have mass, on either side or both, and the
    # temperatures alone doing the same: the order among the entries with mass decides the bound
    g = torch.Generator(device=DEV).manual_seed(V)
    target, draft = [], []
    for low in (-1e4, -1e9, torch.finfo(dtype).min):
        for kept in (3, 50, 2000, 10000):
            q = -1.1 * torch.log(torch.rand(4, V, generator=g, device=DEV).argsort(dim=1) + 1.0)
            q += 0.5 * torch.randn(4, V, generator=g, device=DEV)
            p = q + torch.randn(4, V, generator=g, device=DEV)
            same = torch.rand(1, V, generator=g, device=DEV).argsort(dim=1)[:, kept:]  # one mask for both
            q[0] = _keep(q[:1], kept, low, g)[0]
            p[1] = _keep(p[1:2], kept, low, g)[0]
            q[2, same[0]] = low
            p[2, same[0]] = low                                                        # (row 3 stays whole)
            target.append(q)
            draft.append(p)
    target, draft = torch.cat(target).to(dtype), torch.cat(draft).to(dtype)
    gpu, _ = check(draft, target, KS if temp_target == 1.0 else KS[:3], temp_draft=temp_draft, temp_target=temp_target)
    assert (gpu["bound"] <= 1 + 1e-9).all()


@pytest.mark.parametrize("V", [6144, 12288, 40961])
@pytest.mark.parametrize("kind,temp", [("logw", 1.0), ("logits", 0.7)])
def test_masses_of_every_size_down_to_nothing(V, kind, temp):
    # ln of either mass sweeps from 0 to -800, side by side and against each other, so that products and sums
    # of two masses pass through the smallest normal numbers
    g = torch.Generator(device=DEV).manual_seed(V)
    sweep = -800.0 * torch.arange(V, device=DEV) / V
    rows = [(sweep, sweep - 0.5), (sweep, sweep + 0.01 * torch.randn(V, generator=g, device=DEV)),
            (sweep, sweep + 20.0 * torch.randn(V, generator=g, device=DEV)), (sweep, sweep.flip(0)),
            (sweep, 0.5 * sweep), (2.0 * sweep, sweep)]
    rows += [(q, p) for p, q in rows]
    draft, target = (temp * torch.stack(side) for side in zip(*rows))
    gpu, ref = check(draft, target, KS, kind=kind, temp_draft=temp, temp_target=temp)
    assert torch.isfinite(gpu["relaxed"]).all()
    # two sides that share next to nothing: the relaxed sum is e^-380 or so, and still has its digits
    draft, target = torch.full((2, 1, V), -380.0 * temp, device=DEV)
    draft, target = draft.clone(), target.clone()
    draft[0, 3], draft[0, 5], target[0, 3], target[0, 5] = 0.0, -float("inf"), -float("inf"), 0.0
    gpu = llc.llc_lml_bound(draft, target, KS, kind=kind, temp_draft=temp, temp_target=temp)
    ref = lml.lml_rows(draft.cpu().numpy(), target.cpu().numpy(), KS, kind=kind, temp_draft=temp, temp_target=temp)
    np.testing.assert_allclose(gpu["relaxed"].cpu().numpy(), ref["relaxed"], rtol=1e-6)


def test_splitters_farther_apart_than_an_int():
    # nearly all of the sample has ln r = -400 or 400 and next to no mass, and no quantile falls between the two (1038
    # entries, 64 quantiles, 16.2 entries apart: one is at the 503rd, the next at the 519th), where all that counts
    # lies: some 270 entries of seven pairs of threads, of which the sample holds 14, at 14 ratios 0.5 apart.  Cells are 800 /
    # 1792 wide there, so each ratio has one; the entries of a single cell would be too many to resolve.
    g = torch.Generator(device=DEV).manual_seed(3)
    V = 20011
    td, tq = torch.full((2, V), float("-inf"), device=DEV), torch.full((2, V), float("-inf"), device=DEV)
    pair = _pair_of(V)
    heavy = pair < 7
    td[:, heavy] = torch.round(64.0 * torch.randn(2, int(heavy.sum()), generator=g, device=DEV)) / 64.0
    tq[:, heavy] = td[:, heavy] + (pair - 3.0 + 0.5 * (torch.arange(V, device=DEV) & 1))[heavy]
    at = torch.from_numpy(_sampled(V)).to(DEV)
    at = at[torch.randperm(1024, generator=g, device=DEV)]
    left, right = at[:504], at[504:]
    td[:, left], tq[:, left] = -60.0, -460.0
    td[:, right], tq[:, right] = -460.0, -60.0
    ws = torch.zeros(24 * V * 2 + 256, dtype=torch.uint8, device=DEV)
    for draft, target in ((td, tq), (tq, td)):
        check(draft, target, [1, 4], workspace=ws)
        assert _left_to_sorting(ws, 2, V) == []


# (not probabilities 1e-7 apart: in fp32 most of those are the same, and the order among equal ratios is free,
# which the sorted masses' rounding makes worth up to 2^-23 of a pair's share)
@pytest.mark.parametrize("kind,width", [("logits", 1e-6), ("logits", 1e-7), ("probs", 1e-6)])
def test_ratios_close_to_each_other_are_told_apart(kind, width):
    # ratios within a few 1e-7 of each other, whose order fp32 still tells, in both forms: 6143 entries are sorted, 6145 go
    # by cells (the two more carry no mass).  Sorted masses are rounded to fp32.  A cell between splitters is some
    # 1e-10 wide, and what is beyond the sample, a hundredth of the row on either side, is at most one cell of the whole
    # width, which leaves 0.25 x 5e-6 x 1e-4 of a result open: 2e-10 (entries not told apart at all: 0.25 x 5e-6).
    g = torch.Generator(device=DEV).manual_seed(5)
    B, V = 8, 6143
    tq = -1.1 * torch.log(torch.rand(B, V, generator=g, device=DEV, dtype=torch.float64).argsort(dim=1) + 1.0)
    if kind == "probs":
        tq = torch.exp(tq).float()
        td = (tq.double() * torch.exp(width * torch.randn(B, V, generator=g, device=DEV, dtype=torch.float64))).float()
    else:
        tq = (0.01 * tq).float()   # (so that fp32 logits can lie this close)
        td = (tq.double() + width * torch.randn(B, V, generator=g, device=DEV, dtype=torch.float64)).float()
    ref = lml.lml_rows(td.cpu().numpy(), tq.cpu().numpy(), [1, 4], kind=kind)["bound"]
    by_sorting = llc.llc_lml_bound(td, tq, [1, 4], kind=kind)["bound"]
    np.testing.assert_allclose(by_sorting.cpu().numpy(), ref, rtol=2.0 ** -22)
    none = torch.full((B, 2), 0.0 if kind == "probs" else float("-inf"), device=DEV)
    ws = torch.zeros(24 * (V + 2) * B + 256, dtype=torch.uint8, device=DEV)
    by_cells = llc.llc_lml_bound(torch.cat([td, none], 1), torch.cat([tq, none], 1), [1, 4], kind=kind, workspace=ws)["bound"]
    assert _left_to_sorting(ws, B, V + 2) == []
    np.testing.assert_allclose(by_cells.cpu().numpy(), ref, rtol=2e-9)


def _left_to_sorting(ws, B, V):
    """Which rows the cell kernel left to the sorting one: those have that kernel's second buffer of masses
    where the other writes a 0, behind 16 V bytes of the row's part of the workspace."""
    return [b for b in range(B) if ws[24 * V * b + 16 * V:24 * V * b + 16 * V + 4].view(torch.int32).item() != 0]


@pytest.mark.parametrize("V,dtype", [(160000, torch.float32), (160001, torch.float32), (1 << 18, torch.float32), (1 << 18, torch.bfloat16)])
def test_ordinary_rows_up_to_the_longest_go_by_cells(V, dtype):
    g = torch.Generator(device=DEV).manual_seed(4)
    B = 48
    tq = -1.1 * torch.log(torch.rand(B, V, generator=g, device=DEV).argsort(dim=1) + 1.0)
    td = (tq + 0.5 * torch.randn(B, V, generator=g, device=DEV)).to(dtype)
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    tq = (tq + 0.5 * torch.randn(B, V, generator=g, device=DEV)).to(dtype)
    check(td, tq, [1, 4], rows=[0, 17, B - 1], temp_draft=0.7, temp_target=0.7, workspace=ws)
    assert _left_to_sorting(ws, B, V) == []
    # one more entry is one too many for the form
    if V == 1 << 18:
        more = [torch.cat([x[:2], torch.full((2, 1), float("-inf"), device=DEV, dtype=dtype)], 1) for x in (td, tq)]
        check(*more, [1, 4], temp_draft=0.7, temp_target=0.7)


@pytest.mark.parametrize("kind,dtype", [("logits", torch.float32), ("probs", torch.float32), ("logits", torch.bfloat16)])
def test_rows_of_ratios_shared_by_a_hundred_entries_go_by_cells(kind, dtype):
    # 1200 ratios: the sample holds most of them once, twice or three times, so quantiles fall inside such runs
    g = torch.Generator(device=DEV).manual_seed(6)
    B, V = 6, 128256
    tq = torch.randint(-300, 300, (B, V), generator=g, device=DEV) / 64.0
    td = tq + torch.randint(0, 1200, (B, V), generator=g, device=DEV) / (256.0 if dtype == torch.float32 else 64.0)
    if kind == "probs":
        td, tq = 2.0 ** td.double().round(), (2.0 ** tq.double().round())
        td = td * (1.0 + torch.randint(0, 100, (B, V), generator=g, device=DEV) / 128.0)
    ws = torch.zeros(24 * V * B + 256, dtype=torch.uint8, device=DEV)
    check(td.to(dtype), tq.to(dtype), [1, 4], kind=kind, workspace=ws)
    assert _left_to_sorting(ws, B, V) == []


@pytest.mark.parametrize("V,dtype", [(12288, torch.float32), (20011, torch.float32), (70003, torch.float32), (41011, torch.bfloat16)])
def test_cells_of_hundreds_of_entries(V, dtype):
    # entries that share a cell by the hundred: a crowd beside ratios far from it, at several distances, and values
    # of few bits
    g = torch.Generator(device=DEV).manual_seed(V)
    B = 6
    tq = torch.randn(B, V, generator=g, device=DEV)
    at = torch.rand(B, V, generator=g, device=DEV)
    near, far = torch.randn(B, V, generator=g, device=DEV), 9.0 * torch.randn(B, V, generator=g, device=DEV)
    td = tq + torch.where(at < 0.5, 1e-4 * near, far)
    td[1] = tq[1] + torch.where(at[1] < 0.9, 1e-6 * near[1], far[1])
    td[2] = tq[2] + far[2].sign() * torch.exp(far[2].abs()).clamp(max=60.0)       # tails
    td[3], tq[3] = (4.0 * near[3]).bfloat16().float(), tq[3].bfloat16().float()
    td[4] = tq[4] + 0.37 * torch.floor(40.0 * at[4] ** 3)
    td, tq = td.to(dtype), tq.to(dtype)
    first, _ = check(td, tq, KS, temp_draft=0.9)
    again = llc.llc_lml_bound(td, tq, KS, temp_draft=0.9, workspace=torch.ones(24 * V + 256, dtype=torch.uint8, device=DEV))
    for name in ("bound", "relaxed", "tv"):
        assert torch.equal(again[name], first[name]), name
