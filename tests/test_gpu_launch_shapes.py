"""The launch shapes that a batch's size selects (256, 512 or 1024 threads per workgroup, rows that are one
workgroup or several) against the oracle, at the sizes where one gives way to the next, on rows that start
on no 16-byte boundary (needs an MI355X).  Bar: indices and flags bit for bit (near-ties excused and
counted), keys to 1e-6."""
import pytest
import torch

import paper_2506_05632_amd as llc
from parity_util import compare, oracle_near_ties, oracle_rows, stats_dict

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rows(g, lead, V, dtype):
    """[*lead, V] with an odd row stride and an odd first element."""
    n = 1
    for d in lead:
        n *= d
    x = (2.0 * torch.randn(n, V + 3 - V % 2, generator=g, device=DEV)).to(dtype)
    return x[:, 1:V + 1].unflatten(0, lead)


# (rows, drafts, entries): one row of every split; the last row count of 1024 threads, of 512, and the
# next one; a row shorter than a workgroup, a last tile of one group, a tail of one entry
SHAPES = [(1, 4, 40001), (1, 8, 70003), (3, 2, 4093), (16, 5, 9001), (100, 4, 8197), (256, 4, 4097), (257, 4, 4097),
          (512, 3, 2051), (513, 3, 2051), (64, 16, 5003), (300, 8, 255), (256, 1, 1),
          # drafts in passes of six: one full, two with a padded last, three
          (40, 6, 5001), (33, 11, 4099), (7, 18, 2053)]


@pytest.mark.parametrize("B,K,V", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("min_first", [False, True])
def test_every_split_agrees_with_the_oracle(B, K, V, dtype, min_first):
    g = torch.Generator(device=DEV).manual_seed(B + 7 * K + V)
    target = _rows(g, (B,), V, dtype)
    stats = llc.new_stats(DEV)
    near = 0
    for n, draft in enumerate((_rows(g, (B,), V, dtype), _rows(g, (B, K), V, dtype))):
        for keys in (False, True):
            out = llc.llc_couple(draft, target, K, temp_target=0.8, temp_draft=1.1, seed=5 + n, row_offset=9, want_keys=keys,
                                 stats=stats, flags=llc.FLAG_MIN_FIRST if min_first else 0)
            torch.cuda.synchronize()
            ref = oracle_rows(draft, target, K, (0, B), kind="logits", temp_target=0.8, temp_draft=1.1, seed=5 + n,
                              row_offset=9, min_first=min_first)
            assert compare(out, ref) <= oracle_near_ties(ref)
            near += oracle_near_ties(ref)
    counted = stats_dict(stats)
    assert counted["near_ties"] == near and counted["degenerate"] == 0


def test_binned_selection_in_one_workgroup_and_in_several_agree():
    g = torch.Generator(device=DEV).manual_seed(3)
    B, L, N = 40, 3, 9001
    enc, dec = _rows(g, (B,), N, torch.float32), _rows(g, (B, L), N, torch.float32)
    bins = torch.randint(0, 5, (B, N + 1), generator=g, device=DEV, dtype=torch.uint8)[:, 1:]
    cand, side, source = (torch.randn(*s, generator=g, device=DEV) for s in ((B, N), (B, L), (B,)))
    kw = dict(seed=4, want_keys=True, cand=cand, side=side, source=source, var_w_given_a=0.3, var_t_given_a=0.5)
    outs = [llc.llc_compress_select(enc, dec, bins, v_chunks=c, **kw) for c in (0, 1, 4)]
    torch.cuda.synchronize()
    for out in outs[1:]:
        for name in out:
            if name.startswith("key"):
                torch.testing.assert_close(out[name], outs[0][name], rtol=1e-6, atol=0)
            else:
                assert torch.equal(out[name], outs[0][name]), name


@pytest.mark.parametrize("B,K,V,per_draft", [(2, 4, 70003, False), (300, 8, 9001, False), (600, 4, 4099, False), (40, 4, 9001, True)])
def test_rows_whose_bounds_leave_the_range_in_mid_scan(B, K, V, per_draft):
    # a logit far above the others that the warm-up has not seen: the wavefront that meets it sends the workgroup
    # to the exact form while the others are anywhere in the main loop, and the normalisers have to hold too
    g = torch.Generator(device=DEV).manual_seed(V)
    target = _rows(g, (B,), V, torch.float32).clone()
    draft = _rows(g, (B, K) if per_draft else (B,), V, torch.float32).clone()
    target[::2, V - 1] = 3000.0
    target[1::3, V // 2] = 2500.0
    draft[::3, ..., V - 2] = 2800.0
    draft[1::4, ..., 2 * V // 3] = 1500.0
    stats = llc.new_stats(DEV)
    out = llc.llc_couple(draft, target, K, temp_target=0.8, temp_draft=1.1, seed=5, want_keys=True, stats=stats)
    torch.cuda.synchronize()
    ref = oracle_rows(draft, target, K, (0, B), kind="logits", temp_target=0.8, temp_draft=1.1, seed=5)
    assert compare(out, ref) <= oracle_near_ties(ref)
    assert stats_dict(stats)["slow_blocks"] > 0


@pytest.mark.parametrize("K", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("V", [1024, 1025, 2048, 3077])  # exactly the first tile, one entry more, two, a ragged third
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tiles_in_which_every_lane_has_candidates(K, V, dtype):
    # entries far above those of the first tile, which the warm-up looks at: whole wavefronts meet them at once
    B = 5
    g = torch.Generator(device=DEV).manual_seed(K + V)
    target, shared, own = (_rows(g, lead, V, dtype).clone() for lead in ((B,), (B,), (B, K)))
    for t in (target, shared, own):
        t[..., 1024:1024 + 700] += 9.0
    for draft in (shared, own):
        for keys in (False, True):
            out = llc.llc_couple(draft, target, K, temp_target=0.8, temp_draft=1.1, seed=5, want_keys=keys, v_chunks=1)
            torch.cuda.synchronize()
            ref = oracle_rows(draft, target, K, (0, B), kind="logits", temp_target=0.8, temp_draft=1.1, seed=5)
            assert compare(out, ref) <= oracle_near_ties(ref)
