"""Few rows, whose chunks are as fine as the chip has room for, against the oracle at the sizes where one shape gives way to
another (needs an MI355X).  Bar: indices and flags bit for bit (near-ties excused), keys to 1e-6."""
import pytest
import torch

import paper_2506_05632_amd as llc
from parity_util import compare, oracle_rows
from test_gpu_launch_shapes import _rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (rows x entries: tiles of 2048 entries eleven and twelve, one more entry; sixteen and more of them; rows up to and beyond 32; an odd
# number of tiles of 4096 for the shapes of many drafts)
@pytest.mark.parametrize("B,K,V", [(2, 4, 22528), (2, 4, 22529), (1, 2, 24576), (3, 3, 32768), (3, 4, 32769), (31, 4, 23001), (32, 1, 23001),
                                   (33, 4, 23001), (5, 4, 40003), (2, 8, 18001), (2, 6, 45057), (16, 7, 28673)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_chunks_of_few_rows(B, K, V, dtype):
    g = torch.Generator(device=DEV).manual_seed(B + K + V)
    target = _rows(g, (B,), V, dtype)
    for n, draft in enumerate((_rows(g, (B,), V, dtype), _rows(g, (B, K), V, dtype))):
        for keys in (False, True):
            gpu = llc.llc_couple(draft, target, K, temp_target=0.8, temp_draft=1.1, seed=5 + n, want_keys=keys)
            torch.cuda.synchronize()
            ref = oracle_rows(draft, target, K, (0, B), kind="logits", temp_target=0.8, temp_draft=1.1, seed=5 + n)
            compare(gpu, ref)


@pytest.mark.parametrize("B,K,V", [(1, 4, 4095), (1, 4, 4097), (7, 4, 6145), (42, 3, 12289), (43, 3, 12289), (64, 2, 6001), (20, 4, 24001), (3, 8, 50001)])
def test_chunks_of_few_rows_of_drafts_alone(B, K, V):
    g = torch.Generator(device=DEV).manual_seed(B + K + V)
    for draft in (_rows(g, (B,), V, torch.bfloat16), _rows(g, (B, K), V, torch.bfloat16)):
        gpu = llc.llc_couple(draft, None, K, temp_draft=0.9, seed=9, row_offset=77, flags=llc.FLAG_DRAFT_ONLY)
        torch.cuda.synchronize()
        ref = oracle_rows(draft, draft if draft.dim() == 2 else draft[:, 0], K, (0, B), kind="logits", temp_target=1.0, temp_draft=0.9, seed=9,
                          row_offset=77)
        got = gpu["X"].cpu().numpy()
        assert ((got == ref["X"]) | (ref["gapX"] < 1e-6)).all()


def test_a_workspace_that_holds_fewer_chunks_gets_those():
    g = torch.Generator(device=DEV).manual_seed(1)
    target, draft = _rows(g, (3,), 32001, torch.float32), _rows(g, (3,), 32001, torch.float32)
    ref = llc.llc_couple(draft, target, 4, seed=3)
    for size in (3328, 4096, 1 << 20):
        out = llc.llc_couple(draft, target, 4, seed=3, workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
        for name in ("X", "Y", "accept", "match_k"):
            assert torch.equal(out[name], ref[name]), (size, name)


@pytest.mark.parametrize("B,K,V,own", [(4, 1, 4097, False), (4, 4, 8192, False), (60, 3, 6145, False), (1, 2, 12288, False), (4, 1, 4097, True), (16, 2, 8192, True)])
def test_drafts_alone_in_short_rows_are_one_workgroup_each(B, K, V, own):
    # (it keeps its results to itself: nothing passes through the workspace)
    draft = torch.randn(*((B, K, V) if own else (B, V)), device=DEV)
    ws = torch.full((llc.llc_couple_workspace_size(B, K, V),), 0xA5, dtype=torch.uint8, device=DEV)
    llc.llc_couple(draft, None, K, seed=9, flags=llc.FLAG_DRAFT_ONLY, workspace=ws)
    assert (ws == 0xA5).all()


@pytest.mark.parametrize("with_pool", [False, True])
def test_long_rows_are_cut_into_chunks_of_large_workgroups(with_pool):
    # 30 rows of 100 003 entries: chunks of four tiles of 1024 threads (of 512 threads they would be seven tiles, 14 336 entries)
    B, V, chunk, n = 30, 100003, 4 * 4096, 7
    draft, target = torch.randn(B, V, device=DEV), torch.randn(B, V, device=DEV)
    ws = torch.zeros(llc.llc_couple_workspace_size(B, 1, V), dtype=torch.uint8, device=DEV)
    llc.llc_couple(draft, target if with_pool else None, 1, seed=9, flags=0 if with_pool else llc.FLAG_DRAFT_ONLY, workspace=ws)
    keys = (B * n * 8 + 255) // 256 * 256
    winners = ws[keys:keys + B * n * 4].view(torch.int32).view(B, n)
    assert (winners // chunk == torch.arange(n, device=DEV)).all()
