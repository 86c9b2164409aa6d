"""Rows that would leave CUs half idle as one workgroup each, against the oracle and against one chunk a row, at the row counts and lengths
where one shape gives way to another (needs an MI355X).  Bar: indices and flags bit for bit (near-ties excused), keys to 1e-6."""
import pytest
import torch

import paper_2506_05632_amd as llc
from parity_util import compare, oracle_rows
from test_gpu_launch_shapes import _rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (rows, drafts, entries, own rows: with normalisers from 48 tiles of 1024 entries on, or 16, or 52; then without; shared proposals)
@pytest.mark.parametrize("B,K,V,own", [(257, 4, 48128, True), (257, 4, 48129, True), (341, 3, 49001, True), (342, 4, 30003, True), (384, 4, 30003, True),
                                       (385, 2, 9001, True), (512, 1, 9001, True), (513, 2, 9001, True), (128, 4, 122003, True), (129, 4, 122003, True),
                                       (192, 4, 121857, True), (256, 2, 121856, True), (260, 8, 30721, True), (258, 2, 121857, True),
                                       (257, 8, 121857, False), (341, 6, 121857, False), (342, 4, 121857, False), (342, 4, 16384, True),
                                       (340, 3, 16381, True), (140, 4, 53248, True), (200, 2, 53245, True), (258, 2, 102400, True), (300, 4, 102397, False)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_chunks_that_fill_the_chip(B, K, V, own, dtype):
    g = torch.Generator(device=DEV).manual_seed(B + K + V)
    target, draft = _rows(g, (B,), V, dtype), _rows(g, (B, K) if own else (B,), V, dtype)
    for keys in (False, True):
        kw = dict(temp_target=0.8, temp_draft=1.1, seed=5, want_keys=keys)
        gpu, one = llc.llc_couple(draft, target, K, **kw), llc.llc_couple(draft, target, K, v_chunks=1, **kw)
        torch.cuda.synchronize()
        for name in ("X", "Y", "accept", "match_k"):
            assert torch.equal(gpu[name], one[name]), name
        if keys:
            for name in ("keyX", "keyY"):
                assert torch.allclose(gpu[name], one[name], rtol=1e-6, atol=0.0), name
        for rows in ((0, 1), (B - 1, B)):
            ref = oracle_rows(draft, target, K, rows, kind="logits", temp_target=0.8, temp_draft=1.1, seed=5)
            compare(gpu, ref, rows=rows)


@pytest.mark.parametrize("B,K,V", [(300, 4, 3001), (512, 2, 5120), (257, 1, 2048), (140, 8, 4099)])
def test_short_own_rows_keep_workgroups_of_256_threads(B, K, V):
    # a normaliser's sum is taken in an order that goes with the threads: the same bits as one chunk of 256 (of 512 threads, some of the keys'
    # last bits are others)
    g = torch.Generator(device=DEV).manual_seed(V)
    target, draft = _rows(g, (B,), V, torch.bfloat16), _rows(g, (B, K), V, torch.bfloat16)
    kw = dict(seed=5, want_keys=True)
    out, one = llc.llc_couple(draft, target, K, **kw), llc.llc_couple(draft, target, K, v_chunks=1, **kw)
    for name in ("X", "Y", "accept", "match_k", "keyX", "keyY"):
        assert torch.equal(out[name], one[name]), name
