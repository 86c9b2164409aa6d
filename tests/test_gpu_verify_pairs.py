"""llc_verify's strong form where every row is scanned for all drafts at once (needs an MI355X): few sequences, against the CPU
oracle and against the loop over positions, which a call that asks for counters takes.  Tokens, counts and viability are the same; keys are
normalised by sums of fp32 terms in another order (2^-22 relative is what those sums are held to)."""
import numpy as np
import pytest
import torch

import paper_2506_05632_amd as llc
from parity_util import stats_dict
from test_gpu_verify import compare_verify, oracle_verify

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _tokens(target, S, L, K, V, g, keep=0.7, **kw):
    """Draft tokens of which `keep` are what the loop emits there, so that drafts drop out one after the other."""
    tok = torch.randint(0, V, (S, L, K), generator=g, dtype=torch.int32)
    copy = torch.rand(S, L, K, generator=g) < keep
    for _ in range(L):
        y = torch.from_numpy(oracle_verify(target, tok, (0, S), strong=True, **kw)["Y"][:, :L].copy()).to(torch.int32)
        tok = torch.where(copy & (y[:, :, None] >= 0), y[:, :, None].expand(S, L, K), tok)
    return tok.to(DEV)


def _both(target, tok, size=None, flags=0, **kw):
    """The call as the library takes it, the loop over positions, and whether the first was another form: the two forms leave different
    things in the workspace (of `size` bytes; by default one that holds whatever either needs), the loop with and without counters
    but for a runner-up's key per row and draft."""
    S, L1, K, V = target.shape
    if size is None:
        size = max(llc.llc_verify_workspace_size(S, L1 - 1, K, V), llc.llc_couple_workspace_size(S * L1 * K, K, V) + 12 * S * L1 * K * K + 512)
    out, spaces, stats = [], [], llc.new_stats(DEV)
    for st in (None, stats):
        spaces.append(torch.full((size,), 0xA5, dtype=torch.uint8, device=DEV))
        out.append(llc.llc_verify(target, tok, want_keys=True, strong=True, flags=flags, stats=st, workspace=spaces[-1], **kw))
    torch.cuda.synchronize()
    return out[0], out[1], stats_dict(stats)["near_ties"], int((spaces[0] != spaces[1]).sum()) > 8 * S * L1 * K


def _check(target, tok, at_once=True, **kw):
    out, loop, near_ties, other_form = _both(target, tok, **kw)
    assert other_form == at_once and near_ties == 0
    for name in ("Y", "n_out", "active"):
        assert torch.equal(out[name], loop[name]), name
    np.testing.assert_allclose(out["keyY"].cpu().numpy(), loop["keyY"].cpu().numpy(), rtol=2.0 ** -22 + 2.0 ** -23)
    return {k: out[k] for k in ("Y", "n_out", "active", "keyY")}


# (chunks of a row, one workgroup a row, two and four groups of drafts, ragged rows, one position, an odd number of drafts; sixty-four drafts are the loop's)
@pytest.mark.parametrize("S,L,K,V,dtype", [(1, 1, 2, 777, "f32"), (1, 4, 4, 32003, "bf16"), (3, 6, 8, 5001, "f32"), (5, 3, 9, 2051, "f32"),
                                           (30, 4, 5, 4099, "bf16"), (2, 2, 64, 517, "f32"), (40, 4, 3, 131, "f32"), (1, 4, 32, 517, "f32")])
def test_all_rows_for_all_drafts_at_once(S, L, K, V, dtype):
    g = torch.Generator().manual_seed(S * 1000 + L * 100 + K)
    target = 2.0 * torch.randn(S, L + 1, K, V, generator=g)
    target[:, 0, 1:] = target[:, 0, :1]
    target = target.to(DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    kw = dict(temp_target=0.8, seed=23, row_offset=(1 << 32) - 3, row_stride_s=7, row_stride_j=2)
    tok = _tokens(target, S, L, K, V, g, **kw)
    ref = oracle_verify(target, tok, (0, S), strong=True, **kw)
    compare_verify(_check(target, tok, K <= 32, **kw), ref)
    if L > 2 and S > 2:
        assert ref["n_out"].max() > 2
    _check(target, tok, K <= 32, flags=llc.FLAG_MIN_FIRST, **kw)


def test_strided_rows_log_weights_and_rows_without_mass():
    g = torch.Generator().manual_seed(43)
    S, L, K, V = 8, 4, 4, 2051
    store = (2 * torch.randn(S, K, L + 1, V + 3, generator=g)).to(DEV)   # [S, K, L+1, V'] permuted, odd rows
    target = store.permute(0, 2, 1, 3)[:, :, :, 1:1 + V]
    ninf = float("-inf")
    target[1, 1, 2, :], target[2, 0, :, :], target[4, 2, 0, :] = ninf, ninf, ninf
    target[3, 2, 0, 5], target[5, 1, 1, 7] = float("nan"), float("inf")
    tok = _tokens(target, S, L, K, V, g, kind="logw", seed=19)
    ref = oracle_verify(target, tok, (0, S), kind="logw", seed=19, strong=True)
    got = _check(target, tok, kind="logw", seed=19)
    compare_verify(got, ref)
    assert got["Y"][2, 0].item() == -1 and got["n_out"][2].item() == 1
    # one row for all drafts, and the same buffers again for other tokens
    one = target[:, :, :1].expand(S, L + 1, K, V)
    ref = oracle_verify(one, tok, (0, S), kind="logw", seed=19, strong=True)
    compare_verify(_check(one, tok, kind="logw", seed=19), ref)


def test_captured_and_replayed():
    g = torch.Generator().manual_seed(47)
    S, L, K, V = 6, 3, 4, 9001
    target = (2.0 * torch.randn(S, L + 1, K, V, generator=g)).to(DEV)
    tok = _tokens(target, S, L, K, V, g, seed=3)
    ws = torch.empty(llc.llc_verify_workspace_size(S, L, K, V), dtype=torch.uint8, device=DEV)
    call = lambda: llc.llc_verify(target, tok, seed=3, want_keys=True, strong=True, workspace=ws)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for turn in range(4):
        target.copy_(target.roll(1, dims=3))
        ws.fill_(turn)
        graph.replay()
        torch.cuda.synchronize()
        eager = llc.llc_verify(target, tok, seed=3, want_keys=True, strong=True)
        for name in ("Y", "n_out", "active", "keyY"):
            assert torch.equal(out[name], eager[name]), (turn, name)


@pytest.mark.parametrize("S,L,K,V,mf", [(100, 7, 8, 9000, False), (64, 2, 16, 4000, False), (128, 4, 4, 32000, False), (32, 7, 8, 9000, False), (64, 4, 10, 20000, True), (1, 1, 8, 70000, False), (3, 1, 8, 128256, True)])
def test_calls_that_are_slower_at_once_take_the_loop(S, L, K, V, mf):
    # (where no token is accepted the loop is its first scan and two launches a position without work)
    target = torch.randn(S, L + 1, K, V, device=DEV, dtype=torch.bfloat16)
    tok = torch.randint(0, V, (S, L, K), device=DEV, dtype=torch.int32)
    for size in (None, llc.llc_verify_workspace_size(S, L, K, V)):
        assert not _both(target, tok, size, flags=llc.FLAG_MIN_FIRST if mf else 0)[3]
