"""llc_couple_topm where its list of candidates runs full, or its fp32 prefilter has nothing to go by (needs an
MI355X): many equal values, values of very different sizes, lists longer than a wavefront.  Against the
oracle, indices bit for bit (near-ties excused), keys to 1e-6."""
import pytest
import torch

import paper_2506_05632_amd as llc
from parity_util import compare, oracle_near_ties, stats_dict
from test_gpu_topm import oracle_topm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", ["logits", "logw", "probs"])
@pytest.mark.parametrize("K,M,scale", [(8, 64, 0.0), (3, 65, 2.0), (5, 700, 1e3), (2, 130, 1e30), (70, 33, 1.0), (1, 4097, 3.0)])
def test_prefilter_and_list(kind, K, M, scale):
    g = torch.Generator(device=DEV).manual_seed(M)
    B = 5
    ids = torch.stack([torch.randperm(20000, generator=g, device=DEV)[:M] for _ in range(2 * B)]).int()
    val = scale * torch.randn(2 * B, M, generator=g, device=DEV)
    if kind == "probs":
        # (weights up to e^40: the reported fp32 key S/p then stays above 1e-10 e^-40 = 4e-28; with e^80 it is
        # subnormal, where the rounding of the output alone, 2^-150, is 3e-6 of it)
        val = torch.exp(torch.clamp(val, -40, 40))
    val[0, ::3] = float("-inf") if kind != "probs" else 0.0
    val[B + 1, 0] = float("nan")
    stats = llc.new_stats(DEV)
    args = (ids[:B].contiguous(), val[:B].contiguous(), ids[B:].contiguous(), val[B:].contiguous(), K)
    out = llc.llc_couple_topm(*args, kind=kind, seed=3, temp_target=0.8, temp_draft=1.3, want_keys=True, stats=stats)
    torch.cuda.synchronize()
    ref = oracle_topm(*args, kind=kind, seed=3, temp_target=0.8, temp_draft=1.3)
    # (at 1e30 the fp64 rounding of x / T is 1e14: a log-domain key cannot carry ln S, only the indices say something)
    assert compare(out, ref, check_keys=scale < 1e6) <= oracle_near_ties(ref)
    assert stats_dict(stats)["near_ties"] == oracle_near_ties(ref)


def test_a_full_list_gives_the_same():
    # one value everywhere but for a spread far below the band: every pair is a candidate
    g = torch.Generator(device=DEV).manual_seed(9)
    B, K, M = 3, 9, 900
    ids = torch.stack([torch.randperm(5000, generator=g, device=DEV)[:M] for _ in range(2 * B)]).int()
    val = 1e30 + torch.zeros(2 * B, M, device=DEV)
    out = llc.llc_couple_topm(ids[:B].contiguous(), val[:B].contiguous(), ids[B:].contiguous(), val[B:].contiguous(), K, seed=1)
    flat = llc.llc_couple_topm(ids[:B].contiguous(), 0 * val[:B], ids[B:].contiguous(), 0 * val[B:], K, seed=1)
    torch.cuda.synchronize()
    assert out["X"].shape == (B, K) and (out["X"] >= 0).all() and (flat["X"] >= 0).all()
    # (at 1e30 ln S is lost in the fp64 of x / T: every key of a reduction is the same, and the smallest id wins)
    assert (out["X"] == ids[:B].amin(dim=1, keepdim=True)).all() and torch.equal(out["Y"], ids[B:].amin(dim=1))
    assert torch.equal(out["accept"].bool(), out["X"][:, 0] == out["Y"])
    assert torch.equal(out["match_k"], torch.where(out["X"][:, 0] == out["Y"], 0, -1).int())
    ref = oracle_topm(ids[:B], 0 * val[:B], ids[B:], 0 * val[B:], K, seed=1)
    assert compare(flat, ref) <= oracle_near_ties(ref)


@pytest.mark.parametrize("kind,dtype", [("logits", torch.float32), ("logits", torch.bfloat16), ("probs", torch.float32)])
@pytest.mark.parametrize("K,M", [(400, 50), (401, 50), (167, 256), (168, 256), (1024, 60), (130, 1100)])
def test_many_drafts(kind, dtype, K, M):
    # as many drafts as share the list of candidates, one more, many
    g = torch.Generator(device=DEV).manual_seed(K)
    B = 3
    ids = torch.stack([torch.randperm(20000, generator=g, device=DEV)[:M] for _ in range(2 * B)]).int()
    val = torch.randn(2 * B, M, generator=g, device=DEV)
    if kind == "probs":
        val = torch.softmax(2 * val, dim=1)
    val = val.to(dtype)
    val[0, 3:] = 0.0 if kind == "probs" else float("-inf")
    stats = llc.new_stats(DEV)
    args = (ids[:B].contiguous(), val[:B].contiguous(), ids[B:].contiguous(), val[B:].contiguous(), K)
    out = llc.llc_couple_topm(*args, kind=kind, seed=3, want_keys=True, stats=stats)
    torch.cuda.synchronize()
    ref = oracle_topm(*args, kind=kind, seed=3)
    assert compare(out, ref) <= oracle_near_ties(ref)
    assert stats_dict(stats)["near_ties"] == oracle_near_ties(ref)
    assert stats_dict(stats)["exact_evals"] == 2 * K * M * B - K * (M - 3)


@pytest.mark.parametrize("kind", ["logits", "logw", "probs"])
@pytest.mark.parametrize("K", [2, 70])
def test_a_list_of_candidates_that_overflows_with_finite_keys(kind, K):
    # one id over and over with one value (700 equal keys, all of them the winner's if it wins), others beside it,
    # on either side: every entry is evaluated, and only other ids count as runners-up
    g = torch.Generator(device=DEV).manual_seed(K)
    B, M = 4, 760
    ids = torch.stack([torch.randperm(9000, generator=g, device=DEV)[:M] for _ in range(2 * B)]).int()
    val = torch.randn(2 * B, M, generator=g, device=DEV)
    val[:, 40:740] = 9.0
    ids[:, 40:740] = ids[:, 40:41]
    val[1] = torch.randn(M, generator=g, device=DEV)   # (rows in which one side's candidates are few)
    val[B + 2] = torch.randn(M, generator=g, device=DEV)
    if kind == "probs":
        val = torch.exp(val)
    stats = llc.new_stats(DEV)
    args = (ids[:B].contiguous(), val[:B].contiguous(), ids[B:].contiguous(), val[B:].contiguous(), K)
    out = llc.llc_couple_topm(*args, kind=kind, seed=5, temp_target=0.8, temp_draft=1.3, want_keys=True, stats=stats)
    torch.cuda.synchronize()
    ref = oracle_topm(*args, kind=kind, seed=5, temp_target=0.8, temp_draft=1.3)
    assert compare(out, ref) <= oracle_near_ties(ref)
    assert stats_dict(stats)["near_ties"] == oracle_near_ties(ref)


def _long_lists(B, K, Md, Mt, scale, kind, own=False):
    g = torch.Generator(device=DEV).manual_seed(Md + Mt)
    ids = [torch.stack([torch.randperm(131072, generator=g, device=DEV)[:M] for _ in range(n)]).int().view(*shape, M)
           for n, shape, M in ((B * K if own else B, (B, K) if own else (B,), Md), (B, (B,), Mt))]
    val = [scale * torch.randn(i.shape, generator=g, device=DEV) for i in ids]
    if kind == "probs":
        val = [torch.exp(v) for v in val]
    return ids[0], val[0], ids[1], val[1], K


# (either side of where whole words are drawn for what is near by its half-word, by lists, by the pool, in parts)
@pytest.mark.parametrize("K,Md,Mt", [(5, 65536, 16384), (40, 65536, 50), (50, 65536, 50), (200, 50, 50), (246, 50, 16384), (256, 50, 65536),
                                     (300, 700, 4096), (120, 4096, 700)])
@pytest.mark.parametrize("kind,scale", [("logits", 0.0), ("logits", 3.0), ("probs", 0.0), ("probs", 1.0)])
def test_long_lists(K, Md, Mt, kind, scale):
    args = _long_lists(2, K, Md, Mt, scale, kind)
    stats = llc.new_stats(DEV)
    out = llc.llc_couple_topm(*args, kind=kind, seed=7, want_keys=True, stats=stats)
    torch.cuda.synchronize()
    ref = oracle_topm(*args, kind=kind, seed=7)
    assert compare(out, ref) <= oracle_near_ties(ref)
    assert stats_dict(stats)["near_ties"] == oracle_near_ties(ref)
    assert stats_dict(stats)["exact_evals"] == 2 * K * (Md + Mt)


# (either side of where drafts are taken one at a time, and of where two wavefronts share a list)
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("Md,Mt", [(1, 1), (20, 42), (20, 43), (64, 64), (64, 65), (65, 1), (128, 64), (129, 500), (700, 50)])
@pytest.mark.parametrize("own,kind", [(False, "logits"), (True, "logits"), (False, "probs")])
def test_few_drafts(K, Md, Mt, own, kind):
    args = _long_lists(6, K, Md, Mt, 1.0, kind, own)
    stats = llc.new_stats(DEV)
    out = llc.llc_couple_topm(*args, kind=kind, seed=11, want_keys=True, stats=stats)
    torch.cuda.synchronize()
    ref = oracle_topm(*args, kind=kind, seed=11)
    assert compare(out, ref) <= oracle_near_ties(ref)
    assert stats_dict(stats)["near_ties"] == oracle_near_ties(ref)
    assert stats_dict(stats)["exact_evals"] == 6 * K * (Md + Mt)


@pytest.mark.parametrize("K,Md,Mt,own", [(256, 50, 65536, False), (50, 65536, 65536, True)])
def test_flat_long_lists_leave_few_candidates(K, Md, Mt, own):
    # what overflows the list of candidates is evaluated in 64 bits, all of it, at several times the cost: flat lists must
    # not (values far apart, with some hundred candidates less, show what a call takes otherwise)
    def us(scale):
        args = _long_lists(8, K, Md, Mt, scale, "logits", own)
        llc.llc_couple_topm(*args, seed=7)
        torch.cuda.synchronize()
        taken = []
        for _ in range(3):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            llc.llc_couple_topm(*args, seed=7)
            b.record()
            torch.cuda.synchronize()
            taken.append(a.elapsed_time(b) * 1e3)
        return min(taken)
    flat, apart = us(0.0), us(100.0)
    print(f"flat {flat:.0f} us, apart {apart:.0f} us")
    assert flat < 1.4 * apart
