"""What workspace a call of few rows takes, by dry runs (no GPU): finer chunks are planned only where they fit, so that whatever was
enough before them still is."""
import ctypes

import pytest

import paper_2506_05632_amd as llc
from paper_2506_05632_amd import binding
from test_abi import _args


def _least(**kw):
    """The smallest workspace that a call accepts."""
    lib = llc.load()
    ok = lambda n: lib.llc_couple(ctypes.byref(_args(flags=binding.FLAG_DRY_RUN, workspace_bytes=n, **kw))) == 0
    lo, hi = 0, 1 << 26
    assert ok(hi)
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if ok(mid) else (mid, hi)
    return hi


def _layout(B, K, groups, chunks):
    up = lambda n: (n + 255) // 256 * 256
    return (up(B * K * chunks * 8) + up(B * K * chunks * 4) + up(B * groups * chunks * 8) + 2 * up(B * groups * chunks * 4) +
            up(B * K * chunks * 8) + up(B * groups * chunks * 8) + up(B * (K + 1) * 8) + up(B * (K + 1) * chunks * 8))


# (rows, drafts, entries, groups of drafts, chunks without the finer shapes: two tiles of 1024 threads each)
@pytest.mark.parametrize("B,K,V,groups,chunks", [(4, 4, 32000, 1, 4), (1, 2, 24576, 1, 3), (16, 3, 40001, 1, 5), (2, 8, 50257, 1, 5), (3, 6, 45056, 1, 4)])
def test_the_least_workspace_is_what_it_was(B, K, V, groups, chunks):
    assert _least(B=B, K=K, V=V, draft_stride_b=V, target_stride_b=V) == _layout(B, K, groups, chunks)


# rows for which chunks of 256 threads fill the chip better: the least workspace is that of one chunk a row
@pytest.mark.parametrize("own,kw", [(True, dict(B=300, K=4, V=50257, keyX=0x3000, keyY=0x3000)), (True, dict(B=140, K=4, V=128256, keyX=0x3000, keyY=0x3000)),
                                    (True, dict(B=341, K=4, V=50257)), (False, dict(B=257, K=8, V=128256)), (False, dict(B=300, K=6, V=152064))])
@pytest.mark.parametrize("dtype", [binding.F32, binding.BF16])
def test_a_workspace_for_one_chunk_a_row_is_enough(own, kw, dtype):
    B, K, V = kw["B"], kw["K"], kw["V"]
    strides = dict(draft_stride_b=K * V if own else V, draft_stride_k=V if own else 0, target_stride_b=V)
    assert _least(dtype=dtype, **strides, **kw) == _layout(B, K, 1, 1)
