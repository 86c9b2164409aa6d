"""GPU parity of llc_lml_bound for rows that are sorted in LDS (needs an MI355X), at the ends of a thread's and a wavefront's part and of the
two capacities.  Bound on the error as for every sorted row: masses rounded to fp32, indices whose ratios agree to fp32 in
either order, 2^-22; tv and the relaxed sums are 64-bit sums."""
import numpy as np
import pytest
import torch

import paper_2506_05632_amd as llc
from oracle import lml

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(draft, target, ks, kind="logits", **kw):
    gpu = llc.llc_lml_bound(draft, target, ks, kind=kind, **kw)
    torch.cuda.synchronize()
    ref = lml.lml_rows(draft.float().cpu().numpy(), target.float().cpu().numpy(), ks, kind=kind, **kw)
    np.testing.assert_allclose(gpu["bound"].cpu().numpy(), ref["bound"], rtol=2.0 ** -22, err_msg="bound")
    for name in ("relaxed", "tv"):
        np.testing.assert_allclose(gpu[name].cpu().numpy(), ref[name], rtol=1e-12, atol=1e-15, err_msg=name)
    again = llc.llc_lml_bound(draft, target, ks, kind=kind, **kw)
    for name in ("bound", "relaxed", "tv"):
        assert torch.equal(again[name], gpu[name]), name


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [1, 2, 63, 64, 65, 1000, 1023, 1024, 1025, 2047, 2049, 3072, 4095, 4096, 4097, 5121, 6143, 6145, 8191])
def test_ends_of_parts_and_capacities(V, dtype):
    g = torch.Generator(device=DEV).manual_seed(V)
    target = 3.0 * torch.randn(5, V, generator=g, device=DEV)
    draft = (target + torch.randn(5, V, generator=g, device=DEV)).to(dtype)
    target = target.to(dtype)
    p, q = draft.float().softmax(1), target.float().softmax(1)
    p[0], q[1, V // 2:] = q[0], 0.0
    q[1, 0] = 1e-30
    _check(p, q, [3], kind="probs")
    assert llc.llc_lml_bound(p, q, [3], kind="probs")["tv"][0] == 0.0
    if V > 2:
        draft[1, ::3], target[1, 1::4] = float("-inf"), float("nan")  # no mass on a side, or on both
        target[2, 1:] = target[2, 0]                                  # one flat side; many equal ratios
        draft[3] = target[3]
        draft[4, 0] = float("inf")
        draft[4, V // 2], target[4, V - 1] = 60.0, 60.0               # disjoint heavy entries, one the row's last
    _check(draft, target, [1, 2, 3, 4, 5, 6, 7, 65535], temp_draft=0.7, temp_target=0.9)


def test_rows_without_mass_strides_and_optional_results():
    g = torch.Generator(device=DEV).manual_seed(7)
    wide = 3.0 * torch.randn(2, 700, 1501, generator=g, device=DEV)
    draft, target = wide[0, :, 1:1500], wide[1, :, 1:1500]  # rows that start on no 16-byte boundary
    _check(draft, target, [2, 8])
    draft[:, :] = float("-inf")
    out = llc.llc_lml_bound(draft, target, [1, 16])
    assert (out["bound"] == 0.0).all() and (out["relaxed"] == 0.0).all() and torch.allclose(out["tv"], torch.full_like(out["tv"], 0.5))
