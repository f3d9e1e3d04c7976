"""The implicit non-local mask's global rows: ranges of key blocks, a quarter of each per wavefront, against the oracle."""
import numpy as np
import pytest

import paper_2502_01659_amd as sga
from sga_inputs import MaskSpec, KIND_NONLOCAL, numpy_qkv, torch_qkv
from oracle import reference as R
from gpu_util import TOL, LSE_TOL, to_device, max_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("L,g,W,H", [
    (20, 3, 4, 1), (33, 31, 2, 2), (256, 32, 9, 1), (257, 33, 300, 2), (289, 64, 5, 1), (352, 1, 0, 3),    # 1 to 11 blocks: ranges of 8
    (2049, 64, 40, 1), (3009, 7, 50, 2)])
def test_global_rows_over_ranges(dtype, L, g, W, H):
    """Last ranges of one, two and three blocks (wavefronts without a block), one and two tiles of global rows, windows
    that take whole ranges out of a row."""
    print("case", dtype, L, g, W, H, flush=True)
    spec = MaskSpec(KIND_NONLOCAL, L, window=W, n_global=g)
    Q, K, V = numpy_qkv(H, L, 64, dtype, 0.8, L + g)
    dQ, dK, dV = to_device(Q, K, V)
    ws = sga.alloc_workspace(L, H, 64, dtype, -1)
    ws.fill_(0xFF)
    O, lse = sga.attention_forward_implicit(dQ, dK, dV, spec, 0.125, workspace=ws, want_lse=True)
    want, want_lse = R.attention_masked(Q, K, V, spec, 0.125)
    some = np.isfinite(want_lse)
    got = lse.cpu().numpy()
    assert max_err(O.float().cpu().numpy(), want) <= TOL[dtype]
    assert (np.isfinite(got) == some).all() and (not some.any() or max_err(got[some], want_lse[some]) <= LSE_TOL[dtype])


@pytest.mark.parametrize("L,g,bar", [(3000, 16, 1.882e-7), (20000, 64, 2.734e-7)])
def test_global_rows_are_as_exact_as_of_whole_ranges(L, g, bar):
    """The error against 64 bits over eight inputs is no larger than `bar`, that of ranges which one wavefront walks from
    end to end (measured on these inputs, whatever the kernel)."""
    import torch
    W, error = 50, 0.0
    spec = MaskSpec(KIND_NONLOCAL, L, window=W, n_global=g)
    away = (torch.arange(g, device="cuda:0")[:, None] - torch.arange(L, device="cuda:0")[None, :]).abs() > W
    for seed in range(8):
        Q, K, V = torch_qkv(1, L, 64, "f32", 1.0, 200 + seed, "cuda:0")
        S = (Q[0, :g].double() @ K[0].double().t().contiguous()) * 0.125
        want = torch.softmax(S.masked_fill(~away, -float("inf")), dim=-1) @ V[0].double()
        O = sga.attention_forward_implicit(Q, K, V, spec, 0.125, workspace=sga.alloc_workspace(L, 1, 64, "f32", -1))
        error += ((O[0, :g].double() - want).norm() / want.norm()).item() / 8
    print("error", L, g, error, flush=True)
    assert error <= bar
