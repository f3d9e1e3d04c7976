"""Prepared graphs of short rows of about one length (a row per lane group) against the calls without a plan, whose kernel
takes a row per wavefront, bit for bit."""
import numpy as np
import pytest

import paper_2502_01659_amd as sga
from sga_inputs import torch_qkv
from oracle import rowscan as C

pytestmark = pytest.mark.gpu


def _csr(L, mean, least, most, seed):
    """Rows of `least` to `most` neighbours, anywhere."""
    import torch
    rng = np.random.default_rng(seed)
    deg = rng.integers(least, most + 1, size=L)
    deg[rng.integers(0, L, size=8)] = 0
    deg[-1], deg[0], deg[1], deg[2] = most, 1, 15, 16
    cols = [np.sort(rng.choice(L, size=n, replace=False)).astype(np.int32) for n in deg]
    rp = np.zeros(L + 1, dtype=np.int64)
    rp[1:] = np.cumsum(deg)
    return torch.from_numpy(rp).cuda(), torch.from_numpy(np.concatenate(cols)).cuda()


@pytest.mark.parametrize("dtype,d,L,H,least,most,even", [
    ("f32", 64, 16385, 1, 20, 50, True), ("f32", 64, 8193, 2, 1, 33, True), ("f32", 64, 16390, 1, 90, 130, True),
    ("f32", 128, 16391, 1, 8, 40, True), ("f16", 128, 16387, 1, 20, 70, True), ("f16", 256, 8199, 2, 16, 49, True),
    ("f16", 64, 16400, 1, 20, 50, False),                # (eight rows at a time are not built)
    ("f32", 64, 16000, 1, 20, 50, False),                # too few rows
    ("f32", 64, 16400, 1, 1, 200, True)])
def test_even_rows_bit_for_bit(dtype, d, L, H, least, most, even):
    import torch
    print("case", dtype, d, L, H, least, most, flush=True)
    rp, ci = _csr(L, (least + most) // 2, least, most, L + d)
    nnz = ci.numel()
    Q, K, V = torch_qkv(H, L, d, dtype, 0.7, d, "cuda:0")
    ws = sga.alloc_workspace(L, H, d, dtype, nnz)
    O1, l1 = sga.attention_forward(Q, K, V, rp, ci, -0.11, workspace=ws, want_lse=True)
    plan = sga.graph_prepare(rp, ci, H, d, dtype, ws)
    assert plan.flags & sga.GRAPH_ROWS_EVEN
    assert sga.sga_profile_enable(1) == 0
    O2, l2 = sga.attention_forward_prepared(Q, K, V, rp, ci, -0.11, plan, ws, want_lse=True)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == ("gather_even_rows_kernel" if even else "gather_csr_kernel")
    assert torch.equal(O1, O2) and torch.equal(l1, l2)
    # the same state continued
    sga.attention_accumulate_prepared(Q, K, V, rp, ci, 0.05, plan, ws, O2, l2)
    sga.attention_accumulate(Q, K, V, rp, ci, 0.05, O1, l1, workspace=sga.alloc_workspace(L, H, d, dtype, nnz))
    assert torch.equal(O1, O2) and torch.equal(l1, l2)


def test_rows_of_uneven_length_keep_a_wavefront_each():
    """One row of 400 neighbours among rows of 20 to 50 (average 35: the line is at 134)."""
    import torch
    L = 16500
    rp, ci = _csr(L, 35, 20, 50, 1)
    rp, ci = rp.cpu().numpy(), ci.cpu().numpy()
    long = np.sort(np.random.default_rng(2).choice(L, size=400, replace=False)).astype(np.int32)
    at = 4321
    ci = np.concatenate([ci[:rp[at]], long, ci[rp[at + 1]:]])
    rp[at + 1:] += 400 - (rp[at + 1] - rp[at])
    rp, ci = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
    ws = sga.alloc_workspace(L, 1, 64, "f32", ci.numel())
    plan = sga.graph_prepare(rp, ci, 1, 64, "f32", ws)
    assert not plan.flags & sga.GRAPH_ROWS_EVEN
    Q, K, V = torch_qkv(1, L, 64, "f32", 0.7, 3, "cuda:0")
    O = sga.attention_forward_prepared(Q, K, V, rp, ci, 0.125, plan, ws)
    want, _ = C.attend_gathered(Q[0, at].cpu().numpy(), K[0].cpu().numpy()[long], V[0].cpu().numpy()[long], 0.125)
    assert np.abs(O[0, at].cpu().numpy() - want).max() <= 1e-5


@pytest.mark.parametrize("lo,hi,run,even", [
    (5, 195, 64, False), (5, 195, 1, False), (60, 140, 64, True), (100, 100, 1, True), (36, 164, 1024, False)])
def test_rows_of_two_lengths(lo, hi, run, even):
    """`run` rows of one length, then as many of the other.  None is longer than twice the average and 64, but a variance
    above a third of the squared average (100) plus the average is a mix that a row per lane group slows down."""
    import torch
    L, H, d = 16450, 1, 64
    rng = np.random.default_rng(lo + run)
    deg = np.where((np.arange(L) // run) % 2 == 1, hi, lo)
    cols = [np.sort(rng.choice(L, size=n, replace=False)).astype(np.int32) for n in deg]
    rp = np.zeros(L + 1, dtype=np.int64)
    rp[1:] = np.cumsum(deg)
    rp, ci = torch.from_numpy(rp).cuda(), torch.from_numpy(np.concatenate(cols)).cuda()
    Q, K, V = torch_qkv(H, L, d, "f32", 0.7, 5, "cuda:0")
    ws = sga.alloc_workspace(L, H, d, "f32", ci.numel())
    O1 = sga.attention_forward(Q, K, V, rp, ci, 0.125, workspace=ws)
    plan = sga.graph_prepare(rp, ci, H, d, "f32", ws)
    assert bool(plan.flags & sga.GRAPH_ROWS_EVEN) == even
    assert torch.equal(O1, sga.attention_forward_prepared(Q, K, V, rp, ci, 0.125, plan, ws))
