"""fp32 windows of calls with few tiles: two or four wavefronts per tile, against the per-row kernels."""
import pytest

import paper_2502_01659_amd as sga
from sga_inputs import MaskSpec, KIND_SLIDING, KIND_DILATED, KIND_DILATED_2D, torch_qkv
from gpu_util import TOL, LSE_TOL, check_window_state

pytestmark = pytest.mark.gpu
SHARE, ONE, GROUP = "tile_window_share_kernel", "tile_window_kernel", "tile_window_f32_kernel"


@pytest.mark.parametrize("spec,H,kernel", [
    (MaskSpec(KIND_SLIDING, 97, window=33), 1, SHARE),            # four blocks, the last of one key; a tile of one query
    (MaskSpec(KIND_SLIDING, 96, window=400), 1, ONE),             # three blocks: the class holds no more
    (MaskSpec(KIND_SLIDING, 1000, window=32), 2, ONE),            # three blocks inside
    (MaskSpec(KIND_SLIDING, 1001, window=49), 2, SHARE),          # five blocks for four wavefronts, fewer at the ends
    (MaskSpec(KIND_SLIDING, 10240, window=100), 1, SHARE),        # 320 tiles: four wavefronts each
    (MaskSpec(KIND_SLIDING, 10241, window=100), 1, SHARE),        # 321: two
    (MaskSpec(KIND_SLIDING, 4601, window=60), 8, SHARE),          # 1,152 tiles
    (MaskSpec(KIND_SLIDING, 4609, window=60), 8, ONE),            # 1,160
    (MaskSpec(KIND_SLIDING, 4096, window=64), 12, ONE),           # 1,536 of five blocks
    (MaskSpec(KIND_SLIDING, 4096, window=65), 12, SHARE),         # of six
    (MaskSpec(KIND_SLIDING, 4097, window=65), 12, ONE),           # 1,548
    (MaskSpec(KIND_SLIDING, 4001, window=700), 1, SHARE),         # two ranges of keys would be the other form,
    (MaskSpec(KIND_SLIDING, 4001, window=1000), 1, ONE),          # three are
    (MaskSpec(KIND_DILATED, 3001, window=70, stride=3), 1, SHARE),
    (MaskSpec(KIND_DILATED_2D, 3000, block=601, stride=2), 2, SHARE),
    (MaskSpec(KIND_SLIDING, 40000, window=200), 8, GROUP)])
def test_wavefronts_that_share_a_tile(spec, H, kernel):
    import torch
    L = spec.L
    scale = -0.125 if H == 2 else 0.125
    print("case", spec, H, flush=True)
    Q, K, V = torch_qkv(H, L, 64, "f32", 1.0, L, "cuda:0")
    ws = sga.alloc_workspace(L, H, 64, "f32", -1)
    assert sga.sga_profile_enable(1) == 0
    O1, l1 = sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws, want_lse=True)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == kernel
    O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER, want_lse=True)
    assert ((O1 - O2).abs() / (1 + O2.abs())).max().item() <= 2 * TOL["f32"]
    seen = torch.isfinite(l2)
    assert torch.equal(torch.isfinite(l1), seen) and (l1 - l2)[seen].abs().max().item() <= 2 * LSE_TOL["f32"]
    # continued, and with values whose split is not exact (computed again with fp32 products, per wavefront)
    O3, l3 = O1.clone(), l1.clone()
    sga.attention_accumulate_implicit(Q, K, V, spec, scale, O3, l3, workspace=ws)
    assert ((O3 - O1).abs() / (1 + O1.abs())).max().item() <= 2 * TOL["f32"]
    assert (l3 - l1)[seen].sub(0.6931472).abs().max().item() <= 2 * LSE_TOL["f32"]
    K[:, L // 2] *= 1e-36
    V[:, L // 3] = 1e-37
    O4 = sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws)
    O5 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER)
    assert ((O4 - O5).abs() / (1 + O5.abs())).max().item() <= 2 * TOL["f32"]


WIDE, WIDE_SHARE = "tile_window_wide_kernel", "tile_window_wide_share_kernel"


@pytest.mark.parametrize("spec,H,d,kernel", [
    (MaskSpec(KIND_SLIDING, 97, window=33), 1, 128, WIDE_SHARE),
    (MaskSpec(KIND_SLIDING, 96, window=400), 1, 256, WIDE),
    (MaskSpec(KIND_SLIDING, 1001, window=49), 2, 128, WIDE_SHARE),
    (MaskSpec(KIND_SLIDING, 1001, window=64), 2, 256, WIDE),              # five blocks
    (MaskSpec(KIND_SLIDING, 1001, window=65), 2, 256, WIDE_SHARE),        # six
    (MaskSpec(KIND_SLIDING, 8192, window=100), 1, 128, WIDE_SHARE),       # 256 tiles: four groups each
    (MaskSpec(KIND_SLIDING, 8193, window=100), 1, 128, WIDE_SHARE),       # 257: two
    (MaskSpec(KIND_SLIDING, 4096, window=100), 4, 128, WIDE_SHARE),       # 512
    (MaskSpec(KIND_SLIDING, 4097, window=100), 4, 128, WIDE),             # 516
    (MaskSpec(KIND_SLIDING, 8192, window=100), 1, 256, WIDE_SHARE),       # 256: two
    (MaskSpec(KIND_SLIDING, 8193, window=100), 1, 256, WIDE),
    (MaskSpec(KIND_SLIDING, 4001, window=1000), 1, 128, WIDE),            # three ranges of keys
    (MaskSpec(KIND_DILATED, 3001, window=70, stride=3), 1, 128, WIDE_SHARE),
    (MaskSpec(KIND_DILATED_2D, 3000, block=601, stride=2), 2, 256, WIDE_SHARE)])
def test_groups_that_share_a_wide_tile(spec, H, d, kernel):
    import torch
    L = spec.L
    scale = -0.125 if H == 2 else 0.125
    print("case", spec, H, d, flush=True)
    Q, K, V = torch_qkv(H, L, d, "f32", 1.0, L, "cuda:0")
    ws = sga.alloc_workspace(L, H, d, "f32", -1)
    assert sga.sga_profile_enable(1) == 0
    O1, l1 = sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws, want_lse=True)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == kernel
    O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER, want_lse=True)
    assert ((O1 - O2).abs() / (1 + O2.abs())).max().item() <= 2 * TOL["f32"]
    seen = torch.isfinite(l2)
    assert torch.equal(torch.isfinite(l1), seen) and (l1 - l2)[seen].abs().max().item() <= 2 * LSE_TOL["f32"]
    O3, l3 = O1.clone(), l1.clone()
    sga.attention_accumulate_implicit(Q, K, V, spec, scale, O3, l3, workspace=ws)
    assert ((O3 - O1).abs() / (1 + O1.abs())).max().item() <= 2 * TOL["f32"]
    assert (l3 - l1)[seen].sub(0.6931472).abs().max().item() <= 2 * LSE_TOL["f32"]
    K[:, L // 2] *= 1e-36
    V[:, L // 3] = 1e-37
    O4 = sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws)
    O5 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER)
    assert ((O4 - O5).abs() / (1 + O5.abs())).max().item() <= 2 * TOL["f32"]


@pytest.mark.parametrize("spec,H,d,kernel", [
    (MaskSpec(KIND_SLIDING, 8192, window=129), 1, 128, WIDE_SHARE),       # ten blocks, 256 tiles
    (MaskSpec(KIND_SLIDING, 8192, window=128), 1, 128, WIDE),             # nine
    (MaskSpec(KIND_SLIDING, 8193, window=129), 1, 128, WIDE),             # 257 tiles
    (MaskSpec(KIND_SLIDING, 321, window=400), 3, 128, WIDE_SHARE),        # eleven blocks, all of them in every tile
    (MaskSpec(KIND_SLIDING, 4001, window=600), 1, 128, WIDE_SHARE),
    (MaskSpec(KIND_SLIDING, 4001, window=1000), 1, 128, WIDE),            # three ranges of keys
    (MaskSpec(KIND_SLIDING, 8001, window=400), 1, 256, WIDE),
    (MaskSpec(KIND_DILATED, 3001, window=170, stride=3), 1, 128, WIDE_SHARE),
    (MaskSpec(KIND_DILATED_2D, 3000, block=1001, stride=3), 2, 128, WIDE_SHARE)])
def test_groups_that_share_a_wide_tile_fp16(spec, H, d, kernel):
    import torch
    L = spec.L
    scale = -0.125 if H == 2 else 0.125
    print("case", spec, H, d, flush=True)
    Q, K, V = torch_qkv(H, L, d, "f16", 0.5, L, "cuda:0")
    ws = sga.alloc_workspace(L, H, d, "f16", -1)
    assert sga.sga_profile_enable(1) == 0
    O1, l1 = sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws, want_lse=True)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == kernel
    O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER, want_lse=True)
    assert ((O1.float() - O2.float()).abs() / (1 + O2.float().abs())).max().item() <= 2 * TOL["f16"]
    seen = torch.isfinite(l2)
    assert torch.equal(torch.isfinite(l1), seen) and (l1 - l2)[seen].abs().max().item() <= 2 * LSE_TOL["f16"]
    O3, l3 = O1.clone(), l1.clone()
    sga.attention_accumulate_implicit(Q, K, V, spec, scale, O3, l3, workspace=ws)
    assert ((O3.float() - O1.float()).abs() / (1 + O1.float().abs())).max().item() <= 2 * TOL["f16"]
    assert (l3 - l1)[seen].sub(0.6931472).abs().max().item() <= 2 * LSE_TOL["f16"]


@pytest.mark.parametrize("spec,H,d,dtype,kernel", [
    (MaskSpec(KIND_SLIDING, 97, window=33), 1, 64, "f32", SHARE),
    (MaskSpec(KIND_SLIDING, 12001, window=100), 1, 64, "f32", SHARE),
    (MaskSpec(KIND_DILATED, 3001, window=70, stride=3), 2, 64, "f32", SHARE),
    (MaskSpec(KIND_SLIDING, 1001, window=49), 2, 128, "f32", WIDE_SHARE),
    (MaskSpec(KIND_SLIDING, 9001, window=100), 1, 128, "f32", WIDE_SHARE),
    (MaskSpec(KIND_SLIDING, 1001, window=65), 2, 256, "f32", WIDE_SHARE),
    (MaskSpec(KIND_SLIDING, 1301, window=200), 1, 128, "f16", WIDE_SHARE),
    (MaskSpec(KIND_DILATED, 3001, window=170, stride=3), 1, 128, "f16", WIDE_SHARE)] + [
    # a last class of one, two and three key blocks: ranges without a block
    (MaskSpec(KIND_DILATED_2D, 800 + n, block=400, stride=1), 2, d, dtype, kernel)
    for n in (1, 33, 70) for d, dtype, kernel in ((64, "f32", SHARE), (128, "f32", WIDE_SHARE), (256, "f32", WIDE_SHARE),
                                                  (128, "f16", WIDE_SHARE))])
def test_shared_tiles_continue_a_state(spec, H, d, dtype, kernel):
    """Peaked rows, and a second call of another scale on the state of the first: the old state's weight differs from
    row to row."""
    check_window_state(spec, H, d, dtype, kernel)


@pytest.mark.parametrize("d,L,copies,share,one", [(64, 12001, 4, SHARE, ONE), (128, 8001, 3, WIDE_SHARE, WIDE)])
def test_shared_tiles_are_as_exact(d, L, copies, share, one):
    """Tiles of four blocks, shared and, in a call of the same head several times over, not: the error against 64 bits is no
    larger (means over eight inputs; those of one kernel repeat to 0.1 % with eight others)."""
    import torch
    W, scale = 33, d ** -0.5
    spec = MaskSpec(KIND_SLIDING, L, window=W)
    i = torch.arange(L, device="cuda:0")
    j = i[:, None] + torch.arange(-W, W + 1, device="cuda:0")[None, :]
    inside = (j >= 0) & (j < L)
    j = j.clamp(0, L - 1)
    errors = {share: 0.0, one: 0.0}
    for seed in range(8):
        Q, K, V = torch_qkv(1, L, d, "f32", 1.0, 100 + seed, "cuda:0")
        S = (Q[0].double()[:, None, :] * K[0].double()[j]).sum(-1) * scale
        P = torch.softmax(S.masked_fill(~inside, -float("inf")), dim=-1)
        want = (P[:, :, None] * V[0].double()[j]).sum(1)
        for kernel, n in ((share, 1), (one, copies)):
            q, k, v = (x.expand(n, L, d).contiguous() for x in (Q, K, V))
            assert sga.sga_profile_enable(1) == 0
            O = sga.attention_forward_implicit(q, k, v, spec, scale, workspace=sga.alloc_workspace(L, n, d, "f32", -1))
            torch.cuda.synchronize()
            name = sga.sga_profile_last_kernel()
            sga.sga_profile_enable(0)
            assert name == kernel
            errors[kernel] += ((O[-1].double() - want).norm() / want.norm()).item() / 8
    print(errors, flush=True)
    assert errors[share] <= 1.001 * errors[one]
