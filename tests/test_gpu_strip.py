"""fp16 windows beyond the staged ones: the kernel of 128 queries per workgroup (and the one of 256, on the other side of the
rule) against the per-row kernels, which share no code with them."""
import pytest

import paper_2502_01659_amd as sga
from sga_inputs import MaskSpec, KIND_SLIDING, KIND_DILATED, KIND_DILATED_2D, torch_qkv
from gpu_util import TOL, LSE_TOL

pytestmark = pytest.mark.gpu
STRIP, BAND = "tile_window_strip_kernel", "tile_window_band_kernel"


def _cases():
    out = []
    for L in (300, 513, 640, 1000, 4097):                  # classes of a few workgroups, ragged ends
        for W in (257, 272, 288, 289, 400, 5000):          # three to many interior blocks, even and odd counts, wider than the class
            out.append((MaskSpec(KIND_SLIDING, L, window=W), 2, STRIP))
    out.append((MaskSpec(KIND_DILATED, 5003, window=300, stride=3), 2, STRIP))
    out.append((MaskSpec(KIND_DILATED_2D, 7000, block=1300, stride=2), 1, STRIP))       # 650 queries to a class, the last 250
    out.append((MaskSpec(KIND_DILATED_2D, 2600, block=1299, stride=1), 2, STRIP))       # a last class of two tokens
    out.append((MaskSpec(KIND_SLIDING, 12001, window=12000), 21, BAND))
    return out


@pytest.mark.parametrize("case", range(len(_cases())))
def test_wide_windows_agree_with_row_kernels(case):
    import torch
    spec, H, kernel = _cases()[case]
    L = spec.L
    scale = -0.11 if case % 3 == 1 else 0.125
    print("case", case, spec, H, scale, flush=True)
    Q, K, V = torch_qkv(H, L, 64, "f16", 1.0, 50 + case, "cuda:0")
    assert sga.sga_profile_enable(1) == 0
    O1, l1 = sga.attention_forward_implicit(Q, K, V, spec, scale, want_lse=True)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == kernel
    O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER, want_lse=True)
    assert ((O1.float() - O2.float()).abs() / (1 + O2.float().abs())).max().item() <= 2 * TOL["f16"]
    assert torch.equal(torch.isfinite(l1), torch.isfinite(l2))
    seen = torch.isfinite(l2)
    assert (l1 - l2)[seen].abs().max().item() <= 2 * LSE_TOL["f16"]
    # continued: the same edges again leave O and add ln 2 (two roundings of O, two of the numerators)
    O3, l3 = O1.clone(), l1.clone()
    sga.attention_accumulate_implicit(Q, K, V, spec, scale, O3, l3)
    assert ((O3.float() - O1.float()).abs() / (1 + O1.float().abs())).max().item() <= 2 * TOL["f16"]
    assert (l3 - l1)[seen].sub(0.6931472).abs().max().item() <= 2 * LSE_TOL["f16"]


@pytest.mark.parametrize("L,H,W,kernel", [
    (16384, 1, 300, "tile_window_wide_kernel"), (16385, 1, 300, "tile_window_band128_kernel"),       # 128 and 129 workgroups
    (16500, 1, 240, "tile_window_wide_kernel"), (16500, 1, 255, "tile_window_band128_kernel"),       # 19 and 20 blocks
    (8200, 4, 48, "tile_window_wide_kernel"), (8200, 4, 60, "tile_window_band128_kernel"),           # 260 workgroups, 7 and 8 blocks
    (700, 44, 3000, "tile_window_band128_kernel"), (16384, 4, 1, "tile_window_band128_kernel")])     # classes of 22 blocks; 512 workgroups
def test_d128_windows_agree_with_row_kernels(L, H, W, kernel):
    """Both kernels of d = 128 on both sides of each line between them."""
    import torch
    spec = MaskSpec(KIND_SLIDING, L, window=W)
    print("case", L, H, W, flush=True)
    Q, K, V = torch_qkv(H, L, 128, "f16", 1.0, L + W, "cuda:0")
    assert sga.sga_profile_enable(1) == 0
    O1, l1 = sga.attention_forward_implicit(Q, K, V, spec, 0.088, want_lse=True)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == kernel
    O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, 0.088, path=sga.PATH_GATHER, want_lse=True)
    assert ((O1.float() - O2.float()).abs() / (1 + O2.float().abs())).max().item() <= 2 * TOL["f16"]
    assert (l1 - l2).abs().max().item() <= 2 * LSE_TOL["f16"]
