"""fp16 windows beyond the staged ones: the kernel of 128 queries per workgroup (and the one of 256, on the other side of the
rule) against the per-row kernels, which share no code with them."""
import pytest

import paper_2502_01659_amd as sga
from sga_inputs import MaskSpec, KIND_SLIDING, KIND_DILATED, KIND_DILATED_2D, torch_qkv
from gpu_util import TOL, LSE_TOL, check_window_state

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


@pytest.mark.parametrize("spec,H,kernel", [
    (MaskSpec(KIND_SLIDING, 5003, window=2100), 21, BAND),                    # edges of its own for every sub-tile
    (MaskSpec(KIND_DILATED, 6203, window=1500, stride=2), 16, BAND),          # classes of 3,102 and 3,101 queries
    (MaskSpec(KIND_DILATED, 6203, window=1200, stride=3), 28, BAND),
    (MaskSpec(KIND_DILATED_2D, 2101, block=2050, stride=1), 40, BAND),        # a last class of 51 queries
    (MaskSpec(KIND_DILATED_2D, 6203, block=3100, stride=1), 12, BAND),        # of three
    (MaskSpec(KIND_DILATED_2D, 5003, block=4101, stride=2), 40, BAND),        # 2,051 queries, then 451
    (MaskSpec(KIND_SLIDING, 1301, window=290), 2, STRIP),
    (MaskSpec(KIND_DILATED, 5003, window=300, stride=3), 2, STRIP),
    (MaskSpec(KIND_DILATED_2D, 2600, block=1299, stride=1), 2, STRIP)])
def test_wide_windows_continue_a_state(spec, H, kernel):
    """Peaked rows, and a second call of another scale on the state of the first: the old state's weight differs from
    row to row."""
    check_window_state(spec, H, 64, "f16", kernel)


@pytest.mark.parametrize("spec,H,kernel", [
    (MaskSpec(KIND_SLIDING, 9000, window=1100), 64, STRIP),      # 17.75 rounds of 256 workgroups, 72 blocks
    (MaskSpec(KIND_SLIDING, 9000, window=1700), 64, BAND),       # 110 blocks
    (MaskSpec(KIND_SLIDING, 8192, window=1000), 32, STRIP),      # exactly eight rounds
    (MaskSpec(KIND_SLIDING, 8192, window=1400), 32, BAND)])
def test_line_between_the_wide_kernels(spec, H, kernel):
    """Calls of many rounds: a round that is not full costs its share only."""
    import torch
    Q, K, V = torch_qkv(H, spec.L, 64, "f16", 1.0, 9, "cuda:0")
    assert sga.sga_profile_enable(1) == 0
    O = sga.attention_forward_implicit(Q, K, V, spec, 0.125)
    torch.cuda.synchronize()
    name = sga.sga_profile_last_kernel()
    sga.sga_profile_enable(0)
    assert name == kernel
    O2 = sga.attention_forward_implicit(Q, K, V, spec, 0.125, path=sga.PATH_GATHER)
    assert ((O.float() - O2.float()).abs() / (1 + O2.float().abs())).max().item() <= 2 * TOL["f16"]


SPECIAL = [(64, 1500, 304, 2, STRIP), (64, 5003, 2112, 21, BAND), (128, 1500, 304, 1, "tile_window_wide_share_kernel"),
           (128, 16500, 304, 1, "tile_window_band128_kernel")]


def _special(d, L, W, H, kernel, sigma):
    import torch
    spec = MaskSpec(KIND_SLIDING, L, window=W)
    Q, K, V = torch_qkv(H, L, d, "f16", sigma, 17, "cuda:0")
    ws = sga.alloc_workspace(L, H, d, "f16", -1)

    def run(K, V, scale):
        assert sga.sga_profile_enable(1) == 0
        O, lse = sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws, want_lse=True)
        torch.cuda.synchronize()
        name = sga.sga_profile_last_kernel()
        sga.sga_profile_enable(0)
        assert name == kernel
        return O.float(), lse
    return spec, Q, K, V, run


@pytest.mark.parametrize("d,L,W,H,kernel", SPECIAL)
def test_large_scores(d, L, W, H, kernel):
    """Scores of up to some hundreds, of either sign first.  Bar: the numerators and their sum are rounded to 11 bits, O
    once: 2 * 2^-11 of the largest value and 2^-11 of O on this side, 2^-11 of O on the other."""
    import torch
    spec, Q, K, V, run = _special(d, L, W, H, kernel, 2.0)
    for scale in (1.0, -1.0):
        O1, l1 = run(K, V, scale)
        O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, scale, path=sga.PATH_GATHER, want_lse=True)
        assert torch.isfinite(O1).all()
        assert (O1 - O2.float()).abs().max().item() <= 4 * 2.0 ** -11 * V.abs().max().item()
        # (fp32 sums of d products of the size of the score, and exp2 against a maximum of that size)
        assert ((l1 - l2).abs() <= 2 * LSE_TOL["f16"] + 2.0 ** -18 * l2.abs()).all()


@pytest.mark.parametrize("d,L,W,H,kernel", SPECIAL)
def test_minus_infinity_scores_weigh_nothing_fp16(d, L, W, H, kernel):
    import torch
    spec, Q, K, V, run = _special(d, L, W, H, kernel, 1.0)
    Q[:, :, 3] = Q[:, :, 3].abs() + 0.25
    K[:, ::7, 3] = -float("inf")
    O1, l1 = run(K, V, 0.125)
    O2, l2 = sga.attention_forward_implicit(Q, K, V, spec, 0.125, path=sga.PATH_GATHER, want_lse=True)
    assert torch.isfinite(O1).all() and torch.isfinite(l1).all()
    assert ((O1 - O2.float()).abs() / (1 + O2.float().abs())).max().item() <= 2 * TOL["f16"]
    assert (l1 - l2).abs().max().item() <= 2 * LSE_TOL["f16"]


@pytest.mark.parametrize("d,L,W,H,kernel", SPECIAL)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_values_out_of_reach_fp16(d, L, W, H, kernel, value):
    """Infinite or undefined values from the first key on that the tile of queries u0 .. u0 + 31 does not reach (2W a
    multiple of 32: no block is in part within reach): that tile and those before it give the bits they give without
    them, the rows that attend one hold no finite value."""
    import torch
    spec, Q, K, V, run = _special(d, L, W, H, kernel, 1.0)
    u0 = 512 if L < 5000 else (W + 255) // 256 * 256
    first = u0 + 32 + W
    assert 2 * W % 32 == 0 and first < L
    V2 = V.clone()
    V2[:, first:] = value
    O0, l0 = run(K, V, 0.125)
    O1, l1 = run(K, V2, 0.125)
    assert torch.equal(O0[:, :u0 + 32], O1[:, :u0 + 32]) and torch.equal(l0, l1)
    assert not torch.isfinite(O1[:, first - W:]).any()
