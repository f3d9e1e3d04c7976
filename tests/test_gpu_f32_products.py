"""fp32 storage on the matrix cores: the operands are split into 16-bit parts, so the cases here
are the ones where a split can go wrong: rows of very different magnitude in one key block, channels
of very different magnitude in one row, values near the ends of the fp32 range, huge values in keys
that a query does not attend, and infinities.  The per-row kernels, which use fp32 arithmetic throughout,
are the reference; each of them is compared with the oracle in test_gpu_attention.py."""
import os
import re

import pytest

import paper_2502_01659_amd as sga
from sga_inputs import MaskSpec, KIND_SLIDING, KIND_NONLOCAL, torch_qkv
from gpu_util import TOL

pytestmark = pytest.mark.gpu

# (head dimension, explicit CSR, length, window), run with H heads: window tiles of a small call and of
# one whose workgroups share their key blocks (cut into ranges: 3,333 and 15,001); work items claimed one
# by one, in fours on lists of their own and in fours on merged lists; wide tiles; ragged lengths,
# windows inside one key block and of many blocks
H = 2
FORMS = [(64, False, 333, 20), (64, False, 3333, 3000), (64, False, 30001, 700), (64, False, 15001, 1500),
         (64, False, 140003, 70),
         (64, True, 333, 20), (64, True, 4100, 300), (64, True, 16421, 20), (64, True, 40003, 250),
         (128, False, 333, 40), (256, True, 300, 20)]


# the route of the d = 64 forms: (explicit, claims in fours, key blocks shared by a workgroup)
ROUTES = [(False, None, False), (False, None, False), (False, None, True), (False, None, True), (False, None, True),
          (True, False, None), (True, False, None), (True, True, False), (True, True, True)]


def test_forms_take_the_routes_they_are_for():
    """The lines of the dispatch as the kernels' source states them, against the sizes of FORMS: a line that
    moves must not leave a kernel untested."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    source = open(os.path.join(root, "paper_2502_01659_amd", "csrc", "attention_tile.hip")).read()
    line = {n: int(re.search(r"constexpr int64_t %s = (\d+);" % n, source).group(1)) for n in ("kSharedSteps", "kSharedClaims")}
    for (d, explicit, L, W), (is_explicit, fours, shared) in zip(FORMS, ROUTES):
        assert d == 64 and explicit == is_explicit
        tiles = (L + 31) // 32
        if explicit:                    # (no tile of these windows is cut into segments)
            claims = (tiles + 3) // 4 * H
            blocks = 2 * W // 32 + 1    # of a tile's list, at least
            assert (claims >= line["kSharedClaims"]) == fours
            if fours:
                assert (claims * blocks >= line["kSharedSteps"]) == shared
                assert shared or claims * (blocks + 3) < line["kSharedSteps"]
        else:
            steps = (L + 127) // 128 * H * min((127 + 2 * W) // 32 + 1, tiles)
            assert (steps >= line["kSharedSteps"]) == shared


def _both(form, Q, K, V, scale):
    d, explicit, L, W = form
    spec = MaskSpec(KIND_SLIDING, L, window=W)
    if explicit:
        rp, ci = sga.build_mask(spec)
        ws = sga.alloc_workspace(L, Q.shape[0], d, "f32", ci.numel())
        return [sga.attention_forward(Q, K, V, rp, ci, scale, workspace=ws, path=p, want_lse=True)
                for p in (sga.PATH_TILE, sga.PATH_GATHER)]
    ws = sga.alloc_workspace(L, Q.shape[0], d, "f32", -1)
    return [sga.attention_forward_implicit(Q, K, V, spec, scale, workspace=ws, path=p, want_lse=True)
            for p in (sga.PATH_TILE, sga.PATH_GATHER)]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("q_exp,k_exp,v_exp", [(0, 0, 0), (60, -60, 100), (-90, 90, -60), (-30, 24, 0)])
def test_rows_of_different_magnitude(form, q_exp, k_exp, v_exp):
    """Rows scaled by powers of two: q_exp + k_exp + up to 6 per key stays near 0, the values reach
    2^+-100.  Bar: twice the fp32 tolerance relative to the largest value (a weighted mean of values
    rounds at their size), raised by the size of the scores, which round at 2^-24 of themselves."""
    import torch
    d, _, L, _ = form
    Q, K, V = torch_qkv(H, L, d, "f32", 1.0, 5, "cuda:0")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(9)
    per_key = torch.randint(-12, 3, (H, L, 1), generator=g, device="cuda:0").float()
    Q = Q * 2.0 ** q_exp
    K = K * torch.exp2(per_key + k_exp)
    V = V * 2.0 ** v_exp
    (O1, l1), (O2, l2) = _both(form, Q, K, V, d ** -0.5)
    assert torch.isfinite(O1).all()
    top = V.abs().max().item()
    assert (O1.double() - O2.double()).abs().max().item() <= 2 * TOL["f32"] * 4 * top
    assert (l1 - l2).abs().max().item() <= 1e-4


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("huge", [1e30, 3.39e38])
def test_huge_keys_outside_the_mask(form, huge):
    """A key nobody attends (its row is taken out of every comparison) shares key blocks with keys
    that count: its size must not reach them."""
    import torch
    d, _, L, W = form
    Q, K, V = torch_qkv(H, L, d, "f32", 1.0, 6, "cuda:0")
    O0, _ = _both(form, Q, K, V, d ** -0.5)[0]
    K2 = K.clone()
    j = 5
    K2[:, j] = huge
    O1, _ = _both(form, Q, K2, V, d ** -0.5)[0]
    far = (torch.arange(L, device="cuda:0") - j).abs() > W
    assert far.any()
    assert (O1[:, far] - O0[:, far]).abs().max().item() <= TOL["f32"]


@pytest.mark.parametrize("form", FORMS)
def test_minus_infinity_scores_weigh_nothing(form):
    """Keys with an infinite channel whose product is -inf for every query: weight 0, as on the per-row
    kernels."""
    import torch
    d, _, L, _ = form
    Q, K, V = torch_qkv(H, L, d, "f32", 1.0, 7, "cuda:0")
    Q[:, :, 3] = Q[:, :, 3].abs() + 0.25
    K[:, ::7, 3] = -float("inf")
    (O1, l1), (O2, l2) = _both(form, Q, K, V, d ** -0.5)
    assert torch.isfinite(O2).all() and torch.isfinite(O1).all()
    assert (O1 - O2).abs().max().item() <= 2 * TOL["f32"]
    assert (l1 - l2).abs().max().item() <= 1e-4


@pytest.mark.parametrize("L,density,H", [(1500, 0.6, 3), (4100, 0.3, 1), (8200, 0.5, 2), (6001, 1.0, 1)])
def test_tiles_cut_alike(L, density, H):
    """Dense random masks: every tile is cut into segments, four tiles alike (the last tiles of a ragged
    length are not), with a band of empty rows and three tiles of a quarter of the edges.  The
    prepared graph, whose claims start from what the call before left, repeats the call bit for bit."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(L)
    dense = torch.rand((L, L), generator=g, device="cuda:0") < density
    dense[200:232] = False
    dense[640:736, L // 4:] = False
    rp = torch.zeros(L + 1, dtype=torch.int64, device="cuda:0")
    rp[1:] = dense.sum(dim=1).cumsum(0)
    ci = dense.nonzero()[:, 1].to(torch.int32).contiguous()
    Q, K, V = torch_qkv(H, L, 64, "f32", 1.0, 3, "cuda:0")
    ws = sga.alloc_workspace(L, H, 64, "f32", ci.numel())
    O1, l1 = sga.attention_forward(Q, K, V, rp, ci, 0.125, workspace=ws, path=sga.PATH_TILE, want_lse=True)
    O2, l2 = sga.attention_forward(Q, K, V, rp, ci, 0.125, workspace=ws, path=sga.PATH_GATHER, want_lse=True)
    assert (O1 - O2).abs().max().item() <= 2 * TOL["f32"]
    some = torch.isfinite(l2)
    assert torch.equal(some, torch.isfinite(l1)) and (l1 - l2)[some].abs().max().item() <= 1e-4
    plan = sga.graph_prepare(rp, ci, H, 64, "f32", ws)
    for _ in range(3):
        O3 = sga.attention_forward_prepared(Q, K, V, rp, ci, 0.125, plan, ws, O=torch.full_like(Q, 7.0))
        assert torch.equal(O3, O1)


def _form_qkv(form, seed):
    d, _, L, _ = form
    return torch_qkv(H, L, d, "f32", 1.0, seed, "cuda:0")


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("q_exp,k_exp", [(-100, 112), (112, -100), (-115, 115), (-124, 125), (125, -124), (0, 13)])
def test_scores_of_one_sign(form, q_exp, k_exp):
    """Every product of Q and K is the same negative number, up to -2^19 after scaling: the scores of a row
    are equal, no weight may vanish, and O is the mean of the attended V."""
    import torch
    d = form[0]
    Q, K, V = _form_qkv(form, 11)
    Q = torch.full_like(Q, 2.0 ** q_exp)
    K = torch.full_like(K, -2.0 ** k_exp)
    (O1, l1), (O2, l2) = _both(form, Q, K, V, d ** -0.5)
    assert torch.isfinite(l2).all()
    # lse = score + ln(neighbours): rounds at the size of the score
    assert ((l1 - l2).abs() <= 1e-4 + 2.0 ** -22 * l2.abs()).all()
    assert (O1 - O2).abs().max().item() <= 2 * TOL["f32"]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("big,in_k", [(1e6, True), (1e8, True), (1e12, True), (1e8, False), (1e12, False), (1e30, True)])
def test_one_large_channel(form, big, in_k):
    """One channel of K (or of Q) is larger than the others by any factor and meets a channel of Q (or of K)
    that is smaller by the same factor: all channels count alike in the scores."""
    import torch
    d = form[0]
    Q, K, V = _form_qkv(form, 12)
    large, small = (K, Q) if in_k else (Q, K)
    large[:, :, 3] *= big
    small[:, :, 3] /= big
    (O1, l1), (O2, l2) = _both(form, Q, K, V, d ** -0.5)
    assert (O1 - O2).abs().max().item() <= 2 * TOL["f32"]
    assert (l1 - l2).abs().max().item() <= 1e-4


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("q_exp,k_exp,v_exp", [(-116, 116, 0), (116, -116, 0), (-121, 121, 0), (0, 0, -116), (0, 0, -121)])
def test_operands_near_the_smallest_numbers(form, q_exp, k_exp, v_exp):
    """Values whose low parts lie below the subnormal numbers of bf16: the bar is that of ordinary inputs,
    relative to the largest value."""
    import torch
    Q, K, V = _form_qkv(form, 15)
    (O1, l1), (O2, l2) = _both(form, Q * 2.0 ** q_exp, K * 2.0 ** k_exp, V * 2.0 ** v_exp, form[0] ** -0.5)
    assert (O1.double() - O2.double()).abs().max().item() <= 2 * TOL["f32"] * 2.0 ** v_exp
    assert (l1 - l2).abs().max().item() <= 1e-5


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_values_nobody_attends(form, value):
    """An infinite or undefined value in keys that no query of a 32-query tile attends leaves the tile alone,
    also where the tile attends other keys of their block.  Explicit forms: a mask without the columns
    from `first` on, which hold the value.  Window forms: the keys from `first` on hold it, and the
    tiles out of their reach are compared."""
    import torch
    d, explicit, L, W = form
    Q, K, V = _form_qkv(form, 13)
    V2 = V.clone()
    if explicit:
        rp, ci = sga.build_mask(MaskSpec(KIND_SLIDING, L, window=W))
        first = (L - 1) // 32 * 32 - 21                 # inside a key block
        row = torch.repeat_interleave(torch.arange(L, device="cuda:0"), rp[1:] - rp[:-1])
        keep = ci < first
        ci = ci[keep].contiguous()
        rp = torch.zeros_like(rp)
        rp[1:] = torch.bincount(row[keep], minlength=L).cumsum(0)
        ws = sga.alloc_workspace(L, H, d, "f32", ci.numel())
        run = lambda v: sga.attention_forward(Q, K, v, rp, ci, d ** -0.5, workspace=ws, path=sga.PATH_TILE)
        V2[:, first:] = value
        alone = torch.ones(L, dtype=torch.bool, device="cuda:0")
    else:
        spec = MaskSpec(KIND_SLIDING, L, window=W)
        ws = sga.alloc_workspace(L, H, d, "f32", -1)
        run = lambda v: sga.attention_forward_implicit(Q, K, v, spec, d ** -0.5, workspace=ws, path=sga.PATH_TILE)
        # the first key past the reach of a tile in the middle (of the first tile, if the window is wider)
        u0 = (max(W, L // 2) + 127) // 128 * 128
        if u0 + 32 + W >= L:
            u0 = 0
        first = u0 + 32 + W
        assert first < L
        V2[:, first:] = value
        alone = torch.arange(L, device="cuda:0") < u0 + 32
    O0, O1 = run(V), run(V2)
    assert alone.any()
    assert torch.isfinite(O1[:, alone]).all()
    assert (O1[:, alone] - O0[:, alone]).abs().max().item() <= TOL["f32"]


@pytest.mark.parametrize("d,L,g", [(64, 3001, 16), (64, 9000, 64), (128, 700, 5)])
@pytest.mark.parametrize("case", ["one_sign", "large_channel"])
def test_nonlocal_mask(d, L, g, case):
    """The same inputs on the kernels of the implicit non-local mask."""
    import torch
    Q, K, V = torch_qkv(H, L, d, "f32", 1.0, 14, "cuda:0")
    if case == "one_sign":
        Q = torch.full_like(Q, 2.0 ** -100)
        K = torch.full_like(K, -2.0 ** 112)
    else:
        K[:, :, 3] *= 1e8
        Q[:, :, 3] /= 1e8
    spec = MaskSpec(KIND_NONLOCAL, L, window=40, n_global=g)
    ws = sga.alloc_workspace(L, H, d, "f32", -1)
    (O1, l1), (O2, l2) = [sga.attention_forward_implicit(Q, K, V, spec, d ** -0.5, workspace=ws, path=p, want_lse=True)
                          for p in (sga.PATH_TILE, sga.PATH_GATHER)]
    some = torch.isfinite(l2)
    assert some.any() and torch.equal(some, torch.isfinite(l1))
    assert ((l1 - l2).abs() <= 1e-4 + 2.0 ** -22 * l2.abs())[some].all()
    assert (O1 - O2).abs().max().item() <= 2 * TOL["f32"]
