"""Explicit masks whose rows have one shape within a tile (equal degrees, the same few runs of consecutive columns), which the
CSR -> tile pass reads at the ends of the runs only, and masks that just miss that rule, against the oracle."""
import numpy as np
import pytest

import paper_2502_01659_amd as sga
from sga_inputs import numpy_qkv
from oracle import reference as R
from gpu_util import TOL, LSE_TOL, to_device, max_err

pytestmark = pytest.mark.gpu
L = 2208          # 69 tiles


def _rows(lens, gap, shift, seed):
    """Every tile takes runs of these lengths at random places at least `gap` columns apart, in every row `shift` columns
    further on than in the row above."""
    rng = np.random.default_rng(seed)
    mask = np.zeros((L, L), dtype=bool)
    for t in range(L // 32):
        free = L - sum(lens) - gap * len(lens) - 31 * shift
        cuts = np.sort(rng.integers(0, free + 1, size=len(lens)))
        for r in range(32):
            at = r * shift
            for i, n in enumerate(lens):
                lo = at + cuts[i] - (cuts[i - 1] if i else 0)
                mask[32 * t + r, lo:lo + n] = True
                at = lo + n + gap
    return mask


def _masks():
    out = {}
    few = np.argsort(np.random.default_rng(1).random((L // 32, L // 32)), axis=1) < 6
    out["aligned blocks"] = np.kron(few, np.ones((32, 32), dtype=bool))
    out["eight runs"] = _rows([64, 40, 33, 96, 64, 31, 128, 200], 1, 0, 2)
    out["nine runs"] = _rows([64, 40, 33, 96, 64, 31, 128, 100, 100], 1, 0, 3)
    out["runs that share a block"] = _rows([20, 7, 90, 64], 2, 0, 4)
    out["sloped"] = _rows([33, 64, 150], 5, 1, 5)
    out["touching"] = _rows([64, 64, 64], 0, 0, 6)
    out["1,024 columns"] = _rows([512, 512], 3, 0, 7)
    out["1,025 columns"] = _rows([512, 513], 3, 0, 8)
    out["thin"] = _rows([3, 2, 3, 2, 3, 2, 3, 2], 40, 0, 9)
    out["thin, then dense"] = _rows([2, 2, 2, 2, 2, 2, 2, 900], 40, 0, 10)
    out["dense, sixteen blocks, then thin"] = _rows([500, 2, 2, 2, 2, 2, 2], 40, 0, 11)
    odd = _rows([64, 64, 96], 10, 0, 12)
    for t in range(0, 69, 2):                            # one row of every other tile: as long, but elsewhere
        odd[32 * t + 5 + t % 27] = np.roll(odd[32 * t + 5 + t % 27], 17)
    out["one row elsewhere"] = odd
    split = _rows([64, 64, 96], 10, 0, 13)
    for t in range(0, 69, 2):                            # one row: a column inside a run moved, the run's ends as they are
        row = split[32 * t + 9]
        inside = np.flatnonzero(row)[70]
        row[inside] = False
        row[np.flatnonzero(~row & (np.arange(L) > inside + 64))[0]] = True
    out["a hole in a run"] = split
    out["scattered, as many in every row"] = _rows([1] * 20, 9, 0, 15)
    out["single columns at both ends"] = _rows([1, 64, 90, 1], 10, 0, 16)      # (read run by run)
    out["a single column first"] = _rows([1, 64, 90], 10, 0, 17)
    out["a single column last"] = _rows([64, 90, 1], 10, 1, 18)
    empty = _rows([64, 32], 10, 0, 14)
    empty[::17] = False
    out["empty rows"] = empty
    return out


MASKS = _masks()


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("name", list(MASKS))
def test_tiles_of_rows_of_one_shape(name, dtype):
    """All of the sequence, and with the last tile cut short (2,190 rows and keys)."""
    import torch
    for n in (L, L - 18):
        print("case", name, dtype, n, flush=True)
        mask = MASKS[name][:n, :n]
        rp, ci = (torch.from_numpy(x).cuda() for x in R.csr_from_dense(mask))
        Q, K, V = numpy_qkv(1, n, 64, dtype, 0.8, 7)
        dQ, dK, dV = to_device(Q, K, V)
        ws = sga.alloc_workspace(n, 1, 64, dtype, ci.numel())
        O, lse = sga.attention_forward(dQ, dK, dV, rp, ci, 0.125, workspace=ws, want_lse=True)
        want, want_lse = R.attention_dense(Q[0], K[0], V[0], mask, 0.125)
        assert max_err(O[0].float().cpu().numpy(), want) <= TOL[dtype]
        some = np.isfinite(want_lse)
        got = lse[0].cpu().numpy()
        assert (np.isfinite(got) == some).all() and max_err(got[some], want_lse[some]) <= LSE_TOL[dtype]
