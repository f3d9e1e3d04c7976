"""The rule that sizes the work items of the tile path (seg_shift), evaluated on the host as the kernels
evaluate it: sga_internal.h is compiled for the host and asked over a grid of sizes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "sga_internal.h"
int main() {
  long long L, nnz;
  int H, dtype, d;
  while (scanf("%lld %lld %d %d %d", &L, &nnz, &H, &dtype, &d) == 5) {
    const sga::WorkspacePlan p = sga::plan_workspace(L, H, nnz, dtype, d);
    printf("%d %lld %lld\n", p.seg_shift, (long long)p.n_work, (long long)p.cap_tparts);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    work = tmp_path_factory.mktemp("rule")
    (work / "rule.hip").write_text(PROGRAM)
    exe = str(work / "rule")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2502_01659_amd", "csrc"),
                    str(work / "rule.hip"), "-o", exe], check=True)

    def ask(cases):
        text = "".join("%d %d %d %d %d\n" % c for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return ask


def _grid(dtype):
    for L in (64, 1000, 3000, 8192, 16301, 24576, 40000, 49152, 65536, 100000, 300001, 1 << 20):
        for permille in (1, 5, 20, 62, 63, 70, 100, 150, 250, 300, 500, 750, 1000):
            for H in (1, 2, 8, 64):
                for d in (64, 128, 256):
                    yield L, L * L * permille // 1000, H, dtype, d


def test_segments_of_dense_masks_fit_their_partial_states(plans):
    """A tile of e edges is cut into at most e / S segments, so a call needs at most nnz / S partial states.
    Items of 2^15 edges are the longest: where their segments fit the 32,768 states there are, those of
    the items chosen fit too (else every cut tile would run on the per-row kernels)."""
    cases = list(_grid(0))
    fitted = 0
    for (L, nnz, H, _, d), (shift, n_work, cap) in zip(cases, plans(cases)):
        assert 12 <= shift <= 15
        if nnz >> 15 <= 32768:
            assert nnz >> shift <= cap, (L, nnz, H, d, shift, cap)
            fitted += nnz >> 15 > 8192
    assert fitted > 0


def test_items_of_thin_and_of_half_precision_masks(plans):
    """Masks below a sixteenth of the pairs, d = 256 and fp16: items are halved from 2^15 (2^18) edges until
    a call has 1024 (4096) of them."""
    for dtype, longest, shortest, items in ((0, 15, 12, 1024), (1, 18, 15, 4096)):
        cases = [c for c in _grid(dtype) if dtype == 1 or c[4] == 256 or c[1] // c[0] < c[0] // 16]
        for (L, nnz, H, _, d), (shift, _, _) in zip(cases, plans(cases)):
            want = longest
            while want > shortest and (nnz * H >> want) < items:
                want -= 1
            assert shift == want, (L, nnz, H, d, shift, want)
