"""The rules that size the work items of the tile path (seg_shift) and the chunks of split rows, evaluated on
the host as the kernels evaluate them: sga_internal.h is compiled for the host and asked over a grid of sizes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "sga_internal.h"
#include "tile_merge.h"
int possible(long long L, int H, long long nnz, int dtype, int d) {
  size_t bytes = sga::plan_workspace(L, H, nnz, dtype, d).total_bytes;
  const size_t shortest = sga::plan_workspace(L, H, nnz, dtype, d, sga::seg_shift_min(dtype)).total_bytes;
  if (bytes < shortest) bytes = shortest;
  return sga::shared_chunks_possible(L, H, d, dtype, bytes);
}
int merge_of(int H) {
  sga::AttnArgs a{};
  a.H = H;
  return (int)sga::merge_tiles(a);
}
bool share(const sga::WorkspacePlan& p, long long nnz, long long L, int H, int d, int dtype, uint32_t rows,
           bool finer = false) {      // rows of two chunks, or of ten
  uint32_t ctr[sga::kNumCounters] = {};
  ctr[sga::kCtrLongRows] = rows;
  ctr[sga::kCtrChunksNeeded] = 2 * rows;
  ctr[sga::kCtrFineNeeded] = finer ? 10 * rows : 0xFFFFFFFF;         // (no room for it)
  ctr[sga::kCtrMaxChunks] = 2;
  ctr[sga::kCtrMaxChunksFine] = 10;
  return sga::shared_chunks(p, nnz, L, H, d, dtype, ctr);
}
int least_shared(const sga::WorkspacePlan& p, long long nnz, long long L, int H, int d, int dtype, bool finer) {
  uint32_t rows = 64;
  while (rows < 8192 && !share(p, nnz, L, H, d, dtype, rows, finer)) rows += 64;
  return (int)rows;
}
int main() {
  long long L, nnz, deg;
  int H, dtype, d;
  while (scanf("%lld %lld %d %d %d %lld", &L, &nnz, &H, &dtype, &d, &deg) == 6) {
    const sga::WorkspacePlan p = sga::plan_workspace(L, H, nnz, dtype, d);
    int chunks, len;
    sga::row_split_shape(deg, p, false, chunks, len);
    printf("%d %lld %lld %d %d %d %d %d %d %d %d %d %d %d %d %d %d\n", p.seg_shift, (long long)p.n_work, (long long)p.cap_tparts, p.l2_chunks, chunks, len,
           sga::tile_parts_in_doubt(p), sga::tile_parts_may_be_in_doubt(dtype, p.total_bytes),
           (int)(sga::leftover_workgroups(L, H) | sga::leftover_chunk_workgroups(H) << 16), merge_of(H), p.l2_chunks != 0 && dtype == SGA_F16 ? -1 : 0,
           sga::l2_chunks(L, d, dtype) && L <= sga::kSharedMaxKeys && share(p, nnz, L, H, d, dtype, 1 << 16),
           possible(L, H, nnz, dtype, d), (int)sga::first_xcd((uint32_t)L, (int)deg),
           (int)(sga::staged_blocks(deg, L, 1) << 16 | sga::staged_blocks(deg, L, 2) << 8 | sga::subtile_blocks(deg, L)),
           least_shared(p, nnz, L, H, d, dtype, false), least_shared(p, nnz, L, H, d, dtype, true));
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

    def ask(cases, first=0, last=6):
        text = "".join("%d %d %d %d %d %d\n" % (c if len(c) == 6 else c + (1,)) for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split())[first:last] for line in out.splitlines()]
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
    for (L, nnz, H, _, d), (shift, n_work, cap, _, _, _) in zip(cases, plans(cases)):
        assert 12 <= shift <= 15
        if nnz >> 15 <= 32768:
            assert nnz >> shift <= cap, (L, nnz, H, d, shift, cap)
            fitted += nnz >> 15 > 8192
    assert fitted > 0


def test_items_are_shortened_only_where_tiles_are_cut(plans):
    """Items are halved from 2^15 (fp16: 2^18) edges until a call has 1024 (4096) of them.  Shorter ones, 2^14
    or 2^13 edges, are taken only with fp32, d = 64 and 128, in masks of a sixteenth of the pairs whose average
    tile has two segments at 2^15 already, and only until a call has 16,384 (4096 before the last halving): a
    band or a block mask would be cut into segments of a few full blocks otherwise."""
    shorter = set()
    for dtype, longest, shortest, items in ((0, 15, 12, 1024), (1, 18, 15, 4096)):
        cases = list(_grid(dtype))
        for (L, nnz, H, _, d), (shift, *_) in zip(cases, plans(cases)):
            want = longest
            while want > shortest and (nnz * H >> want) < items:
                want -= 1
            if shift == want:
                continue
            assert dtype == 0 and d <= 128 and 13 <= shift < want, (L, nnz, H, d, shift, want)
            assert 32 * nnz >= 65024 * L and 16 * nnz >= L * (L - 15), (L, nnz, H, d)
            assert nnz * H >> (shift + 1) < (8192 if shift == 14 else 4096), (L, nnz, H, d, shift)
            shorter.add(shift)
    assert shorter == {13, 14}


def test_rows_cut_by_l2_share_have_all_their_chunks(plans):
    """Chunk c of every such row runs on XCD c % 8 against the c-th part of the keys: with a chunk less, an
    XCD idles and the others' parts no longer fit their L2."""
    cases = [(L, L * L // 10, 1, dtype, 64, deg) for dtype, L in ((0, 7000), (0, 24576), (1, 13000), (1, 30000))
             for deg in (1024, 1025, 1055, 1106, 1121, 1536, 1537, 2047, 2048, 2049, 2458, 5000, L)]
    seen = 0
    for (L, _, _, dtype, _, deg), (_, _, _, n, chunks, length) in zip(cases, plans(cases)):
        assert (chunks - 1) * length < deg <= chunks * length
        if n and deg >= 128 * n:
            assert chunks == n, (L, dtype, deg, chunks)
            seen += 1
    assert seen >= 40


def test_doubtful_calls_are_recognised_by_their_workspace(plans):
    """A call whose partial states may not fit records its split rows in a launch of its own, which the host adds
    by the size of the workspace alone: every such call has one that large, and calls of ordinary size do not."""
    doubtful = ordinary = 0
    for dtype, shift in ((0, 15), (1, 18)):
        least = 32767 << shift
        cases = [(L, nnz, H, dtype, d) for L in (32768, 100000, 1 << 20, 1 << 24) for H in (1, 3, 64) for d in (64, 128, 256)
                 for nnz in (least // 64, least - 1, least, least + (1 << shift), 3 * least) if nnz <= L * L]
        for case, (sure, maybe) in zip(cases + list(_grid(dtype)), plans(cases + list(_grid(dtype)), 6, 8)):
            assert maybe or not sure, case
            assert sure == (case[1] >= least), case
            doubtful += sure
            ordinary += case[1] < least // 2 and case[2] == 1 and not maybe
    assert doubtful > 50 and ordinary > 50


def test_rows_left_over_have_a_chip_full_of_workgroups(plans):
    """Without a plan one launch takes the rows that the tiles leave over and the chunks of split rows.  In a scattered
    mask the one or the other are all rows: a wavefront each, or a chip full; chunk c runs on XCD c % 8, which
    multiples of 8 keep."""
    cases = [(L, L * L // 20, H, dtype, 64) for dtype in (0, 1) for H in (1, 2, 4, 8, 64, 1000)
             for L in (1, 31, 2049, 3001, 5000, 13001, 16384, 24576, 1 << 20)]
    for (L, _, H, _, _), (both,) in zip(cases, plans(cases, 8, 9)):
        rows, chunks = both & 0xFFFF, both >> 16
        assert rows % 8 == 0 and 4 * rows >= min(L, 4096 // H), (L, H, rows)
        assert chunks % 8 == 0 and chunks * H >= 1024, (L, H, chunks)
        assert rows * H <= 2048 + 264 * H and chunks * H <= 2048 + 136 * H, (L, H, rows, chunks)


def test_idle_merge_workgroups_do_not_grow_with_the_heads(plans):
    """A call without a plan launches the merge of tiles that most calls do not have: four rounds of the
    chip's 2,048 workgroups at most, and a workgroup for each row of a tile and head at least."""
    cases = [(4096, 1 << 17, H, 0, 64) for H in (1, 2, 8, 16, 17, 32, 64, 128, 256, 1000, 65535)]
    for (_, _, H, _, _), (tiles,) in zip(cases, plans(cases, 9, 10)):
        assert 1 <= tiles <= 16 and (tiles == 1 or 32 * H * tiles <= 8192), (H, tiles)
        assert H > 16 or tiles == 16


def test_workspaces_tell_whether_split_rows_may_share_key_blocks(plans):
    """Without a plan the host decides by the workspace whether the kernel that shares key blocks is launched, and the
    mask whether it is used.  A workspace sized for a mask that uses it says yes, and so does any larger one (the same
    call in the library's own scratch gives the same bits); fp16 calls whose rows are always cut by L2 share never say
    yes."""
    used = refused = 0
    for dtype in (0, 1):
        for d in (64, 128):
            for H in (1, 2, 3, 8, 32):
                for L in (6300, 7001, 9001, 12001, 13001, 16321, 18017, 20000, 24576, 33000, 44001, 65001, 65536):
                    nnz = sorted({L * (L // f) for f in (31, 30, 29, 27, 26, 25, 24, 20, 19, 18, 17, 14, 10, 8, 5, 3, 2, 1)})
                    found = plans([(L, n, H, dtype, d) for n in nnz], 10, 13)
                    reached = False
                    for n, (never, uses, possible) in zip(nnz, found):
                        assert possible or not uses, (L, n, H, dtype, d)
                        reached |= bool(uses)
                        used += uses
                    if dtype == 1 and all(never for never, _, _ in found):
                        assert not any(possible for _, _, possible in found), (L, H, d)
                        refused += 1
    assert used > 200 and refused > 5


def test_only_rows_of_few_chunks_start_at_an_xcd_of_their_own(plans):
    """Up to four chunks: eight neighbouring rows put the same number of chunks on every XCD.  From five on chunk c
    of every row is on XCD c % 8, so that an L2 sees one part of the keys."""
    for z in list(range(1, 18)) + [24, 25, 63, 64, 100, 1024]:
        starts = [x for x, in plans([(s, 0, 1, 0, 64, z) for s in range(1, 65)], 13, 14)]
        load = [0] * 8
        for first in starts:
            for c in range(z):
                load[(first + c) % 8] += 1
        if z <= 4:
            assert len(set(load)) == 1, (z, load)
        else:
            assert set(starts) == {0}, z


def test_staged_windows_have_room_for_their_blocks_and_no_more(plans):
    """The key blocks that tile_window_wg_kernel and tile_window_kv_kernel copy and meet, counted as they count them,
    for every workgroup and sub-tile of a class of Lc tokens: the most there are is what they are given.  The space also
    holds the output tiles of the four wavefronts, 32 rows of 144 bytes each."""
    shapes = [(Lc, W) for Lc in list(range(1, 70)) + [96, 97, 128, 129, 130, 160, 161, 192, 193, 224, 225, 256, 257, 258, 300, 400, 900, 2000]
              for W in (1, 5, 16, 31, 32, 33, 63, 64, 65, 80, 96, 97, 128, 129, 144, 160, 161, 200, 255, 256) if W < Lc]
    for (Lc, W), (word,) in zip(shapes, plans([(Lc, 0, 1, 1, 64, W) for Lc, W in shapes], 14, 15)):
        most = most_sub = 0
        for q0 in range(0, Lc, 128):
            first, last = max(q0 - W, 0), min(q0 + 127 + W, Lc - 1)
            most = max(most, (last - first) // 32 + 1)
            for u0 in range(q0, min(q0 + 128, Lc), 32):
                lo, hi = max(u0 - W, first), min(u0 + 31 + W, last)
                most_sub = max(most_sub, (hi - first) // 32 - (lo - first) // 32 + 1)
        sub = word & 255
        assert most_sub <= sub <= (Lc + 31) // 32, (Lc, W, sub)
        for sets, staged in ((1, word >> 16), (2, word >> 8 & 255)):
            out = -(-4 * 32 * 144 // (sets * 4096))
            assert max(most, out) <= staged <= max(out, (Lc + 31) // 32), (Lc, W, sets, staged)
            assert staged <= max(out, (127 + 2 * W) // 32 + 1), (Lc, W, sets, staged)


def test_rows_share_key_blocks_where_they_fill_the_chip(plans):
    """The least number of rows of two chunks that share their key blocks (2,048 at any rate): with 64 to a workgroup and
    all heads, the chunks are enough for a quarter (fp32) or all (fp16) of the 512 (d = 64) or 256 (d = 128) places.
    Rows of the finer split, here of ten chunks: fp32 only, and all of the places."""
    L = 32768
    cases = [(L, L * L // 10, H, dtype, d) for H in (2, 4, 8, 16) for dtype in (0, 1) for d in (64, 128)]
    cases.append((L, L * L // 10, 1, 0, 64))
    for (_, _, H, dtype, d), (least, finer) in zip(cases, plans(cases, 15, 17)):
        places = 512 if d == 64 else 256
        assert least == max(2048, 32 * places // (1 if dtype else 4) // H), (H, dtype, d, least)
        assert finer == (8192 if dtype else max(2048, -(-places * 64 // (10 * H * 64)) * 64)), (H, dtype, d, finer)
