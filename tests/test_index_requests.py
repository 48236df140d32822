"""The index requests of the matrix-core kernels run ahead of the work, past the end of the triplet list; the buffer
descriptor has to reject those.  It compares the offset operand of a load with the array's size; an address part in the
scalar offset operand may not take part in the comparison, so none may be there, and the offset may not wrap."""
import os
import re
import subprocess

import pytest

from paper_2511_23227_amd.build import COMMON, CSRC, SOURCES

WALK = r"""
#include <stdio.h>
#include <algorithm>
#include <vector>
#include "mvmr_rows_common.h"
#include "mvmr_stage.h"
#include "mvmr_walk.h"
using namespace pcpp;

// The requests of every wave of weight_any_kernel for a list of n triplets in runs [seg[k], seg[k + 1]); the largest number
// of words past the list, -1: a triplet that is missed or taken twice.
static long walk(const std::vector<long> &seg, long n, long chunk)
{
    long past = 0;
    std::vector<int> taken(n, 0);
    for (long p0 = 0; p0 < n; p0 += chunk)
        for (int wave = 0; wave < 4; ++wave) {
            const uint32_t p_end = (uint32_t)(std::min(p0 + chunk, n) - p0);
            auto end_of = [&](int k) { return (uint32_t)std::min<long>(seg[k + 1] - p0, p_end); };
            int k = 0;
            while (seg[k + 1] <= p0) ++k;
            BatchCursor c{0u, end_of(k), k};
            std::vector<uint32_t> rows;                    // positions whose rows the wave requests, in order
            auto request = [&] { past = std::max(past, p0 + c.pos + 32 - n); };
            auto settle = [&](uint32_t start) { settle_batch(c, start, p_end, (uint32_t)(WINDOW * wave), end_of); };
            auto load_rows = [&] { rows.push_back(c.pos);
                for (uint32_t t = c.pos; t < c.end && t < c.pos + WINDOW; ++t) ++taken[p0 + t]; };
            settle(WINDOW * wave);
            request(); load_rows(); settle(c.pos + WINDOW * 4); request();
            size_t done = 0;
            for (uint32_t p = 0; p < p_end;) {
                const uint32_t q = end_of(k);
                if (q <= p) { ++k; continue; }
                for (uint32_t b = p + WINDOW * wave; b < q; b += WINDOW * 4) {
                    if (rows[done++] != b) return -1;      // the batch in registers is not the one multiplied
                    load_rows(); settle(c.pos + WINDOW * 4); request();
                }
                p = q; ++k;
            }
        }
    for (int t : taken) if (t != 1) return -1;
    return past;
}

int main()
{
    long most = 0;
    unsigned r = 1;
    auto rnd = [&](unsigned m) { r = r * 1664525u + 1013904223u; return (r >> 8) % m; };
    for (long n : {1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 512, 768, 1000, 1537, 5000})
        for (long chunk : {256, 384, 768})
            for (int cells : {1, 2, 27, 216})
                for (int form = 0; form < 4; ++form) {
                    std::vector<long> seg{0};
                    for (int k = 1; k < cells; ++k) seg.push_back(form == 0 ? n : (form == 1 ? n * k / cells : (long)rnd((unsigned)n + 1)));
                    seg.push_back(n);
                    std::sort(seg.begin(), seg.end());
                    const long past = walk(seg, n, chunk);
                    if (past < 0) { printf("n %ld chunk %ld cells %d form %d: wrong walk\n", n, chunk, cells, form); return 1; }
                    most = std::max(most, past);
                }
    const uint64_t list = MAX_BUFFER_BYTES / 4;            // longest list that these kernels take
    printf("%ld words past the list at most\n", most);
    if (most > 287 || (list + 287) * 4 > 0xffffffffull) return 1;
    return index_offset((uint32_t)list, 286u) == (list + 286) * 4 ? 0 : 1;
}
"""


def test_walk_covers_the_list_and_stays_within_its_bound(tmp_path):
    src, exe = tmp_path / "walk.hip", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["hipcc", "--offload-host-only", str(src), "-o", str(exe)] + COMMON, check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("name", ["mvmr_weight.hip", "mvmr_rows_tile.hip"])
def test_whole_offset_is_checked(name, tmp_path):
    out = tmp_path / "kernel.s"
    subprocess.run(["hipcc", "-S", "--offload-device-only", os.path.join(CSRC, name), "-o", str(out)] + COMMON + SOURCES[name],
                   check=True, capture_output=True)
    loads = re.findall(r"^\s*(buffer_load_\S+\s.*)$", out.read_text(), re.M)
    assert len(loads) > 100
    for l in loads:
        operands = re.split(r",\s*", l.split(None, 1)[1])
        assert operands[3].split()[0] == "0" and "offen" in l, l        # destination, offset, descriptor, scalar offset
