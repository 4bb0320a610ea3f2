"""The row kernel for rows of any start and length, on the CPU: its generated
code, and the packs its index arithmetic gives each row."""
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2607_05804_amd import turnkl as T
from test_compiler_guards import CSRC, FLAGS, HIPCC, ROOT, kernel_budgets, store_data_hazards


@pytest.mark.parametrize("source,kernels", [
    ("rowkl_ragged.hip", 2 * 15),          # packs per thread x dtypes
    ("rowkl_whole.hip", 2 * 2 * (8 + 6)),  # also: whole packs or any start and length
    ("rowfwd.hip", 2 * 2),
])
def test_generated_code(source, kernels, tmp_path):
    """Every instantiation within 256 VGPRs, no AGPRs, no scratch, no store data
    rewritten early (see test_compiler_guards.py)."""
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "ragged.s"
    subprocess.run([HIPCC, *FLAGS, os.path.join(CSRC, source), "-o", str(out)],
                   check=True, capture_output=True, timeout=900)
    asm = out.read_text()
    rows = [b for b in kernel_budgets(asm) if re.search("rowkl_kernel|rowfwd_kernel", b[0])]
    assert len(rows) == kernels
    bad = [b for b in rows if b[1] > 256 or b[2] > 0 or b[3] > 0]
    assert not bad, bad
    assert not store_data_hazards(asm)


DRIVER = r"""
#include <cstdint>
#include <cstdio>
#include "turnkl_internal.h"
// One row tiling per line of input (vocab dtype start stride): packs per
// thread, line mask, threads, and the first pack of each chunk with the end.
int main() {
  long long v, start, stride;
  int dtype;
  while (scanf("%lld %d %lld %lld", &v, &dtype, &start, &stride) == 4) {
    turnkl::RowTiling t = turnkl::whole_tiling(v, dtype, true, (uintptr_t)start, stride);
    if (!t.threads) t = turnkl::ragged_tiling(v, dtype, (uintptr_t)start, stride);
    printf("%d %d %d", t.vpt, t.line_mask, t.threads ? t.threads : 256);
    for (int c = 0; c <= t.n_chunks; ++c)
      printf(" %lld", turnkl::chunk_start(t.packs, t.n_chunks, t.align, c));
    printf("\n");
  }
}
"""


@pytest.fixture(scope="module")
def tilings(tmp_path_factory):
    """ragged_tiling of the built library for a list of (V, es, start, stride)."""
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("tiling")
    (d / "driver.hip").write_text(DRIVER)
    exe = str(d / "driver")
    subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), str(d / "driver.hip"),
                    "-L" + os.path.dirname(T.LIB_PATH), "-l:" + os.path.basename(T.LIB_PATH),
                    "-Wl,-rpath," + os.path.dirname(T.LIB_PATH), "-o", exe],
                   check=True, capture_output=True, timeout=900)

    def ask(cases):
        text = "".join(f"{v} {0 if es == 2 else 1} {start} {stride}\n"
                       for v, es, start, stride in cases)
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout
        return [[int(x) for x in line.split()] for line in out.splitlines()]
    return ask


def test_every_element_belongs_to_one_pack(tilings):
    """For rows at every place within a line: the packs that a chunk's threads
    read lie inside the row, each element counts once over all chunks, and
    only a thread's first or last pack needs a check."""
    rng = np.random.default_rng(5)
    sizes = [8, 9, 15, 16, 17, 63, 65, 511, 513, 4031, 4095, 8191, 16319, 16321, 16383, 16385, 2040, 2041, 2047, 2049, 2056, 4097, 8193, 45055, 45057, 50257,
             90113, 151937] + [int(x) for x in rng.integers(8, 160000, 60)]
    cases = []
    for v in sizes + [4, 5, 7]:
        for es in (2, 4) if v >= 8 else (4,):
            start = es * int(rng.integers(0, 64)) + (1 << 20)
            for pad in (0, int(rng.integers(1, 90)), -v % 64):
                cases.append((v, es, start, (v + pad) * es))
    for (v, es, start, stride), (vpt, mask, size, *lo) in zip(cases, tilings(cases), strict=True):
        epv = 16 // es
        threads = np.arange(size)
        assert (1 if size == 64 else 3) <= vpt <= (8 if size == 64 else 22)
        assert vpt >= 8 or lo[-1] <= 2048
        for row in (0, 1, 2, 5):
            pre = (start + row * stride) & mask
            n_row = (pre + v * es + 15) // 16
            seen = np.zeros(v, np.int64)
            for c in range(len(lo) - 1):
                n = min(lo[c + 1], n_row) - lo[c]
                for k in range(vpt):
                    e = lo[c] * epv - pre // es + (k * size + threads) * epv
                    at = e
                    if k in (0, vpt - 1):
                        at = np.clip(e, 0, v - epv)
                    else:
                        assert (k * size + size - 1) < n
                    assert at.min() >= 0 and at.max() + epv <= v, (v, es, start, stride, row, c, k)
                    j = np.arange(epv)[None, :] - (e - at)[:, None]
                    own = (j >= 0) & (j < epv) & ((k * size + threads) < n)[:, None]
                    np.add.at(seen, (at[:, None] + np.arange(epv)[None, :])[own], 1)
            assert (seen == 1).all(), (v, es, start, stride, row)
