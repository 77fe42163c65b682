"""The rule that cuts a table into buckets (bwd_common.h: partition_bits), compiled for the host: what it gives on either side of its
lines, and that the copy of it by which other tests state their digits is the same.  Needs hipcc, no GPU."""
import os
import subprocess

import numpy as np
import pytest

from paper_1906_00091_amd import build as hip_build

from hotpath_util import partition_bits

PROGRAM = """#include "bwd_common.h"
#include <cstdio>
int main() {
  long long nnz, rows;
  int K, d;
  while (std::scanf("%lld %d %d %lld", &nnz, &K, &d, &rows) == 4) std::printf("%d\\n", dlrm::partition_bits(nnz, K, d, rows));
}
"""


@pytest.fixture(scope="module")
def library_bits(tmp_path_factory):
    path = tmp_path_factory.mktemp("bits")
    src, exe = str(path / "bits.hip"), str(path / "bits")
    with open(src, "w") as f:
        f.write(PROGRAM)
    r = subprocess.run([hip_build._hipcc()] + hip_build.HIPCC_FLAGS + ["--cuda-host-only", "-o", exe, src], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def bits(batches):
        r = subprocess.run([exe], input="".join("%d %d %d %d\n" % b for b in batches), capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        return [int(x) for x in r.stdout.split()]
    return bits


# lookups a table, tables, columns, most rows: the bits on the near side of a line and, with a lookup more (or a table or row less),
# on the far side
@pytest.mark.parametrize("batch,bits", [
    # small batches: buckets of 128 pairs whatever the width
    ((2048, 32, 256, 10 ** 6), 4), ((2048, 32, 4, 10 ** 6), 4), ((65536, 1, 64, 10 ** 6), 9),
    # narrow rows: of 224 (192 at eight lanes) where buckets of 128 take six bits (five) or fewer, or ten
    ((224 * 16, 40, 16, 10 ** 6), 4), ((224 * 16 + 1, 40, 16, 10 ** 6), 5), ((112 * 32, 40, 20, 10 ** 6), 5), ((96 * 32, 40, 20, 10 ** 6), 4),
    ((128 * 32, 24, 16, 10 ** 6), 5), ((128 * 32 + 1, 24, 20, 10 ** 6), 6), ((128 * 64, 12, 16, 10 ** 6), 6), ((224 * 32, 12, 16, 10 ** 6), 5),
    ((128 * 64 + 1, 12, 16, 10 ** 6), 7), ((128 * 512, 2, 16, 10 ** 6), 9), ((128 * 512 + 1, 2, 16, 10 ** 6), 9), ((224 * 512 + 1, 1, 16, 10 ** 6), 10),
    ((192 * 512, 1, 20, 10 ** 6), 9), ((192 * 512 + 1, 1, 20, 10 ** 6), 10),
    # wide rows: a bit more from a mean bucket on
    ((240 * 16 - 1, 100, 32, 10 ** 6), 4), ((240 * 16, 100, 32, 10 ** 6), 5), ((400 * 64 - 1, 25, 32, 10 ** 6), 6), ((400 * 64, 25, 32, 10 ** 6), 7),
    ((200 * 64 - 1, 26, 64, 10 ** 6), 6), ((200 * 64, 26, 64, 10 ** 6), 7),
    ((160 * 32 - 1, 50, 128, 10 ** 6), 5), ((3785, 79, 116, 10 ** 6), 5), ((160 * 32, 50, 128, 10 ** 6), 6), ((112 * 64 - 1, 26, 128, 10 ** 6), 6), ((112 * 64, 26, 128, 10 ** 6), 7),
    ((112 * 32 - 1, 50, 256, 10 ** 6), 5), ((112 * 32, 50, 256, 10 ** 6), 6),
    # tables with fewer rows than lookups
    ((8192, 26, 128, 8192), 7), ((8192, 26, 128, 8191), 6), ((168 * 64, 26, 128, 8191), 7), ((300 * 64 - 1, 26, 64, 8191), 6), ((300 * 64, 26, 64, 8191), 7),
    ((8192, 26, 256, 8191), 7),
    # 512 digits and 1024
    ((112 * 256, 6, 128, 10 ** 6), 9), ((400 * 256 - 1, 6, 64, 10 ** 6), 8), ((400 * 256, 6, 64, 10 ** 6), 9), ((336 * 256 - 1, 6, 128, 80000), 8),
    ((336 * 256, 6, 128, 80000), 9), ((112 * 512 - 1, 4, 256, 10 ** 6), 9), ((112 * 512, 4, 256, 10 ** 6), 10), ((224 * 512 - 1, 4, 256, 80000), 9), ((224 * 512, 4, 256, 80000), 10), ((224 * 512, 4, 128, 10 ** 6), 9),
    # never more buckets than the batch fills, never more bits than the row ids have
    ((524288, 64, 128, 10 ** 6), 9), ((120000, 1, 4, 20000), 10), ((120000, 1, 132, 1024), 10), ((120000, 1, 132, 1023), 10), ((120000, 1, 4, 512), 9),
    ((120000, 1, 4, 37), 6), ((120000, 1, 4, 1), 0)])
def test_bits_on_either_side_of_a_line(library_bits, batch, bits):
    per, K, d, rows = batch
    assert library_bits([(per * K, K, d, rows)]) == [bits]


def test_the_copy_in_the_tests_gives_the_library_s_bits(library_bits):
    rng = np.random.default_rng(3)
    batches = []
    for _ in range(20000):
        K = int(np.exp(rng.uniform(0, np.log(200))))
        nnz = int(np.exp(rng.uniform(np.log(1000), np.log(4e7))))
        batches.append((nnz // K * K if rng.random() < 0.5 else nnz, K, 4 * int(rng.integers(1, 65)), int(np.exp(rng.uniform(0, np.log(4e7))))))
    assert [partition_bits(*b) for b in batches] == library_bits(batches)
