"""Batches of the regrouping's rows (csrc/row_batch.h), built for the CPU with
undefined-behaviour and address checks: every row of a length above zero is
moved exactly once and in order, no batch holds more rows than its array, its
scratch or its length allow, and rows of length 0 (the moments of an empty
active pool, 118 of them at SH degree 3, their pointers not null) are left
alone."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "row_batch.h"

// rows: pairs (count, len) of arguments after scratch_words
int main(int argc, char** argv) {
  const long scratch = std::atol(argv[1]);
  std::vector<uint32_t> words(1 << 16);
  std::vector<std::pair<uint32_t*, long>> want, got;
  gs::RowBatcher rows(scratch, [&](const gs::RowBatch& b, int64_t len) {
    if (len < 1 || b.count < 1 || b.count > gs::kPermRows) std::abort();
    if (b.count > 1 && b.count * gs::row_stride(len) > scratch) std::abort();
    for (int r = 0; r < b.count; ++r) got.push_back({b.row[r], (long)len});
    std::printf("%d ", b.count);
  });
  uint32_t* next = words.data();
  for (int a = 2; a + 1 < argc; a += 2) {
    const long len = std::atol(argv[a + 1]);
    for (int r = 0; r < std::atoi(argv[a]); ++r, ++next) {
      rows.add(next, len);
      if (len > 0) want.push_back({next, len});
    }
  }
  rows.flush();
  if (got != want) std::abort();
  return 0;
}
"""


@pytest.fixture(scope="module")
def batches(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_batch")
    (d / "t.cpp").write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=undefined,address", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "paper_2604_02851_amd", "csrc"), str(d / "t.cpp"), "-o", str(d / "t")])

    def run(scratch_words, *rows):
        args = [str(x) for pair in rows for x in pair]
        r = subprocess.run([str(d / "t"), str(scratch_words)] + args, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return [int(x) for x in r.stdout.split()]
    return run


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
def test_empty_active_pool_moves_no_moments(batches, degree):
    rows = 11 + 3 * (degree + 1) ** 2
    n = 9000
    assert sum(batches(12 * n, (rows + 2, n), (2 * rows, 0))) == rows + 2


def test_batches_are_bounded_by_rows_scratch_and_length(batches):
    assert batches(12 * 8 * 1000, (59 + 59, 1000)) == [64, 54]          # eight views: whole batches
    assert batches(12 * 1000, (59, 1000)) == [12, 12, 12, 12, 11]       # one view
    assert batches(64, (3, 1)) == [3]                                   # rows are padded to four words
    assert batches(1004, (3, 1001)) == [1, 1, 1]                        # at least one row at a time
    assert batches(12 * 1000, (5, 1000), (4, 999), (2, 0), (1, 999), (1, 1000)) == [5, 5, 1]
