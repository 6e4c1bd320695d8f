"""Pair lists whose length reaches 2^31: the prefix sums saturate instead of
wrapping, no entry is written or read outside the list's storage, and a
synchronous call reports the error.

The sums and the slot rule are plain C++ (csrc/listsum.h) and checked on the
host against 64-bit arithmetic; they are exact, so there is no tolerance."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include <algorithm>
#include <cstdio>
#include <vector>
#include "listsum.h"
using namespace pse;
// rows of `rows` entries each, `n` rows, a list of capacity cap: starts by
// chunked scans (chunk totals first, as the kernels do), then every row's
// first, last and limiting entries
static int check(int64_t n, int64_t rows, int64_t cap, int chunk) {
  std::vector<int> start(n + 1);
  std::vector<int> total((n + chunk - 1) / chunk);
  for (int64_t i = 0; i < n; ++i) total[i / chunk] = list_add(total[i / chunk], (int)rows);
  int carry = 0;
  for (int &t : total) {
    const int v = t;
    t = carry;
    carry = list_add(carry, v);
  }
  for (int64_t i = 0; i < n; ++i)
    start[i] = i % chunk ? list_add(start[i - 1], (int)rows) : total[i / chunk];
  start[n] = carry;
  const int limit = list_limit(cap);
  if (limit < 0 || limit > cap || limit > LIST_MAX) return 1;
  int64_t written = 0;
  for (int64_t i = 0; i < n; ++i) {
    const int64_t exact = i * rows, next = exact + rows;
    if (start[i] != std::min<int64_t>(exact, LIST_MAX)) return 2;
    const int end = list_row_end(start[i + 1], limit);
    if (end > limit || end > std::min(next, cap)) return 3;
    // what readers reach: [start, end), a group of 16 looking one group ahead
    if ((int64_t)start[i] + 15 + 16 > INT32_MAX) return 4;
    const int64_t ranks[] = {0, 1, rows / 2, rows - 1, (int64_t)limit - start[i] - 1,
                             (int64_t)limit - start[i]};
    for (int64_t r : ranks) {
      if (r < 0 || r >= rows) continue;
      const int s = list_slot(start[i], r, limit);
      if (s >= 0 ? s != exact + r || s >= limit : exact + r < limit) return 5;
    }
    for (int s = start[i]; s < end; s = end)   // every readable entry was written
      if (list_slot(start[i], end - 1 - start[i], limit) != end - 1) return 6;
    written += std::max(0, end - start[i]);
  }
  if (written != std::min<int64_t>(n * rows, limit)) return 7;
  return (n * rows >= LIST_MAX) == (start[n] == LIST_MAX) ? 0 : 8;
}
int main() {
  for (int64_t n : {1, 2, 1000, 46341, 46342, 65536, 65537, 92700})
    for (int64_t cap : {0l, 16l, 40000l, 2147483392l, 2147483647l, 5000000000l})
      for (int chunk : {4, 1024})
        if (int e = check(n, n - 1, cap, chunk)) {
          printf("n %ld cap %ld chunk %d: %d\n", (long)n, (long)cap, chunk, e);
          return 1;
        }
  const int v[] = {0, 1, 255, LIST_MAX - 1, LIST_MAX};
  for (int a : v)
    for (int b : v)
      for (int c : v)
        if (list_add(list_add(a, b), c) != list_add(a, list_add(b, c)) ||
            list_add(a, b) != std::min<int64_t>((int64_t)a + b, LIST_MAX))
          return printf("sum %d %d %d\n", a, b, c), 1;
  puts("ok");
}
'''


def test_sums_saturate_and_slots_stay_in_the_list(tmp_path):
    src, exe = tmp_path / 't.cpp', tmp_path / 't'
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, 'paper_1709_06946_amd', 'csrc')
    subprocess.run(['g++', '-O1', '-std=c++17', '-Wall', '-fsanitize=undefined',
                    '-fno-sanitize-recover', '-I', inc, '-o', exe, src], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == 'ok\n', r.stdout + r.stderr


# one sphere more than whose N (N - 1) pairs fit 31 bits, all in one place
@pytest.mark.gpu
@pytest.mark.parametrize('precision', [0, 1])
@pytest.mark.parametrize('where,code', [(np.nan, '-4'), (7.0, '-2')])
def test_coincident_spheres_beyond_the_longest_list(precision, where, code):
    import torch

    from gpu_common import dev, host
    from paper_1709_06946_amd import pse
    n, L = 46343, 100.0
    h = pse.PSE(n, L, grid=64, tol=1e-3, precision=precision)
    q = dev(np.random.default_rng(1).normal(size=(n, 11)))
    out = torch.zeros((n, 11), dtype=torch.float64, device='cuda:0')
    with pytest.raises(pse.PSEError, match=code):
        h.mobility_apply(dev(np.full((n, 3), where)), q, out, pse.PSE_REAL)
    # the handle serves the next call
    m = int(np.ceil(n ** (1 / 3)))
    site = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing='ij'), -1).reshape(-1, 3)[:n]
    h.mobility_apply(dev(site * (L / m)), q, out, pse.PSE_REAL)
    assert np.isfinite(host(out)).all()
