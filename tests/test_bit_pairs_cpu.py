"""The plan of the in-place bit exchange (csrc/bit_pairs.h, plain C++), compiled
here and checked on the host: for every size up to the largest state the grid
stays below the 2^32 threads of one grid dimension, and on small states the
tiles that the workgroups stride through move every amplitude to its place."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <vector>
#include "bit_pairs.h"
using namespace qs;

static uint64_t insert_zero(uint64_t x, int pos) {
  const uint64_t lo = x & ((uint64_t(1) << pos) - 1);
  return lo | ((x ^ lo) << 1);
}

// the sweep of k_bit_pairs, one "workgroup" after another
static std::vector<uint64_t> sweep(int n, const BitPairs& g, unsigned grid) {
  std::vector<uint64_t> v(uint64_t(1) << n);
  std::iota(v.begin(), v.end(), uint64_t(0));
  const uint64_t tiles = uint64_t(1) << (n - g.tile);
  const int size = 1 << g.tile;
  auto at = [&](uint64_t base, int t) {
    for (int j = 0; j < g.tile; ++j) base |= uint64_t((t >> j) & 1) << g.bit[j];
    return base;
  };
  for (unsigned b = 0; b < grid; ++b)
    for (uint64_t w = b; w < tiles; w += grid) {
      uint64_t base = w;
      for (int j = 0; j < g.tile; ++j) base = insert_zero(base, g.bit[j]);
      uint64_t image = base;
      for (int j = 0; j < g.n; ++j) {
        const uint64_t d = ((image >> g.a[j]) ^ (image >> g.b[j])) & 1;
        image ^= (d << g.a[j]) | (d << g.b[j]);
      }
      if (image < base || (image == base && !g.moves)) continue;
      std::vector<uint64_t> x(size), y(size);
      for (int t = 0; t < size; ++t) x[t] = v[at(base, t)], y[t] = v[at(image, t)];
      for (int t = 0; t < size; ++t) {
        int s = 0;
        for (int j = 0; j < g.tile; ++j) s |= ((t >> j) & 1) << g.to[j];
        v[at(image, t)] = x[s];
        if (image != base) v[at(base, t)] = y[s];
      }
    }
  return v;
}

int main() {
  srand(1);
  for (int n = 4; n <= 34; ++n)
    for (int kind = 0; kind < 40; ++kind) {
      int image[64];
      for (int q = 0; q < n; ++q) image[q] = q;
      if (kind == 0) {
        for (int q = 0; q < n; ++q) image[q] = n - 1 - q;
      } else {  // random disjoint pairs, few to many
        for (int k = 0; k < kind; ++k) {
          const int a = rand() % n, b = rand() % n;
          if (a != b && image[a] == a && image[b] == b) image[a] = b, image[b] = a;
        }
      }
      const BitPairs g = plan_bit_pairs(n, image);
      const unsigned grid = bit_pairs_grid(n, g);
      if (uint64_t(grid) * 256 >= uint64_t(1) << 32 || grid < 1) {
        printf("n = %d: grid %u\n", n, grid);
        return 1;
      }
      if (n > 14) continue;
      for (unsigned wg : {grid, 1 + grid / 3, 1u}) {
        const std::vector<uint64_t> v = sweep(n, g, wg);
        for (uint64_t i = 0; i < v.size(); ++i) {
          uint64_t src = 0;
          for (int q = 0; q < n; ++q) src |= ((i >> q) & 1) << image[q];
          if (v[i] != src) {
            printf("n = %d kind %d grid %u: wrong amplitude at %llu\n", n, kind, wg,
                   (unsigned long long)i);
            return 1;
          }
        }
      }
    }
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_plan_of_the_bit_exchange(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2304_14969_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
