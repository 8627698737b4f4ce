// Plan of an exchange of disjoint pairs of index bits in one in-place sweep
// (k_bit_pairs in k_gates.hip). Plain host C++.
#pragma once

#include <cstdint>

namespace qs {

constexpr int kSwapTileMax = 11;
struct BitPairs {
  int n, low, tile;       // pairs; contiguous tile bits; tile bits (ascending)
  int a[32], b[32];       // the pairs outside the tile
  int bit[kSwapTileMax];  // the tile's bits
  int to[kSwapTileMax];   // tile bit -> its image among the tile's bits
  int moves;              // whether the exchange moves anything inside a tile
};

// image[q] is the bit that bit q's value moves to (image[image[q]] == q).
inline BitPairs plan_bit_pairs(int n, const int* image) {
  // tile bits: the lowest bits with their images, as many as fit
  constexpr int kWant = 10;
  BitPairs g{};
  uint64_t tile = 0;
  for (int q = 0; q < n; ++q) {
    const uint64_t with = tile | (uint64_t(1) << q) | (uint64_t(1) << image[q]);
    if (__builtin_popcountll(with) > kSwapTileMax) break;
    tile = with;
    g.low = q + 1;
    if (__builtin_popcountll(tile) >= kWant) break;
  }
  while (g.low < n && ((tile >> g.low) & 1)) ++g.low;
  int rank[64];
  for (int q = 0; q < n; ++q)
    if ((tile >> q) & 1) {
      rank[q] = g.tile;
      g.bit[g.tile++] = q;
    }
  for (int j = 0; j < g.tile; ++j) {
    g.to[j] = rank[image[g.bit[j]]];
    g.moves |= g.to[j] != j;
  }
  for (int q = 0; q < n; ++q)
    if (!((tile >> q) & 1) && image[q] > q) {
      g.a[g.n] = q;
      g.b[g.n++] = image[q];
    }
  return g;
}

// Workgroups of the sweep, which stride through the 2^(n - tile) tiles: a
// tile each at 34 qubits would be 2^32 threads of 256 to a workgroup, one more
// than a grid dimension takes.
inline unsigned bit_pairs_grid(int n, const BitPairs& g) {
  const uint64_t tiles = uint64_t(1) << (n - g.tile), most = uint64_t(1) << 20;
  return unsigned(tiles < most ? tiles : most);
}

}  // namespace qs
