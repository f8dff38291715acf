// How the matrix-core score sweeps share out the middle tokens: tiles of 32 tokens to a workgroup, workgroups to a row.  Plain
// arithmetic, for the launch, the workspace's size and a test on the host.  eps: tokens by which a share laps over its neighbours', at
// most 16.
#pragma once
#include <stdint.h>

namespace esa {

constexpr int kMaxTilesPerBlock = 16;    // 512 tokens: 128 KB of LDS (d_c = 128); one load instruction per thread and 8 KB
constexpr int kComputeUnits = 256;       // each holds one such workgroup

constexpr int64_t shares_of(int64_t n, int eps, int64_t tiles) {
  const int64_t own = 32 * tiles - 2 * eps;
  return (n + own - 1) / own;
}
// Whole rounds of workgroups, one per compute unit: as few as hold all rows in the longest shares.  (Full shares of 512 tokens for all
// but the last were 274 workgroups for 140 thousand tokens, a second round for eighteen of them: steps of 512 and 128 tokens there 124.3 ->
// 111.3 us and 76.2 -> 68.9, 300 at 190 thousand 109.1 -> 102.4.  Shares by a row's length alone gave two sequences of 33 thousand tokens 344
// workgroups, four of 20 thousand 628: score of 512 and 64 tokens 36.0 -> 26.9 us, 26.7 -> 16.1.)
constexpr int64_t share_rounds(int64_t n, int eps, int batch) {
  return (batch * shares_of(n, eps, kMaxTilesPerBlock) + kComputeUnits - 1) / kComputeUnits;
}
// Then the shortest shares that need no more rounds, each row rounded up by itself.  (Shares of a round's mean length gave three rows of
// 10900 tokens 258 workgroups, six of 5400 258, seven of 4661 259, a second round for three: score of 512
// tokens 29.3 -> 19.5 us, 33 -> 20.0, 30.1 -> 21.1; seven of 18500 61.4 -> 47.3, nine of 14500, 77 tokens, 36.8 -> 29.7.)
constexpr int64_t share_tiles(int64_t n, int eps, int batch) {
  const int64_t most = share_rounds(n, eps, batch) * kComputeUnits;
  int64_t tiles = 2;                     // even
  while (tiles < kMaxTilesPerBlock && batch * shares_of(n, eps, tiles) > most) tiles += 2;
  return tiles;
}
constexpr int64_t share_count(int64_t n, int eps, int batch) { return shares_of(n, eps, share_tiles(n, eps, batch)); }
// Workgroups of all rows: at least batch * share_count of these sizes and of any fewer tokens and rows, so that a workspace for the longest
// context serves the shorter ones.
constexpr int64_t most_shares(int64_t n, int eps, int batch) {
  const int64_t rounds = share_rounds(n, eps, batch) * kComputeUnits, shortest = batch * shares_of(n, eps, 2);
  return rounds < shortest ? rounds : shortest;
}
// s / n is the upper half of s * inverse_of(n), or one more: s (2^32 - n * inverse) / (n 2^32) <= s / 2^32 < 1 is missing from the quotient.
constexpr uint32_t inverse_of(uint32_t n) { return 0xFFFFFFFFu / n; }
// Whether the second sweep pools over +-eps: the shares then lap over their neighbours', and where that would take another round
// a kernel of its own pools.  (512 tokens over 131072, eps 1: score
// 48.7 us pooled by the sweep, 40.0 so; five rows of 13000, 300 tokens, 35.6 / 22.9.)
constexpr bool sweep_pools(int64_t n, int eps, int batch, int most_eps) {
  return eps <= most_eps && share_rounds(n, eps, batch) == share_rounds(n, 0, batch);
}

}  // namespace esa
