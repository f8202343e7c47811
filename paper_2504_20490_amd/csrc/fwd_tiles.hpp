// Which key tiles the waves of a forward work item walk, and in which of the kernel's loops.  Plain index arithmetic,
// usable on the host as well: the order of copies, reads and barriers that follows from it is tested there.
#pragma once
#include "schedule.hpp"

namespace hspmd {

// Iteration kt of a wave computes S(kt+1), which reads K(kt+1) in K buffer (kt+1) & 1, and P V of tile kt, which reads V(kt) in
// V buffer kt & 1; it issues the wave's share of the copies of K(kt+2) into K buffer kt & 1 and of V(kt+1) into V buffer
// (kt+1) & 1.  S(0) is computed ahead of iteration 0.  Iterations 1, 2, ... start with a barrier.
struct FwdTiles {
    int n_passes;    // iterations that every wave of the workgroup passes
    int n_tiles;     // tiles of the wave's team: n_passes, or one fewer where two teams take the item's tiles in turn
    int n_tiles_w;   // tiles that hold a key visible to one of the wave's rows (SPLIT: in the wave's block of the tile)
    int n_plain;     // the first of them that need no mask and have a successor
    int n_spread;    // the first of those whose copies K(kt+2) and V(kt+1) are whole tiles that the workgroup needs
    // Iteration 0 copies K(2) onto K(0), which S(0) has read: with no barrier in front of iteration 0, one has to stand between
    // the two.  (No wave copies a tile that the workgroup does not need, so this is known to all of them alike.)
    constexpr bool reuses_first_k() const { return n_passes > 2; }
};

// Lq rows and L keys of the chunk, key j visible to row r iff j <= r + off; q_row0: first row of the (half) item;
// row_block: the wave's 32 rows; split: the wave takes 32-key block `key_block` of every tile instead of both; tile kt of team
// `team` is tile teams * kt + team of the item
constexpr FwdTiles fwd_tiles(bool split, int Lq, int L, int off, int q_row0, int row_block, int key_block, int teams = 1,
                             int team = 0) {
    constexpr auto lower = [](int a, int b) { return a < b ? a : b; };
    constexpr auto higher = [](int a, int b) { return a > b ? a : b; };
    constexpr int BK = kFwdKTile;
    const int rows = split ? kFwdQTile / 2 : kFwdQTile;
    const auto share = [=](int n) { return (n - team + teams - 1) / teams; };   // the team's part of the first n tiles
    FwdTiles t{};
    // the item's last row sees keys 0 .. kv_end-1
    const int kv_end = higher(0, lower(L, lower(Lq, q_row0 + rows) + off));
    const int item_tiles = (kv_end + BK - 1) / BK;
    t.n_passes = (item_tiles + teams - 1) / teams;
    t.n_tiles = share(item_tiles);
    // the wave's own share: a wave whose rows lie past the end of the chunk computes nothing, and on the diagonal the upper
    // waves of a workgroup see fewer tiles than the lower ones
    const int row0 = q_row0 + row_block * 32;
    const int kv_end_w = row0 < Lq ? higher(0, lower(L, lower(Lq, row0 + 32) + off)) : 0;
    const int visible = (higher(0, kv_end_w - key_block * 32) + BK - 1) / BK;
    t.n_tiles_w = share(visible);
    // tiles that are visible to all of the wave's rows
    const int n_interior_w = split ? higher(0, lower(visible, (lower(row0 + off + 1, L) - key_block * 32 + 32) / BK))
                                   : higher(0, lower(lower(visible, (row0 + off + 1) / BK), L / BK));
    t.n_plain = lower(share(n_interior_w), t.n_tiles_w - 1);
    t.n_spread = higher(0, lower(t.n_plain, lower(t.n_tiles, share(L / BK)) - 2));
    return t;
}

}  // namespace hspmd
