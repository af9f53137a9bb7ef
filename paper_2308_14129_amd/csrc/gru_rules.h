// How the GRU workgroups of a launch (k_gru.hip) divide the column tiles of their winners.  Plain functions, evaluated by the
// host, by the kernel and by the tests.
#pragma once

namespace tig {

// `slices` items per tile of winners, `tiles` column tiles each; `finer`: the items there would be with one column tile fewer
// in each (0: none has one to give).
struct ColumnSlices {
    int slices, tiles, finer;
};

// Tiles of `rows` winners that the slices of wins winners (of `most` entries) are counted for: with an eighth to spare.
constexpr int winner_tiles(int wins, int most, int rows)
{
    const int wide = wins + wins / 8 < most ? wins + wins / 8 : most;
    return wide > rows ? (wide + rows - 1) / rows : 1;
}

// As many slices of n_ct column tiles as keep n_gru workgroups busy with n_tiles > 0 tiles of winners.
constexpr ColumnSlices column_slices(int n_ct, int n_gru, int n_tiles)
{
    int most = n_gru / n_tiles;
    most = most < 1 ? 1 : (most > n_ct ? n_ct : most);
    const int tiles = (n_ct + most - 1) / most;
    return ColumnSlices{(n_ct + tiles - 1) / tiles, tiles, tiles > 1 ? (n_ct + tiles - 2) / (tiles - 1) : 0};
}

// Whether s is column_slices of this number of tiles: its items fit the workgroups, those of the next finer ones don't.
constexpr bool slices_hold(const ColumnSlices &s, int n_gru, int n_tiles)
{
    return (s.slices == 1 || n_tiles * s.slices <= n_gru) && (s.finer == 0 || n_tiles * s.finer > n_gru);
}

}  // namespace tig
