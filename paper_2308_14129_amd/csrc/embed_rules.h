// How an embedding launch (embed_tile.h, k_embed.hip) divides its query rows over workgroups.  Plain functions, evaluated by the
// host, by the kernel and by the tests.
#pragma once

namespace tig {

constexpr int kLeastRows = 8;  // of a tile that is not one of the fewest

constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Rows a workgroup's tile can have.  fp32 products keep the matrix units busy for as long as a tile has rows (172 state
// columns: 18 of the 43 us of a launch over 600 rows, with half of every 16-row block empty), so fp32 tiles also come in 4
// and 8 rows and in 24 (groups of four rows, Prec<TIG_FP32>::mma_four): a step of 200 events of 172 columns 54.3 -> 36.8 us, of
// 500 57.6 -> 46.2, of 1600 92.7 -> 79.1, a training step of 200 224 -> 203.  bf16 products take a fifth of that and are bound by the
// weights' way from L2, which is the same for any number of rows.
// The sums of blocks of 16 rows and of groups of four differ in order.  A tile of 24 rows has both, so its last eight must not be
// rows whose place in the set is a matter of timing: only in a launch with negatives (`negatives`), whose places are fixed, which
// come last and which are a third of its rows or more.
constexpr int kHeights[] = {4, 8, 16, 24, 32, 48};
constexpr bool height_of(bool fp32, bool negatives, int rows)
{
    return rows % 16 == 0 || (fp32 && (rows < 16 || negatives));
}

// The lowest tile whose workgroups, one per compute unit at hand, take `rows` query rows: a workgroup's latency grows
// with its rows.  fp32: evaluated by the kernel, from the rows that the step has (k_embed), because the heights differ in the
// order of a product's sum and with it in the last bits.  bf16: by the host, from the rows that recent steps had; every height
// gives the same bits there.
constexpr int embed_height(bool fp32, bool negatives, int most_mt, int rows, int units)
{
    for (const int h : kHeights)
        if (height_of(fp32, negatives, h) && h < 16 * most_mt && ceil_div(rows, h) <= units)
            return h;
    return 16 * most_mt;
}

// Tiles of at most `height` rows that n_rows rows are dealt over: as many as there are compute units to take them (`units`)
// while each gets eight rows, because the attention phase is as long as the rows of a compute unit are many (a row of
// twenty 444-column slots is 2.7 us of a SIMD: 187 tiles of 32 rows took 30 us there, 223 of 27 take 26), while the
// products cost the same for any number of rows.  Against the fewest tiles, timed in turn: 2000 events of 444-column slots 69.2 -> 65.9 us
// a step; where the attention phase is short it is worth less: 4000 of 208 columns 35.9 -> 35.6, 1000 of a million nodes
// 28.7 -> 28.2.  A launch whose workgroups loop (`loop` of them) gives each equally many.
constexpr int tiles_in_use(int n_rows, int height, int units, int loop)
{
    const int least = ceil_div(n_rows, height), most = ceil_div(n_rows, kLeastRows);
    if (loop > 0 && least > loop)
        return ceil_div(least, loop) * loop;
    const int even = most < units ? most : units;
    return least > even ? least : even;
}

// Workgroups that take the tiles of at most `most` rows in tiles of `height`, one tile each (the tiles beyond those in use
// return).
constexpr int step_workgroups(int most, int height, int units) { return tiles_in_use(most, height, units, 0); }

// The same where the kernel takes the height for its rows, `top` for the most of them: more tiles than compute units are in
// use only at that height.
constexpr int any_workgroups(int most, int top, int units)
{
    const int tiles = ceil_div(most, top) > units ? ceil_div(most, top) : units;
    const int lowest = ceil_div(most, kHeights[0]);
    return tiles < lowest ? tiles : lowest;
}

// A layer of a stack, whose workgroups take tile after tile: no more than there are compute units, and no fewer tiles at a
// time than these could take.  (Without regard to the height, a workgroup for every eight rows, tiles of
// four rows went two by two through half of the workgroups they needed: two layers over 100 events of 172 columns 143 us
// instead of 114, over 300 173 instead of 146; with tiles of 16 rows at least 136 and 166.)
constexpr int layer_workgroups(int most, int top, int units)
{
    const int tiles = any_workgroups(most, top, units);
    return tiles < units ? tiles : units;
}

// Workgroups of `waves` wavefronts that the memory overwrite of `wins` winners has if it has its own.
constexpr int overwrite_workgroups(int wins, int waves)
{
    const int n = ceil_div(wins, 4 * waves);
    return n < 1 ? 1 : (n > 16 ? 16 : n);
}

// The workgroups that prepare the next batch's queries (n_prepare, 0: nothing to prepare) do the overwrite behind that: they
// end long before the tiles do, and every workgroup of its own takes a compute unit from these.  But not if they are fewer
// than it would have of its own, as before a short last batch: of 4000 events with eight left behind them the one workgroup
// took until long after the tiles, 251 us a step of 200 000 nodes with few repeats and 69 with many, with sixteen of its own 60 and 39.
constexpr bool overwrite_beside(int n_prepare, int wins, int waves) { return n_prepare >= overwrite_workgroups(wins, waves); }

}  // namespace tig
