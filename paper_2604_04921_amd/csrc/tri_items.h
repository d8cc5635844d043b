// Host-side rules of the score kernels: how a batch is cut into work items, and which kernel takes it.  Plain C++: the CPU tests
// compile this file by itself.
#pragma once
#include <stdint.h>

namespace tri {

// Keys per work item of the MFMA score kernels (= keys per entry of `partials` on that path): kFastChunk on large batches (the
// sixteen-lane kernel always), less where that would leave resident workgroups without work (item_keys), kMinChunk at least.
constexpr int kFastChunk = 8192;
constexpr int kMinChunk = 512;
constexpr int kItemCost = 448;
// Waves per workgroup of the sixteen-lane kernel: with more than four query heads per KV head a wave needs more than 128
// registers, so only three waves fit a SIMD; 12-wave workgroups fill them (8-wave ones would leave one of three unused).
constexpr int fast_waves(int G) { return G > 4 ? 12 : 8; }

// Rows that a tile with cnt (1 to 64) of its keys in the sequence is loaded from, a group of `rows` keys at a time: row r of the group that
// begins at key `first` is row min(r, tile_last) from key tile_first on.  Keys past the end repeat the sequence's last one: a slot beyond
// the length need not exist, not even in the block that the last one is in.
constexpr int tile_first(int first, int cnt) { return first < cnt ? first : cnt - 1; }
constexpr int tile_last(int rows, int first, int cnt) { return first + rows < cnt ? rows - 1 : cnt - 1 - tile_first(first, cnt); }

// Eight or more items of kFastChunk keys per CU.
inline bool large_batch(int64_t instances, int max_seq_len, int n_cu)
{
    return instances * (((int64_t)max_seq_len + kFastChunk - 1) / kFastChunk) >= 8 * (int64_t)(n_cu > 0 ? n_cu : 1);
}

// Resident workgroups take items until none is left, so a batch takes about (items per workgroup, rounded up) x (an item's keys
// + the item's own cost in keys: its last tiles, for which there are fewer than the workgroup has waves, and two barriers).  Every
// head-instance is cut into the number of equal pieces that makes this least, in whole tiles of 64; large batches stay with
// kFastChunk.  Measured against about four items per CU, whole steps: one layer of eight x 32768 keys 66.5 -> 57.8 us, four layers
// 126 -> 109, 36 layers 693 -> 674; one layer of eight x 12289, half-split, 150 -> 44.5.  The cost was 768 keys while an item also
// waited for its list entry, table and first rows; with those asked for an item ahead 448 is the better one: 144 x 2176 keys, scores
// and selection, 53.1 -> 47.8 us, 576 129.5 -> 122, 288 x 1400 70.4 -> 62.4, 288 x 3000 97.7 -> 91.6, 288 x 17000, a step, 393 -> 385, the
// others of 27 shapes equal; 256 is equal everywhere.  (Batches that take stretches now among them: stretch_rounds.)  Counting an item's waves without a last tile as half or as whole idle ones takes 288 x
// 2176 from 81.0 to 76.2, but 576 from 122 to 130, 288 x 3000 from 91.6 to 98 and 288 x 32768, a step, from 640 to 658.
inline int item_keys(int64_t instances, int max_seq_len, int n_cu)
{
    constexpr int unit = 64;                            // a tile
    const int64_t workgroups = n_cu > 0 ? n_cu : 1;     // one per CU
    const int64_t len = max_seq_len, fewest = (len + kFastChunk - 1) / kFastChunk;
    if (large_batch(instances, max_seq_len, n_cu)) return kFastChunk;
    constexpr int least = kMinChunk;
    static_assert(kMinChunk % unit == 0, "whole tiles");
    int best = kFastChunk;
    int64_t best_cost = INT64_MAX;
    for (int64_t pieces = fewest; pieces < fewest + 1024; ++pieces) {
        int keys = (int)(((len + pieces - 1) / pieces + unit - 1) / unit * unit);   // kFastChunk at most
        const bool last = keys <= least;
        if (last) keys = least;
        const int64_t items = instances * ((len + keys - 1) / keys);
        const int64_t cost = (items + workgroups - 1) / workgroups * (keys + kItemCost);
        if (cost < best_cost) {
            best_cost = cost;
            best = keys;
        }
        if (last) break;
    }
    return best;
}

// Where work items leave some CUs with more than others, the general MFMA kernel takes stretches instead: the tiles of all head-instances,
// (layer, KV head) by (layer, KV head) and in them sequence by sequence, one after the other, are cut into stretches of equal length (to
// a tile), the same number for every CU, whatever head-instances they begin and end in.  The lengths are known on the device only, which
// cuts a batch there (plan_stretches).
constexpr int kStretchTile = 64;
constexpr int kStretchSeqs = 1024;   // sequences at most: one workgroup counts their tiles
constexpr int64_t kStretchTiles = (int64_t)1 << 30;   // tiles of all head-instances stay below
// Stretches per CU, or 0: work items.  Both sides measured in one process, us with items / with stretches.  Scores and selection of 288 x 2176
// scattered keys 75 / 61, half-split 76 / 61, 576 x 2176 115 / 102, 1152 192 / 179, 2016 305 / 299; scores of 960 ragged post-RoPE
// head-instances up to 20011 684 / 651, of 160 140 / 122; steps on 768 ragged paged ones of 4096 to 65536 1795 / 1761, on 128 375 / 332, on
// 576, 864, 1152 x 32768 1271 / 1244, 1911 / 1850, 2494 / 2430.  Items stay where
//  - a CU has sixteen tiles at most: they begin sooner (8 x 12289 half-split, a step, 33.8 / 35.0, 64 x 2176 29.4 / 30.5);
//  - the batch is large and the sequences are short (4608 x 2176 668 / 673, 9216 half-split 1331 / 1336), or there are more than four query heads (240 x
//    131072 at G = 8 2225 / 2250: less arithmetic to spare for reads in a less even order), or 32 items per CU and more are even enough
//    (2304 x 32768 4885 / 4929).
// 64 tiles in a stretch: neighbouring workgroups then read 1 MB from one another (288 x 32768, a step, 635 with 64, 650 with 96, 649 with 128 and
// 665 with 256; paged 768 1762, 1778, 1778; 576 x 8192 scattered half-split, the other way, 328, 319, 320).
inline int stretch_rounds(int G, int64_t instances, int max_seq_len, int n_cu)
{
    const int64_t cus = n_cu > 0 ? n_cu : 1, tiles = instances * (((int64_t)max_seq_len + kStretchTile - 1) / kStretchTile);
    if (tiles <= 16 * cus || tiles >= kStretchTiles) return 0;
    if (large_batch(instances, max_seq_len, n_cu) && (G > 4 || max_seq_len < kFastChunk || tiles >= 32 * cus * (kFastChunk / kStretchTile))) return 0;
    return (int)((tiles + 64 * cus - 1) / (64 * cus));
}
// tiles of a stretch at least: eight, more where a stretch has more anyway and a row would have more than sixty entries of moments
inline int stretch_least(int64_t instances, int max_seq_len, int64_t stretches)
{
    const int64_t tiles = ((int64_t)max_seq_len + kStretchTile - 1) / kStretchTile, each = instances * tiles / stretches;
    const int64_t few = (tiles + 59) / 60, least = each < few ? each : few;
    return least > 8 ? (int)least : 8;
}
// stretches of `total` tiles; the first tile of stretch i; the stretch that holds a tile
constexpr uint32_t stretch_count(uint32_t total, uint32_t least, uint32_t most)
{
    const uint32_t fit = total / least;
    return total == 0 ? 0 : fit < 1 ? 1 : fit < most ? fit : most;
}
struct Stretches {
    uint32_t count, least, longer;   // the first `longer` ones have least + 1 tiles, the others least
};
constexpr Stretches stretches_of(uint32_t total, uint32_t least, uint32_t most)
{
    const uint32_t count = stretch_count(total, least, most), per = count > 0 ? count : 1;
    return Stretches{count, total / per, total % per};
}
constexpr uint32_t stretch_begin(const Stretches &st, uint32_t i) { return i * st.least + (i < st.longer ? i : st.longer); }
constexpr uint32_t stretch_of(const Stretches &st, uint32_t tile)
{
    const uint32_t split = st.longer * (st.least + 1);
    return tile < split ? tile / (st.least + 1) : st.longer + (tile - split) / st.least;
}
// stretches that a head-instance of max_seq_len keys can lie in, at most
constexpr int stretch_entries(int max_seq_len, int least)
{
    const int tiles = (max_seq_len + kStretchTile - 1) / kStretchTile;
    return tiles < 2 ? 1 : (tiles - 2) / least + 2;
}

// Which kernel takes bf16 keys (item: item_keys() of the batch): that of tri_score_lane.hip, but paged pre-RoPE keys with interleaved pairs
// in items of kFastChunk go to the one that spreads a key over sixteen lanes, with more than four query heads per KV head always, with up
// to four on large batches of short sequences.  The line was drawn where that one was the faster before the other's items followed one
// another without a gap.  It no longer is: whole steps, this kernel / the other, 768 x 4096 to 65536 keys at G = 8 2588 / 2466 us, at G = 5
// 2433 / 2298, 32 x 65536 at G = 8 201 / 197, 512 x 8192 530 / 518; 4608 x 2176 at G = 4 2537 / 2491, at G = 1 2499 / 2447, 3072 x 4096 2048 / 2003.
// tests/test_item_rules.py and test_gpu_sixteen_lanes.py state the line, and test_gpu_precision.py takes this kernel as the yardstick of
// the other's sums: moving it means restating those.
inline bool sixteen_lane_kernel(int G, int item, int64_t instances, int max_seq_len, int n_cu, bool half_split, bool paged, bool rotated)
{
    if (!paged || half_split || rotated || item != kFastChunk) return false;
    return G > 4 || (max_seq_len <= kFastChunk && large_batch(instances, max_seq_len, n_cu));
}

}  // namespace tri
