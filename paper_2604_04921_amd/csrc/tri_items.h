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

// Waves per workgroup of the general MFMA kernel: three per SIMD where their registers allow it (168 each).
constexpr int lane_waves(int G, bool paged, bool rotated, bool half_split) { return G <= 4 || !(paged || rotated || half_split) ? 12 : 8; }

// Where work items leave some CUs with more than others, the general MFMA kernel takes stretches instead: the tiles of all head-instances,
// (layer, KV head) by (layer, KV head) and in them sequence by sequence, one after the other, are cut into stretches of equal length (to
// a tile), the same number for every CU, whatever head-instances they begin and end in.  The lengths are known on the device only, which
// cuts a batch there (plan_stretches).
constexpr int kStretchTile = 64;
constexpr int kStretchLong = 64;     // tiles of a stretch where all sequences are max_seq_len long and a CU has several
constexpr int kStretchSeqs = 1024;   // sequences at most: one workgroup counts their tiles
constexpr int64_t kStretchTiles = (int64_t)1 << 30;   // tiles of all head-instances stay below
// Stretches per CU where all sequences are max_seq_len long, and at most, or 0: work items.  Both sides measured in one process, us with items /
// with stretches.  Scores and selection of 288 x 2176 scattered keys 72.7 / 59.9; scores of 1152 x 2176 half-split 178 / 167, of 960 ragged post-RoPE
// head-instances up to 20011 587 / 564, of 114 ragged ones up to 21284 116 / 82; steps on 768 ragged paged ones of 4096 to 65536 1592 / 1548, on 576 and
// 1152 x 32768 1254 / 1226, 2476 / 2433.  Over 260 drawn batches of one to 60 sequences that come here, scores with stretches take 0.99 of items' time
// where all sequences are max_seq_len long, 0.83 where they are ragged, 0.82 where they end far below it.  (What the host cannot see is that items are
// even for the lengths at hand; stretches then cost what they begin with, about 1 us, or up to 4 %: 20 x 4 x 8 x 3854 post-RoPE 136.5 / 141.4, 1152 x 4096 at
// G = 8 298 / 310.)  Items stay where
//  - a CU has sixteen tiles at most: they begin sooner (8 x 12289 half-split, a step, 33.8 / 35.0, 64 x 2176 29.4 / 30.5);
//  - the batch is large and the sequences are short (4608 x 2176 668 / 673, 9216 half-split 1331 / 1336), or there are more than four query heads (240 x
//    131072 at G = 8 2225 / 2250: less arithmetic to spare for reads in a less even order), or 32 items per CU and more are even enough
//    (2304 x 32768 4885 / 4929).
inline int stretch_rounds(int G, int64_t instances, int max_seq_len, int n_cu)
{
    const int64_t cus = n_cu > 0 ? n_cu : 1, tiles = instances * (((int64_t)max_seq_len + kStretchTile - 1) / kStretchTile);
    if (tiles <= 16 * cus || tiles >= kStretchTiles) return 0;
    if (large_batch(instances, max_seq_len, n_cu) && (G > 4 || max_seq_len < kFastChunk || tiles >= 32 * cus * (kFastChunk / kStretchTile))) return 0;
    return (int)((tiles + kStretchLong * cus - 1) / (kStretchLong * cus));
}
// What a row's entries of moments are counted on: tiles of a stretch at least, eight, more where a stretch has more anyway and a row would have more
// than sixty entries.
inline int stretch_least(int64_t instances, int max_seq_len, int64_t stretches)
{
    const int64_t tiles = ((int64_t)max_seq_len + kStretchTile - 1) / kStretchTile, each = instances * tiles / stretches;
    const int64_t few = (tiles + 59) / 60, least = each < few ? each : few;
    return least > 8 ? (int)least : 8;
}
// stretches of `total` tiles, of `least` each at least
constexpr uint32_t stretch_count(uint32_t total, uint32_t least, uint32_t most)
{
    const uint32_t fit = total / least;
    return total == 0 ? 0 : fit < 1 ? 1 : fit < most ? fit : most;
}
// The number of stretches, as the device works it out from the lengths.  Long batches keep the number that max_seq_len asks for as long as that leaves
// 24 tiles to a stretch: where lengths differ, shorter stretches even out better (steps on 768 ragged paged head-instances of 4096 to 65536 keys, 34
// tiles to a stretch, 1552 us, with 60 1569).  Others, and sequences further below it, get as many per CU as make a stretch five rounds of twelve waves
// or eight of eight, one more or less by what a CU needs for them: rounds of its waves, and seven tiles' time for a stretch's beginning and end (1 x 2 x 8
// x 76303 scattered keys at G = 5, 75 tiles per CU, a step, 149.7 us as two stretches of a CU, 142.7 as one; six sequences of 22293 x 8 heads 80.6 / 73.9).
constexpr uint32_t stretch_cost(uint32_t each, uint32_t stretches, uint32_t waves)
{
    const uint32_t tiles = (each + stretches - 1) / stretches;
    return stretches * ((tiles + waves - 1) / waves * waves + 7);
}
// total: tiles of the batch, longest: of its longest sequence; most: what stretch_rounds says, for all CUs.  Fewer than asked for where a
// head-instance would lie in more than `entries` of them, or they would have fewer than eight tiles although every CU has a stretch; a multiple of the
// CUs as long as all have one.
// (With the least length and the number counted on from max_seq_len alone, sequences far below it were cut into the wrong number: 8 x 2176 keys in
// rows of 131072 into 7 stretches, 288 x 2176 into 279, 512 x 1000 in 32768 into 910.  Scores and selection, work items / that / now: 37.7 / 40.6 /
// 23.5 us, 101.6 / 106.2 / 88.9 and 70.0 / 81.9 / 75.6.)
constexpr uint32_t stretches_wanted(uint32_t total, uint32_t longest, uint32_t entries, uint32_t most, uint32_t cus, uint32_t waves)
{
    if (total == 0) return 0;
    const uint32_t room = longest > 2 && entries > 1 ? (longest - 2) / (entries - 1) + 1 : 1;   // (stretch_entries)
    const uint32_t few = total >= 8 * cus ? 8 : total >= cus ? total / cus : 1;
    const uint32_t fit = stretch_count(total, room > few ? room : few, total), each = (total + cus - 1) / cus;
    const uint32_t goal = waves == 12 ? 60 : 64, low = each / goal > 0 ? each / goal : 1;
    uint32_t rounds = most / cus;
    if (rounds < 4 || each < 24 * rounds) rounds = stretch_cost(each, low + 1, waves) < stretch_cost(each, low, waves) ? low + 1 : low;
    const uint32_t want = rounds * cus < most ? rounds * cus : most;
    return fit >= want ? want : fit >= cus ? fit / cus * cus : fit;
}
struct Stretches {
    uint32_t count, least, longer;   // the first `longer` ones have least + 1 tiles, the others least
};
constexpr Stretches stretches_of(uint32_t total, uint32_t least, uint32_t most)
{
    const uint32_t count = stretch_count(total, least, most), per = count > 0 ? count : 1;
    return Stretches{count, total / per, total % per};
}
// the first tile of stretch i; the stretch that holds a tile
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

// Whether the stretch that a workgroup takes behind stretch `id` is its own (id + grid) or the counter's.  The counter is asked an item ahead,
// and a stretch of more pieces than an item holds is two items, so that of workgroups that do as much work some ask a stretch ahead of others: of
// three stretches per CU some took four and others two.  Up to eight per CU, which every batch of full sequences shorter than kStretchLong tiles stays below, all
// are their workgroup's own; beyond, the counter's evenness is worth more than the one stretch that it may get wrong.  Scores, us, two own and the
// others asked for / eight own: 1056 x 2433 half-split scattered keys at G = 8 281 / 236, 2016 x 2176 429 / 392, 1008 x 2562 at G = 5 270 / 226, 1584 x 2502
// interleaved 311 / 288; all own: 1152 x 32768 at G = 4 2057 / 2096, 768 ragged paged ones of 4096 to 65536 1594 / 1621.
constexpr int kOwnStretches = 8;
constexpr bool own_stretch(int id, int grid, int stretches) { return id < grid || stretches <= kOwnStretches * grid; }

// Which kernel takes bf16 keys (item: item_keys() of the batch): that of tri_score_lane.hip, but paged pre-RoPE keys with interleaved pairs
// in items of kFastChunk go to the one that spreads a key over sixteen lanes, with more than four query heads per KV head always, with up
// to four on large batches of short sequences.  It is the slower one there, by 0 - 10 % on long dense sequences and up to twice on short ones
// (scores and selection, this kernel / the other, us: 96 x 8 x 4096 to 65536 keys at G = 8 2147 / 2005, at G = 5 2047 / 1871, 32 x 65536 at G = 8 186 /
// 189, 512 x 8192 332 / 310, scattered 431 / 361, 4608 x 2176 at G = 4 624 / 582, scattered 797 / 673, 4096 x 19 to 300 217 / 112), and the nearer one to
// 64 bits on short dense ones: its raw scores by 1 - 2 % of their error, the final ones by up to 2 % above four heads (1024 keys, G = 8, dense and
// sparse, 9.25e-8 / 9.38e-8 and 9.24e-8 / 9.43e-8; 65536 keys, the other way, 9.85e-8 / 9.66e-8).  These calls keep its sums until the other's are as
// near there.
inline bool sixteen_lane_kernel(int G, int item, int64_t instances, int max_seq_len, int n_cu, bool half_split, bool paged, bool rotated)
{
    if (!paged || half_split || rotated || item != kFastChunk) return false;
    return G > 4 || (max_seq_len <= kFastChunk && large_batch(instances, max_seq_len, n_cu));
}

}  // namespace tri
