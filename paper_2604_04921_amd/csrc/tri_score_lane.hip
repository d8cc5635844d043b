// Score kernel for bf16 keys (Sections 4.1-4.2).
//
// A wave takes 64 consecutive slots of a head-instance -- a tile -- in two steps, and scores them against all query heads of the
// group.  The contraction over (band, component) x query head runs on v_mfma_f32_4x4x1_16b_f32: block b of the instruction
// holds lanes 4b..4b+3, its columns are those four lanes' keys (operand B: the lane's own rotated component or modulus of the band
// in turn), its rows four query heads (operand A: the folded table's entries, held in registers by one block and broadcast by the
// instruction to the others).  Lane l of the accumulator ends up with key l's scores of four heads: no cross-lane reduction over keys
// or heads; turned within the blocks (four keys of one head per lane), they leave in one 16-byte store per lane.  Two ways to hand
// out the work (rows_layout()):
//   * half rows: a lane owns one key; step 0 takes bands 0-31 of the 64 keys, step 1 bands 32-63.  Needs the two components of a
//     band in the same half of the row, i.e. interleaved pairs.
//   * rows: step 0 takes keys 0-31 of the tile, step 1 keys 32-63, and two lanes share a key: lane l has its bands 0-31 (l < 32)
//     or 32-63.  The accumulators then hold half of the bands; one lane swap per register adds the halves for both steps'
//     keys.  With whole rows in LDS the pair layouts differ in which pieces a lane reads and in nothing else.
// Half-split pairs need the second; post-RoPE keys, which have the registers for it, gain 1 - 2 % from its whole-row loads (24 x 5 x 8
// ragged head-instances up to 20011 keys, scores only: 848 -> 834 us; 36 x 2 x 8 x 32768, a step: 1261 -> 1245).  Pre-RoPE interleaved
// keys keep the first: equal or 0.7 % slower in position order, 1 - 4 % at sparse or scattered positions.
//
// What it takes to get there:
//   * K rows reach their lanes through LDS: the wave loads half rows (128 bytes per key, whole cache lines) or rows with coalesced
//     16-byte loads, writes them to its own staging area and each lane reads its key back 16 bytes at a time: four
//     bands, or the real or imaginary parts of eight.  The area is XOR-swizzled so that both the writes (16 lanes = 2 half
//     rows or one row) and the reads (16 lanes = 16 keys, one piece) touch every bank once.
//   * Rotation of the key (Appendix B.2): k e^{i w p} = (k e^{i w r}) e^{i w base} with base a position in the middle of
//     the tile's positions and |r| < kLaneRange.  e^{i w |r|} comes from a table in LDS (one 16-byte read per two bands; a
//     negative r flips the sign of the sine), e^{-i w base} is folded into the head-instance's table, for every tile or, rows, for a
//     step: a lane works out one band's sine / cosine pair, hands it to the other three of its block, and forms its entries, four complex
//     products per quad of heads.  A tile (rows: also either step) whose positions span 2 kLaneRange - 1 or more takes the direct path
//     (phase in double, v_sin_f32 / v_cos_f32 per lane and band).  88 positions: with 64, about half of the tiles of a cache that has kept
//     one position in two took the direct path (36 x 2 x 8 x 32768 sparse keys, a step, 1287 -> 1264 us, at G = 8 16 x 8 x 131072 1304 -> 1216,
//     one layer of 8 x 32768 52.0 -> 50.3; dense and scattered ones equal).
//   * The table lies in registers, 12 per quad of heads, a band's four entries in the lanes of one block: a matrix instruction names the
//     block (cbsz, abid).  Read from LDS four bands at a time by every lane instead, it took 48 (G > 4: 96) of a tile's 104 (152) LDS
//     reads, 26 KB of LDS, and the registers of two pieces' entries: 64 x 8 x 131072 keys at G = 8, a step, 4999 -> 4662 us (half of it from
//     the third wave per SIMD that now fits), 9216 x 2176 half-split scattered, scores and selection,
//     1346 -> 1316, one layer of 8 x 12289 half-split 35.5 -> 34.7, 6 x 16 x 8 x 4096 to 65536 paged within what its caches' places cost from process to
//     process, 36 x 8 x 8 x 32768 equal (bound by its reads and the raw scores' writes).  Pre-RoPE kernels that spill vector registers: contiguous interleaved ones
//     above four heads 2 - 4, half-split stretches of up to four heads 2 contiguous, 4 (8 at G = 1) paged, paged interleaved stretches at G = 1 2.
//     Scalar ones go to vector registers in all of them, 4 - 27 in work items, 25 - 56 in stretches, most of them between items (post-RoPE 0 - 2 and 7 - 26).
// The vector instructions of four bands are issued first and their twelve (24) matrix instructions in one run after
// them: a wave that alternates between the two kinds loses about 3.5 clocks per matrix instruction.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "tri_score_common.h"

namespace tri {

namespace {

constexpr int kMaxDevices = 64;

typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kTileKeys = 64;
constexpr int kStageBytes = kTileKeys * 128;                    // 64 half rows or 32 rows, swizzled, no padding
constexpr bool rows_layout(bool rotated, bool half_split) { return rotated || half_split; }
// Where a kernel took caches over from the sixteen-lane one, its fp32 sums are kept as short as that kernel's, which added four
// bands and then those in a tree; sums of 16 (rows) or 64 bands in a chain left scores further from 64-bit ones.  The moduli's products
// (small, of one sign) have a chain of their own, and the others' end after chain_pieces() pieces of four bands.  Distance of final
// scores from 64 bits x 1e7, sixteen-lane kernel / those chains / now, G = 4: half-split dense 1.48 / 1.62 / 1.40,
// scattered 1.32 / 1.73 / 1.29, post-RoPE 1.25 / 1.42 / 1.16, paged interleaved 1.50 / 2.23 / 1.45, scattered 1.30 / 2.14 / 1.27.  Steps
// take the same time (9216 x 2176 half-split scattered keys 1373 us with the longer chains and 1374, dense 1214 and 1212, 768 x 4096 to
// 65536 paged 2067 and 2050); chains of four bands spill (dense 1931), a centred phase on the direct path does as well as shorter chains
// there but costs 2 %.
constexpr bool short_chains(bool paged, bool rotated, bool half_split) { return paged || rotated || half_split; }
constexpr int chain_pieces(bool rotated, bool half_split, bool table) { return rotated || (!half_split && !table) ? 2 : 3; }

// The folded table as the matrix instructions take it: a register per (component, quad of heads, quarter v of the lane's bands) whose lane
// (b, j) holds head 4 q + j's entry of band table_band(lane, v).  An instruction broadcasts one block's four lanes to all sixteen blocks
// (half rows) or to the eight of its half of the wave (rows).
constexpr int table_block(bool rows, int band) { return rows ? 8 * (band / 32) + band % 8 : band % 16; }   // the block that holds a band
constexpr int table_quarter(bool rows, int band) { return rows ? band % 32 / 8 : band / 16; }
constexpr int kTabQuad = 64 * 4;                                // floats per (component, quad of heads): four a lane
constexpr int lane_quads(int G) { return (G + 3) / 4; }
constexpr int lane_slots(int G) { return G > 4 ? 2 : 4; }   // pieces of an item: as many tables as LDS has room for
constexpr int lane_lds_bytes(int G, bool paged, bool rotated, bool half_split, bool stretch)
{
    return (rotated ? 0 : kLanePhasorBytes) + (stretch ? lane_slots(G) : 1) * 3 * lane_quads(G) * kTabQuad * 4 + lane_waves(G, paged, rotated, half_split) * kStageBytes;
}
// acc + (four heads' entries of block BLOCK, lanes 4 BLOCK ..) x (every lane's key): lane l of the result holds key l's products
template <bool ROWS, int BLOCK>
__device__ __forceinline__ float4v head_products(float entries, float key, float4v acc)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(entries, key, acc, ROWS ? 3 : 4, BLOCK, 0);
}
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}
// v of lane 4 b + K in all four lanes of a block; v of lane ^ 1, ^ 2
template <int CTRL>
__device__ __forceinline__ float quad_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
constexpr int quad_same(int k) { return k * 0x55; }
constexpr int kQuadXor1 = 0xb1, kQuadXor2 = 0x4e;

// Byte offset of 16-byte piece p of key k in a wave's staging area, such that 16 lanes that hold whole rows or half rows (the
// writes) or one piece of 16 keys (the reads) fall into 16 different groups of four banks.  Half rows: rows k and k ^ 1 swap
// places when bit 3 of k is set and the piece index is XORed with k & 7; rows: the piece index is XORed with k & 15.
template <bool ROWS>
__device__ __forceinline__ int stage_offset(int k, int p)
{
    return ROWS ? (k << 8) + ((p ^ (k & 15)) << 4) : ((k ^ ((k >> 3) & 1)) << 7) + ((p ^ (k & 7)) << 4);
}

// Smallest or largest of lanes 0-31 and of lanes 32-63, by DPP.
struct HalfExtremes {
    int v[2];
};
template <bool MAX>
__device__ __forceinline__ HalfExtremes half_extremes(int v)
{
    auto step = [&](auto ctrl, auto rows) {
        const int t = __builtin_amdgcn_update_dpp(v, v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
        v = MAX ? max(v, t) : min(v, t);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});   // row_shr 1, 2, 4, 8
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});   // row_bcast 15 into rows 1, 3
    return {{__builtin_amdgcn_readlane(v, 31), __builtin_amdgcn_readlane(v, 63)}};
}

// ROTATED: the keys are stored post-RoPE (no rotation, no positions).  PAGED: block_size >= 16.  HALF: half-split pairs.
template <int G, bool PAGED, bool ROTATED, bool HALF, bool STRETCH>
__global__ __launch_bounds__(lane_waves(G, PAGED, ROTATED, HALF) * 64) void score_lane_kernel(ScoreArgs a)
{
    constexpr int NG = lane_quads(G), W = lane_waves(G, PAGED, ROTATED, HALF), kThreads = W * 64;
    constexpr int P = STRETCH ? lane_slots(G) : 1, kSlot = 3 * NG * kTabQuad;   // pieces of an item, floats of a piece's table
    constexpr bool ROWS = rows_layout(ROTATED, HALF), kShortChains = short_chains(PAGED, ROTATED, HALF);
    extern __shared__ __align__(16) char lds[];
    constexpr int kSums = 2 * 4 * NG;
    __shared__ double red[W][P * kSums];
    __shared__ double lds_rev[kBands];                    // omega_f / 2pi
    constexpr int kPieceInts = 8;   // lh, sequence, first tile, entry of the moments, end of the keys, end of the item's tiles, rotation
    __shared__ __align__(16) int lds_piece[3][P][kPieceInts];   // an item's pieces,
    __shared__ int lds_size[3][2];                              // its tiles and how many pieces

    const CacheView &c = a.c;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 3, b = lane >> 2;                // column (query head within a quad) and block of the lane

    char *const ph_base = lds;                                                  // phasor table (absent when ROTATED)
    float *const item_tab = reinterpret_cast<float *>(lds + (ROTATED ? 0 : kLanePhasorBytes));   // the pieces' tables, [piece][component][quad][lane][v]
    char *const stage = reinterpret_cast<char *>(item_tab + P * kSlot) + wave * kStageBytes;   // this wave's rows

    // the phasor table: all of a thread's entries asked for at once, stored further down
    constexpr int kPhasors = ROTATED ? 0 : (kLanePhasorBytes / 16 + kThreads - 1) / kThreads;
    uint4v ph[kPhasors + 1];
#pragma unroll
    for (int k = 0; k < kPhasors; ++k) ph[k] = reinterpret_cast<const uint4v *>(a.phasors)[min(tid + k * kThreads, kLanePhasorBytes / 16 - 1)];
    const double rev = a.band_rev[tid % kBands];
    // entries of heads that do not exist (G not a multiple of four) stay zero for the whole launch
    if constexpr (G % 4 != 0)
        for (int k = tid; k < P * kSlot; k += kThreads) item_tab[k] = 0.f;

    // (constant for the whole launch, unlike the counter in front of it: scalar loads)
    typedef const __attribute__((address_space(4))) int32_t *ConstInts;
    const ConstInts work_list = (ConstInts)a.work, seq_len = (ConstInts)c.seq_len;
    const int per_lh = work_list[1];   // items, or tiles, of a (layer, KV head)
    const Stretches cut = STRETCH ? stretches_of((uint32_t)per_lh * (uint32_t)(a.n_layers * c.n_kv_heads), 1, (uint32_t)work_list[2]) : Stretches{};
    const int n_items = STRETCH ? (int)cut.count : per_lh * a.n_layers * c.n_kv_heads;
    // A workgroup's first two items are its own: a permutation of its index, and the same behind the grid's first ones; the others come
    // from the counter (own_stretch: those of a few stretches are all its own).
    const int first_item = (int)(((uint32_t)blockIdx.x * (uint32_t)a.first_mult) % gridDim.x);
    int later_item = 0;   // (thread 0's) the counter's answer for the item after the next
    // (zero, which the compiler does not know to be uniform: it would wait for the counter's answer at once to hand it to all lanes)
    int own_zero = 0;
    asm volatile("" : "+v"(own_zero));

    const uint32_t slot_bytes = (uint32_t)c.stride_slot * 2u;
    // loads: instruction t of a step brings its keys 8t .. 8t+7, eight lanes (128 contiguous bytes) per key, or 4t .. 4t+3, sixteen
    // lanes (256 bytes) per key
    constexpr int kLoadKeys = ROWS ? 4 : 8;   // keys per load instruction
    const int ld_key = ROWS ? lane >> 4 : lane >> 3, ld_piece = ROWS ? lane & 15 : lane & 7;
    const int bmask = PAGED ? (1 << c.block_shift) - 1 : 0;
    uint32_t ld_off = (uint32_t)ld_key * slot_bytes + (uint32_t)ld_piece * 16u;   // the lane's part of a load address
    uint32_t ld_more[16 / kLoadKeys];   // that of each instruction of sixteen keys (paged, where registers allow: 0.3 % at G = 8)
#pragma unroll
    for (int i = 0; i < 16 / kLoadKeys; ++i) ld_more[i] = ld_off + (uint32_t)(kLoadKeys * i) * slot_bytes;
    // where the lane writes its loaded pieces (rows: load t at 1024 t, with 4 (t % 4) XORed into the piece index; half rows: at
    // 1024 t plus one of two offsets, by the parity of t) and reads its key's (its piece p lies at st_rd ^ (p << 4))
    const int hh = ROWS ? lane >> 5 : 0;   // rows: which half of the bands
    const int st_wr0 = stage_offset<ROWS>(ld_key, ld_piece), st_wr1 = ROWS ? 0 : stage_offset<ROWS>(8 + ld_key, ld_piece) - 1024;
    const int st_rd = ROWS ? stage_offset<ROWS>(lane & 31, HALF ? 4 * hh : 8 * hh) : stage_offset<ROWS>(lane, 0);
    // the band whose phase the lane works out when a base is folded in: table_band(lane, j)
    const int my_band = ROWS ? 32 * hh + 8 * j + (b & 7) : 16 * j + b;

    // A piece: consecutive tiles of a head-instance.  An item: one piece (a chunk from the list), or the next P at most of a stretch.
    // Everything here is wave-uniform, and of a stretch as little as possible is held: a piece is worked out again where it is needed again.
    struct Walk {
        uint32_t lh;                // layer << 16 | KV head
        int s, off, entry, rem;     // `rem` tiles from tile `off` of sequence s on; which of the head-instance's entries the first piece has
    };
    struct Piece {
        const char *krow;
        const int32_t *prow, *bt;
        int inst, off, c_end, t0, t1, slot, rot;   // from tile off on, keys up to c_end; its tiles are the item's [t0, t1), in an order rotated by rot
    };
    // what follows the piece that begins at w and has n tiles
    auto behind = [&](Walk w, int n) {
        w.rem -= n;
        w.off = w.entry = 0;
        if (++w.s == c.n_seqs) {
            w.s = 0;
            w.lh = (w.lh & 0xffffu) + 1u == (uint32_t)c.n_kv_heads ? (w.lh & 0xffff0000u) + 0x10000u : w.lh + 1u;
            if ((int)(w.lh >> 16) >= a.n_layers) w.rem = 0;
        }
        if constexpr (!STRETCH) w.rem = 0;
        return w;
    };
    // w moved to where its next piece begins (past empty sequences); the piece's length in tiles (0: there is none), and where its keys end
    auto settle = [&](Walk &w, int &c_end) {
        int len = clamp_len(seq_len[w.s], c.max_seq_len), n = (len + kTileKeys - 1) / kTileKeys - w.off;
        while (n <= 0 && w.rem > 0) {
            w = behind(w, 0);
            len = clamp_len(seq_len[w.s], c.max_seq_len);
            n = (len + kTileKeys - 1) / kTileKeys;
        }
        n = max(min(n, w.rem), 0);
        c_end = min(len, (w.off + n) * kTileKeys);
        return n;
    };
    auto instance_of = [&](uint32_t lh, int s) { return ((int)(lh >> 16) * c.n_seqs + s) * c.n_kv_heads + (int)(lh & 0xffffu); };
    auto piece_from = [&](uint32_t lh, int s, int off, int c_end, int t0, int t1, int slot, int rot) {
        const int l = (int)(lh >> 16), h = (int)(lh & 0xffffu);
        Piece p;
        p.inst = instance_of(lh, s);
        p.krow = (const char *)c.k + ((int64_t)l * c.stride_layer + (int64_t)h * c.stride_head) * 2 + (PAGED ? 0 : (int64_t)s * c.stride_sb * 2);
        p.prow = c.pos + (int64_t)l * c.pos_stride_layer + (int64_t)h * c.pos_stride_head + (PAGED ? 0 : (int64_t)s * c.pos_stride_sb);
        p.bt = PAGED ? c.block_table + (int64_t)s * c.max_blocks : nullptr;
        p.off = off, p.c_end = c_end, p.t0 = t0, p.t1 = t1, p.slot = slot, p.rot = rot;
        return p;
    };
    // Item i takes a piece's tiles in an order rotated by 5 i: workgroups that run side by side work on neighbouring
    // chunks and would otherwise read the same offset of their chunk (addresses one chunk apart) at the same
    // time, all the way through.  Measured on 36 x 16 x 8 head-instances of 32768 keys in one process: 8.13 ->
    // 7.97 ms and 7.74 -> 7.53 ms (steps of 2 to 6 tiles alike, 1, 11 to 37 less, 7 and 9 little or nothing); with more
    // than four query heads the kernel is bound by its arithmetic and the rotation costs 0.7 %, so it stays off.
    auto rotation = [&](int id, int n) { return G <= 4 ? (int)(((unsigned)id * 5u) % (unsigned)max(n, 1)) : 0; };
    // where item id (of a stretch: its first) begins
    auto start_of = [&](int id) {
        if constexpr (STRETCH) {
            const ConstInts plan = (ConstInts)a.stretches;
            if (id < a.n_first) {   // (its length is 0 where there are fewer stretches)
                const ConstInts st = plan + kStretchSeqs + kStretchInts * id;
                return Walk{(uint32_t)st[0], st[1], st[2], st[3], st[4]};
            }
            if (id >= n_items) return Walk{};
            const StretchStart st = stretch_start((uint32_t)id, cut, (uint32_t)per_lh, c.n_seqs, (uint32_t)c.n_kv_heads, plan);
            return Walk{(uint32_t)st.lh, st.s, st.off, st.entry, st.tiles};
        }
        if (id >= n_items) return Walk{};
        const int lh = id / per_lh, wi = id - lh * per_lh, l = lh / c.n_kv_heads, per = a.chunk_keys / kTileKeys;
        const int s = work_list[kWorkHeader + 2 * wi], chunk = work_list[kWorkHeader + 2 * wi + 1];
        return Walk{(uint32_t)l << 16 | (uint32_t)(lh - l * c.n_kv_heads), s, chunk * per, chunk, per};
    };
    // One wave lists an item's pieces, an item ahead of all others, which read them from LDS.  (Every wave for itself: a wait for the
    // length and some sixty scalar instructions per piece, three times an item.)  Leaves w behind them.
    auto list_piece = [&](int buf, int k, const Walk &w, int c_end, int t1, int rot) {
        if (lane != 0) return;
        int *const o = lds_piece[buf][k];
        *reinterpret_cast<int4 *>(o) = make_int4((int)w.lh, w.s, w.off, w.entry);
        *reinterpret_cast<int4 *>(o + 4) = make_int4(c_end, t1, rot, 0);
    };
    auto list_size = [&](int buf, int n_tiles, int n_pieces) {
        if (lane == 0) lds_size[buf][0] = n_tiles, lds_size[buf][1] = n_pieces;
    };
    auto list_item = [&](Walk &w, int id, int buf) {
        int n_tiles = 0, n_pieces = 0;
#pragma unroll 1
        for (; n_pieces < P && w.rem > 0; ++n_pieces) {
            int c_end;
            const int n = settle(w, c_end);
            if (n == 0) break;
            n_tiles += n;
            list_piece(buf, n_pieces, w, c_end, n_tiles, rotation(id, n));
            w = behind(w, n);
        }
        list_size(buf, n_tiles, n_pieces);
    };
    auto spent = [&](const Walk &w) { return !STRETCH || w.rem <= 0; };
    struct Item {
        int buf, n_tiles, n_pieces;   // n_tiles 0: none
    };
    auto item_in = [&](int buf) {
        return Item{buf, __builtin_amdgcn_readfirstlane(lds_size[buf][0]), __builtin_amdgcn_readfirstlane(lds_size[buf][1])};
    };
    auto listed = [&](int buf, int k, int i) { return __builtin_amdgcn_readfirstlane(lds_piece[buf][k][i]); };
    // the piece that holds the item's tile t (t < n_tiles)
    auto piece_of = [&](const Item &it, int t) {
        int k = 0, t0 = 0, t1 = STRETCH ? listed(it.buf, 0, 5) : it.n_tiles;
#pragma unroll 1
        while (k + 1 < P && t >= t1) {
            ++k;
            t0 = t1;
            t1 = listed(it.buf, k, 5);
        }
        return piece_from((uint32_t)listed(it.buf, k, 0), listed(it.buf, k, 1), listed(it.buf, k, 2), listed(it.buf, k, 4), t0, t1, k, listed(it.buf, k, 6));
    };
    // A tile: where its rows, positions and block-table entries are, its first slot, its keys that exist.
    struct Tile {
        const char *krow;
        const int32_t *prow, *bt;
        int n0, cnt;
    };
    // tile t of the item, which lies in piece p
    auto tile_of = [&](const Piece &p, int t) {
        const int t0 = STRETCH ? p.t0 : 0, n = p.t1 - t0, u = t - t0 + p.rot, n0 = (p.off + (u >= n ? u - n : u)) * kTileKeys;
        return Tile{p.krow, p.prow, p.bt, n0, min(kTileKeys, p.c_end - n0)};
    };

    // what step `half` takes of the tile at slot n0 (cnt keys exist): eight 16-byte loads per lane.  For a whole tile every address is a
    // wave-uniform pointer (sixteen keys never straddle a block) plus the lane's constant offset; in the last, partial tile a key past
    // the end repeats the last one.  Kernels short of registers keep that constant and cut it off at the last row (tile_first,
    // tile_last), a minimum per load, instead of a row number per load: half-split contiguous ones spill six registers more without it (9216 x
    // 2176 scattered, scores and selection, 1301 / 1306 us); the others lose 0.3 us with it on small calls.  Paged ones go that way with every tile (a
    // branch of its own for the last one took registers that were spilled: 1.5 - 2 % half-split, 0.5 % interleaved).
    // Paged caches: lane j of `btv` holds the physical block of keys n0 + 16 j .. + 15 (load_blocks; a block holds
    // 16 slots or more), asked for a tile ahead like the positions, so that no load here waits for a block-table
    // entry.
    auto load_half = [&](const Tile &ti, int half, uint4(&kd)[8], int btv) {
        const int first_key = ROWS ? 32 * half : 0, byte = ROWS ? 0 : 128 * half;
        constexpr int kPer16 = 16 / kLoadKeys;   // instructions per sixteen keys
        constexpr bool kMinForm = HALF && !ROTATED && G <= 4;   // (of the contiguous kernels)
        // where key k of the tile is, which lies in the block of key `in`
        auto row = [&](int in, int k) {
            const int n = ti.n0 + k;
            if constexpr (PAGED) {
                const int blk = __builtin_amdgcn_readlane(btv, in / 16);
                return ti.krow + (int64_t)blk * c.stride_sb * 2 + (int64_t)(n & bmask) * slot_bytes + byte;
            }
            return ti.krow + (int64_t)n * slot_bytes + byte;
        };
        // the instructions t0 .. of a group of kRows keys, any of which may lie past the end
        auto load_group = [&](int t0, auto rows) {
            constexpr int kRows = decltype(rows)::value;
            const int first = first_key + kLoadKeys * t0;
            const char *p = row(first, tile_first(first, ti.cnt));
            const uint32_t last = (uint32_t)tile_last(kRows, first, ti.cnt) * slot_bytes + (uint32_t)ld_piece * 16u;   // (32 rows fit 32 bits: mfma_path)
#pragma unroll
            for (int i = 0; i < kRows / kLoadKeys; ++i) {
                if constexpr (PAGED && G > 4) {
                    asm volatile("" : "+v"(ld_more[i]));   // keeps (scalar base + 32-bit lane offset) addressing
                    kd[t0 + i] = load_stream16(p + min(ld_more[i], last));
                } else {
                    asm volatile("" : "+v"(ld_off));
                    kd[t0 + i] = load_stream16(p + min(ld_off + (uint32_t)(kLoadKeys * i) * slot_bytes, last));
                }
            }
        };
        if constexpr (PAGED) {
#pragma unroll
            for (int t = 0; t < 8; t += kPer16) load_group(t, std::integral_constant<int, 16>{});
        } else if (ti.cnt == kTileKeys) {
#pragma unroll
            for (int t = 0; t < 8; t += kPer16) {
                const char *p = row(0, first_key + kLoadKeys * t);
#pragma unroll
                for (int i = 0; i < kPer16; ++i) {
                    asm volatile("" : "+v"(ld_off));   // (see above)
                    kd[t + i] = load_stream16(p + (int64_t)(kLoadKeys * i) * slot_bytes + ld_off);
                }
            }
            // The compiler would let the branches end in one common last load, whose registers it takes for pending: it then waits for
            // the seven loads just issued before it issues the eighth, once per tile.
            asm volatile("; whole tile");
        } else {
            if constexpr (kMinForm) {
                load_group(0, std::integral_constant<int, 32>{});
            } else {
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const uint32_t k = min(first_key + kLoadKeys * t + ld_key, ti.cnt - 1);   // (64 rows fit 32 bits: mfma_path)
                    kd[t] = load_stream16(row(0, 0) + (k * slot_bytes + (uint32_t)ld_piece * 16u));
                }
            }
            asm volatile("; last tile");
        }
    };
    auto load_blocks = [&](const Tile &ti) -> int {
        if constexpr (!PAGED) return 0;
        return ti.bt[(ti.n0 + min(16 * (lane & 3), ti.cnt - 1)) >> c.block_shift];
    };
    auto load_pos = [&](const Tile &ti, int btv) -> int {
        if constexpr (ROTATED) return 0;
        const int k = min(lane, ti.cnt - 1), n = ti.n0 + k;
        if constexpr (PAGED) return ti.prow[(int64_t)__shfl(btv, k >> 4, 64) * c.pos_stride_sb + (n & bmask)];
        return ti.prow[n];
    };
    auto stage_half = [&](const uint4(&kd)[8]) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int at = ROWS ? st_wr0 ^ (64 * (t & 3)) : (t & 1) ? st_wr1 : st_wr0;
            *reinterpret_cast<uint4 *>(stage + at + 1024 * t) = kd[t];
        }
    };

    // The folded table of a head-instance, [F][3][G], spread over the workgroup's threads.
    constexpr int kTabEach = (kBands * 3 * G + kThreads - 1) / kThreads;
    uint4 kd[8];
    int pos_next = 0, bt_cur = 0, bt_next = 0;
    const bool whole_lines = (c.max_seq_len & 31) == 0 && ((uintptr_t)a.raw & 127) == 0;   // a tile's 64 scores start on a 128-byte line
    // Items follow one another without a gap: while one is scored, the next one's table entries (of each of its pieces) and every wave's first
    // tile of it are on their way, so that between two items there are two barriers and no wait for memory.  (Asking for an item, its chunk, its
    // rows and its table one after the other cost about as much as twelve tiles of an idle CU.)  9216 x 2176 keys, scores and selection:
    // 1385 -> 1335 us half-split scattered, 1227 -> 1173 in slot order; 288 x 2176 interleaved scattered 90.7 -> 78.8, in slot order 83.5 -> 68.5;
    // 64 x 8 x 131072 at G = 8, a step, 5218 -> 5004
    // (with the waits that load_half and the stores below speak of).
    float tab[P][kTabEach];
    auto load_table = [&](int i, int inst) {
        const float *tbl = a.table + (int64_t)inst * (kBands * 3 * G);
#pragma unroll
        for (int k = 0; k < kTabEach; ++k) tab[i][k] = tbl[min(tid + k * kThreads, kBands * 3 * G - 1)];
    };
    auto load_tables = [&](const Item &it) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (i >= it.n_pieces) break;
            load_table(i, instance_of((uint32_t)listed(it.buf, i, 0), listed(it.buf, i, 1)));
        }
    };
    auto store_tables = [&](const Item &it) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (i >= it.n_pieces) break;
#pragma unroll
            for (int k = 0; k < kTabEach; ++k) {
                const int e = tid + k * kThreads, f = e / (3 * G), comp = e / G - 3 * f, g = e % G;
                if (kBands * 3 * G % kThreads != 0 && e >= kBands * 3 * G) break;
                item_tab[i * kSlot + ((comp * NG + g / 4) * 64 + 4 * table_block(ROWS, f) + g % 4) * 4 + table_quarter(ROWS, f)] = tab[i][k];
            }
        }
    };
    // the lane's four entries of a component and quad of heads
    const float *piece_tab = item_tab;
    auto table_of = [&](int comp, int q) { return *reinterpret_cast<const float4v *>(piece_tab + ((comp * NG + q) * 64 + lane) * 4); };
    auto load_first = [&](const Tile &ti) {
        bt_cur = load_blocks(ti);
        pos_next = load_pos(ti, bt_cur);   // (ahead of the rows: needed first)
        load_half(ti, 0, kd, bt_cur);
    };
    // The first item: every wave for itself.
    constexpr int kLister = W - 1;      // the wave that most often has a tile less than others
    Walk rest = start_of(first_item);   // (the listing wave's) where what it lists next begins
    int id = first_item;                // (the listing wave's) and of which item or stretch that is
    Piece at{};                         // that of the wave's tile
    Item cur{0, 0, 0};
    {
        Walk &w = rest;
        bool found = false;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (w.rem <= 0) break;
            int c_end;
            const int n = settle(w, c_end);
            if (n == 0) break;
            load_table(i, instance_of(w.lh, w.s));
            const int rot = rotation(id, n);
            if (!found) at = piece_from(w.lh, w.s, w.off, c_end, cur.n_tiles, cur.n_tiles + n, i, rot);
            cur.n_tiles += n;
            if (wave == kLister) list_piece(0, i, w, c_end, cur.n_tiles, rot);
            cur.n_pieces = i + 1;
            found = found || wave < cur.n_tiles;
            w = behind(w, n);
        }
    }
    if (cur.n_tiles == 0) return;   // (the whole workgroup)
    load_first(tile_of(at, min(wave, at.t1 - 1)));   // (a wave without a tile: no branch that the wait for the table would have to allow for)
    if (wave == kLister) {
        list_size(0, cur.n_tiles, cur.n_pieces);
        if (spent(rest)) id = (int)gridDim.x + first_item, rest = start_of(id);
        list_item(rest, id, 1);
    }
#pragma unroll
    for (int k = 0; k < kPhasors; ++k) reinterpret_cast<uint4v *>(ph_base)[min(tid + k * kThreads, kLanePhasorBytes / 16 - 1)] = ph[k];
    if (tid < kBands) lds_rev[tid] = rev;
    __syncthreads();   // (the zeros are written)
    store_tables(cur);
    __syncthreads();
    // the counter's answer to the listing wave: the item or stretch behind those that are the workgroup's own
    auto ask = [&]() {
        if (lane == 0) later_item = atomicAdd(a.work + own_zero, 1);
    };
    // (the listing wave's) whether the stretch behind `id` is the workgroup's own too
    auto own_next = [&]() { return STRETCH && own_stretch(id, (int)gridDim.x, n_items); };
    for (;;) {
        const Item nxt = item_in(cur.buf == 2 ? 0 : cur.buf + 1);
        const bool asks = wave == kLister && nxt.n_tiles > 0 && spent(rest) && !own_next();
        if (nxt.n_tiles > 0) load_tables(nxt);
        if (lane < P * kSums) red[wave][lane] = 0.0;   // (pieces without a tile of this wave's)
        double s1[NG], s2[NG];
        float4v t_re[NG], t_im[NG], t_m[NG];   // the table, with the tile's base folded in
        auto begin_piece = [&]() {
            if constexpr (STRETCH) piece_tab = item_tab + at.slot * kSlot;
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                s1[q] = s2[q] = 0.0;
                t_m[q] = table_of(2, q);
                if constexpr (ROTATED) t_re[q] = table_of(0, q), t_im[q] = table_of(1, q);
            }
        };
        begin_piece();
        if (wave >= cur.n_tiles) {
            // No tile of this item to load the next one's first behind.  (What is asked for here is waited for here, where the wave has
            // nothing else to do: left pending, it would have to be waited for wherever the other waves' path joins this one.)
            if (wave < nxt.n_tiles) {
                at = piece_of(nxt, wave);
                load_first(tile_of(at, wave));
            }
            if (asks) ask();
            __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        } else for (int t_idx = wave;;) {
            const Tile now = tile_of(at, t_idx);
            const int n0 = now.n0, cnt = now.cnt;
            int p_key = pos_next;
            // the wave's next tile: of this piece, of a later one, or its first of the next item
            const bool last = t_idx + W >= cur.n_tiles, ahead = !last || wave < nxt.n_tiles, leaves = t_idx + W >= at.t1;
            // Work items: `at` is the next tile's piece from here on.  (Worked out for the loads and once more behind the tile, pieces cost 1 - 4 % of
            // short items: scores, us, 5760 x 655 post-RoPE keys at G = 4 222.2 -> 218.0, 5760 x 279 165.6 -> 160.6, 4608 x 300 half-split 141.2 -> 136.5;
            // 2048 x 2176 equal.  Stretches, whose pieces take more registers, spill up to six more of them so and lose 2 % at G = 1.)
            const int inst = at.inst;   // this tile's
            Tile nt;
            if constexpr (STRETCH) {
                if (!leaves || !ahead) nt = tile_of(at, t_idx + W);
                else if (last) nt = tile_of(piece_of(nxt, wave), wave);
                else nt = tile_of(piece_of(cur, t_idx + W), t_idx + W);
            } else {
                if (last && ahead) at = piece_of(nxt, wave);
                nt = tile_of(at, last && ahead ? wave : t_idx + W);
            }
            asm volatile("" : "+v"(p_key));   // (waits for the position here, and not for a copy between registers further down)
            if (ahead) {
                if constexpr (PAGED) bt_next = load_blocks(nt);   // needed when its first loads go out, half a tile from now
                else pos_next = load_pos(nt, 0);
            }
            if (last && asks) ask();

            // ---- the tile's base
            int base = 0, base1 = 0;   // rows: step 1's may be one of its own
            bool in_table = true, mirrored = false;   // wave-uniform
            // fold e^{-i w base} into the wave's table: a lane works out one band's phasor and hands it to the other three of its
            // block.  (The phase in [-1/2, 1/2] revolutions: in fp32 twice as fine as in [0, 1].)
            auto fold_base = [&]() {
                const double turns = (double)base * lds_rev[my_band];
                const float x = (float)(turns - __builtin_rint(turns));
                const float bs = __builtin_amdgcn_sinf(x), bc = __builtin_amdgcn_cosf(x);
                static_for<0, 4>([&](auto quarter) {
                    constexpr int v = quarter;
                    const float s = quad_lane<quad_same(v)>(bs), c = quad_lane<quad_same(v)>(bc);
#pragma unroll
                    for (int q = 0; q < NG; ++q) {
                        const float qr = table_of(0, q)[v], qi = table_of(1, q)[v];
                        t_re[q][v] = qr * c + qi * s;
                        t_im[q][v] = qi * c - qr * s;
                    }
                });
            };
            if constexpr (!ROTATED) {
                // Usual case: slots in the order of their positions, all within the table's range of the first: base = the first, r >= 0.
                // (The lowest and highest position of every tile through twelve LDS shuffles, each waiting for the one before,
                // cost 64 x 8 head-instances of 131072 keys at G = 8 1 %.)
                base = base1 = __builtin_amdgcn_readfirstlane(p_key);
                // (The difference of two int32 positions fits 32 bits without a sign once none lies below the first.)
                if (__builtin_amdgcn_ballot_w64(p_key < base || (uint32_t)p_key - (uint32_t)base >= (uint32_t)kLaneRange) != 0ull) {
                    const HalfExtremes lo = half_extremes<false>(p_key), hi = half_extremes<true>(p_key);
                    base = min(lo.v[0], lo.v[1]);
                    const int64_t span = (int64_t)max(hi.v[0], hi.v[1]) - (int64_t)base;
                    // positions within the range of the lowest: base = the lowest, r >= 0.  Else base = the middle and the table
                    // serves |r| (a negative r flips the sine), as long as the span stays below twice the range.
                    mirrored = span >= kLaneRange;
                    in_table = span < 2 * kLaneRange - 1;
                    if (mirrored) base = (int)((int64_t)base + (span >> 1));
                    base1 = base;
                    if (!in_table) {
                        // the direct path takes any base: with 0 the folded table keeps its own rounding only
                        base = base1 = 0;
                        if constexpr (ROWS) {
                            // A step's 32 keys may fit the table by themselves: a middle each, the table folded again between
                            // the steps.  9216 x 2176 half-split keys, scores and selection, one position in 2 / 3 / 4 / 6 kept: 1370,
                            // 1436, 1441, 1444 us with a base per tile, 1305, 1320, 1407, 1451 so (1323, 1336, 1359, 1404 on the
                            // sixteen-lane kernel, which takes a base per sixteen keys; from one in 8 on it is the slower one).
                            const int64_t span0 = (int64_t)hi.v[0] - lo.v[0], span1 = (int64_t)hi.v[1] - lo.v[1];
                            if (max(span0, span1) < 2 * kLaneRange - 1) {
                                in_table = true;
                                base = (int)(lo.v[0] + (span0 >> 1));
                                base1 = (int)(lo.v[1] + (span1 >> 1));
                            }
                        }
                    }
                }
                fold_base();
            }
            // the lane's relative position: of its key, or (rows) of its key of either step
            const char *ph_lane = ph_base;
            float sgn = 1.f;
            double rel_d = 0.0;
            auto take_position = [&](int p) {
                if constexpr (ROTATED) return;
                const int64_t rel = (int64_t)p - (int64_t)base;
                rel_d = (double)rel;
                sgn = rel < 0 ? -1.f : 1.f;
                const int r = in_table ? (int)(rel < 0 ? -rel : rel) : 0;   // (0 keeps the unused table address in range)
                ph_lane = ph_base + r * 16 + hh * (16 * kLanePairStride);
            };
            if constexpr (!ROWS) take_position(p_key);

            float4v acc[NG], acc2[NG];   // two chains, so that consecutive matrix instructions do not depend on each other
            float4v acc_m[NG];           // kShortChains: the moduli's products, a third chain
            float4v sum[NG];             // kShortChains: the chains ended so far
            float4v first[NG];           // rows: step 0's scores, over the lane's half of the bands

            // Everything a piece (four bands of the lane's key) needs from LDS: the key's 16 bytes, the phasors of its
            // four bands at the lane's relative position, the lane's table entries.  Pieces are fetched one ahead of
            // the piece being scored, in straight-line code, so that the LDS latency hides behind the arithmetic.
            struct Piece {
                uint4 kq;   // interleaved: four bands; half-split: the real parts of eight
                uint4 ki;   // half-split: their imaginary parts
                float4 e0, e1;
            };
            auto fetch = [&](const Piece &prev, int half, int pc, auto table_tag) {
                constexpr bool TABLE = decltype(table_tag)::value;
                const int f0 = (ROWS ? 0 : 32 * half) + 4 * pc;   // first of the piece's four bands (rows: of the lane's 32)
                Piece o;
                if constexpr (HALF) {
                    o.kq = pc & 1 ? prev.kq : *reinterpret_cast<const uint4 *>(stage + (st_rd ^ ((pc / 2) << 4)));
                    o.ki = pc & 1 ? prev.ki : *reinterpret_cast<const uint4 *>(stage + (st_rd ^ ((8 + pc / 2) << 4)));
                } else {
                    o.kq = *reinterpret_cast<const uint4 *>(stage + (st_rd ^ (pc << 4)));
                }
                if constexpr (TABLE) {
                    o.e0 = *reinterpret_cast<const float4 *>(ph_lane + (f0 / 2) * kLanePairStride);
                    o.e1 = *reinterpret_cast<const float4 *>(ph_lane + (f0 / 2 + 1) * kLanePairStride);
                }
                return o;
            };
            // The vector instructions of the piece first, then its matrix instructions in one run.
            auto score_piece = [&](const Piece &pz, auto half, auto pc, auto table_tag, auto mirror_tag) {
                constexpr bool TABLE = decltype(table_tag)::value, MIRROR = decltype(mirror_tag)::value;
                constexpr int f0 = (ROWS ? 0 : 32 * half) + 4 * pc;
                const uint32_t w[4] = {pz.kq.x, pz.kq.y, pz.kq.z, pz.kq.w};
                const uint32_t wi[4] = {pz.ki.x, pz.ki.y, pz.ki.z, pz.ki.w};
                float cs[4] = {1.f, 1.f, 1.f, 1.f}, sn[4] = {0.f, 0.f, 0.f, 0.f};
                if constexpr (!ROTATED) {
                    if constexpr (TABLE) {
                        cs[0] = pz.e0.x, sn[0] = pz.e0.y, cs[1] = pz.e0.z, sn[1] = pz.e0.w;
                        cs[2] = pz.e1.x, sn[2] = pz.e1.y, cs[3] = pz.e1.z, sn[3] = pz.e1.w;
                        if constexpr (MIRROR) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) sn[k] *= sgn;
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float x = (float)__builtin_amdgcn_fract(rel_d * lds_rev[32 * hh + f0 + k]);
                            sn[k] = __builtin_amdgcn_sinf(x);
                            cs[k] = __builtin_amdgcn_cosf(x);
                        }
                    }
                }
                float kr[4], ki[4], m[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float re, im;
                    if constexpr (HALF) {
                        const int d = 2 * (pc & 1) + (k >> 1);
                        re = (k & 1) ? bf16_hi(w[d]) : bf16_lo(w[d]);
                        im = (k & 1) ? bf16_hi(wi[d]) : bf16_lo(wi[d]);
                    } else {
                        re = bf16_lo(w[k]);
                        im = bf16_hi(w[k]);
                    }
                    m[k] = __builtin_amdgcn_sqrtf(fmaf(re, re, im * im));
                    kr[k] = ROTATED ? re : re * cs[k] - im * sn[k];
                    ki[k] = ROTATED ? im : re * sn[k] + im * cs[k];
                }
                // memory instructions may move across; vector and matrix instructions stay apart
                __builtin_amdgcn_sched_barrier(0x4 | 0x20 | 0x100);
                // A wave in its vector part outranks the waves that are in their matrix runs (whose instructions each
                // hold the pipe for eight cycles and leave issue slots between them): measured in one process, 36 x 16 x 8
                // head-instances of 32768 keys 7.90 -> 7.60 ms, sparse positions 8.51 -> 8.01, G = 8 (64 x 8 of 131072 keys)
                // 4.63 -> 4.38; the other way round gains half of that, the levels themselves (1 / 0, 3 / 0, 2 / 1) nothing.
                __builtin_amdgcn_s_setprio(0);
                static_for<0, 4>([&](auto k) {
                    constexpr int f = f0 + k, v = table_quarter(ROWS, f), kBlock = table_block(ROWS, f);
#pragma unroll
                    for (int q = 0; q < NG; ++q) acc[q] = head_products<ROWS, kBlock>(t_re[q][v], kr[k], acc[q]);
#pragma unroll
                    for (int q = 0; q < NG; ++q) acc2[q] = head_products<ROWS, kBlock>(t_im[q][v], ki[k], acc2[q]);
#pragma unroll
                    for (int q = 0; q < NG; ++q) {
                        float4v &to = kShortChains ? acc_m[q] : acc[q];
                        to = head_products<ROWS, kBlock>(t_m[q][v], m[k], to);
                    }
                });
                __builtin_amdgcn_s_setprio(2);
                __builtin_amdgcn_sched_barrier(0x4 | 0x20 | 0x100);
            };
            auto score_tile = [&](auto table_tag, auto mirror_tag) {
                constexpr int kPieces = ROWS ? 8 : 16;   // of a sum
                constexpr int kChain = chain_pieces(ROTATED, HALF, decltype(table_tag)::value);
                static_for<0, 2>([&](auto half) {
                    stage_half(kd);   // waits for the step's loads, then 8 LDS writes
                    if constexpr (ROWS && !ROTATED) {
                        if constexpr (decltype(mirror_tag)::value)   // (nowhere else do the steps' bases differ)
                            if (half == 1 && base1 != base) {        // wave-uniform
                                base = base1;
                                fold_base();
                            }
                        const auto p = __builtin_amdgcn_permlane32_swap((uint32_t)p_key, (uint32_t)p_key, false, false);
                        take_position((int)p[(int)half]);
                    }
                    if (ROWS || half == 0)
#pragma unroll
                        for (int q = 0; q < NG; ++q) acc[q] = acc2[q] = acc_m[q] = float4v{0.f, 0.f, 0.f, 0.f};
                    // the next loads go out while this step's are scored
                    if (half == 0) {
                        load_half(now, 1, kd, bt_cur);
                    } else if (ahead) {
                        if constexpr (PAGED) pos_next = load_pos(nt, bt_next);   // (ahead of the rows: needed first)
                        load_half(nt, 0, kd, bt_next);
                    }
                    Piece cur = fetch(Piece{}, half, 0, table_tag);
                    static_for<0, 8>([&](auto pc) {
                        Piece nxt = cur;
                        if (pc + 1 < 8) nxt = fetch(cur, half, pc + 1, table_tag);
                        score_piece(cur, half, pc, table_tag, mirror_tag);
                        cur = nxt;
                        constexpr int done = (ROWS ? 0 : 8 * half) + pc + 1;   // pieces of this sum scored so far
                        if (kShortChains && (done % kChain == 0 || done == kPieces)) {
#pragma unroll
                            for (int q = 0; q < NG; ++q) {
                                const float4v chain = acc[q] + acc2[q];
                                sum[q] = done == kChain ? chain : sum[q] + chain;
                                acc[q] = acc2[q] = float4v{0.f, 0.f, 0.f, 0.f};
                            }
                        }
                    });
#pragma unroll
                    for (int q = 0; q < NG; ++q) {
                        if (ROWS || half == 1) acc[q] = kShortChains ? sum[q] + acc_m[q] : acc[q] + acc2[q];
                        if (ROWS && half == 0) first[q] = acc[q];
                    }
                });
            };
            if (ROTATED || !in_table) score_tile(std::false_type{}, std::false_type{});
            else if (mirrored) score_tile(std::true_type{}, std::true_type{});
            else score_tile(std::true_type{}, std::false_type{});

            bt_cur = bt_next;
            // rows: the two halves of the bands together, step 0's keys in lanes 0-31 and step 1's in lanes 32-63
#pragma unroll
            for (int q = 0; q < NG; ++q)
#pragma unroll
                for (int k = 0; ROWS && k < 4; ++k) {
                    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(first[q][k]), __float_as_uint(acc[q][k]), false, false);
                    acc[q][k] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
                }
            // (16-byte stores need floats' alignment only; the rows' bytes fit 32 bits with room above them: mfma_path)
            constexpr uint32_t kNowhere = 0xffffffe0u;
            constexpr int kNonTemporal = 2;
            float *const rw = a.raw + (int64_t)inst * G * c.max_seq_len;
            const __amdgpu_buffer_rsrc_t raw_rows = __builtin_amdgcn_make_buffer_rsrc(rw, 0, (uint32_t)G * (uint32_t)c.max_seq_len * 4u, 0x00027000);
            // ---- lane l holds key n0 + l for heads 4q .. 4q + 3: turned within the blocks, lane (b, j) holds keys n0 + 4b .. + 3 for head 4q + j
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                const bool odd = j & 1, high = j & 2;
                const float4v r = acc[q];
                const float4v x = {quad_lane<kQuadXor1>(r[0]), quad_lane<kQuadXor1>(r[1]), quad_lane<kQuadXor1>(r[2]), quad_lane<kQuadXor1>(r[3])};
                const float4v t = {odd ? x[1] : r[0], odd ? r[1] : x[0], odd ? x[3] : r[2], odd ? r[3] : x[2]};
                const float4v y = {quad_lane<kQuadXor2>(t[0]), quad_lane<kQuadXor2>(t[1]), quad_lane<kQuadXor2>(t[2]), quad_lane<kQuadXor2>(t[3])};
                acc[q] = float4v{high ? y[2] : t[0], high ? y[3] : t[1], high ? t[2] : y[0], high ? t[3] : y[1]};
            }
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                const int g = 4 * q + j, live = g < G ? min(4, cnt - 4 * b) : 0;   // keys of this lane that exist
                // One store for all lanes on every path, so that the compiler can count it (a lane with nothing to store lies beyond the
                // buffer): the wait for the next tile's loads, which went out before, then does not wait for this store too.
                const uint32_t at = ((uint32_t)g * (uint32_t)c.max_seq_len + (uint32_t)(n0 + 4 * b)) * 4u, to = live == 4 ? at : kNowhere;
                // The selection reads the raw scores from HBM whatever the cache policy of this store.  Where tiles cover whole cache lines
                // the non-temporal hint gains 1 % (36 x 16 x 8 x 32768 keys: 7.71 -> 7.63 ms where the stores hurt most, equal where they
                // hurt least; post-RoPE keys 6.80 -> 6.60); where neighbouring tiles share lines it costs 2 - 6 %, since the halves then
                // go to memory one by one (6 x 8 x 8 x 30001 keys, a step: 830 us with it, 778 without, 812 with 4-byte stores; 30008: 817, 769).
                const uint4v scores = __builtin_bit_cast(uint4v, acc[q]);
                if (whole_lines) __builtin_amdgcn_raw_buffer_store_b128(scores, raw_rows, to, 0, kNonTemporal);
                else __builtin_amdgcn_raw_buffer_store_b128(scores, raw_rows, to, 0, 0);
                if (cnt != kTileKeys) {   // (wave-uniform)
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (live < 4 && k < live) rw[at / 4 + k] = acc[q][k];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double v = k < live ? (double)acc[q][k] : 0.0;
                    s1[q] += v;
                    s2[q] += v * v;
                }
            }
            t_idx += W;
            if (!leaves) continue;
            // per-head sums over the wave's keys of the piece: lanes with equal lane % 4 hold the same head
#pragma unroll
            for (int q = 0; q < NG; ++q) {
#pragma unroll
                for (int o = 4; o < 64; o <<= 1) {
                    s1[q] += __shfl_xor(s1[q], o, 64);
                    s2[q] += __shfl_xor(s2[q], o, 64);
                }
                if (lane < 4) {
                    red[wave][(STRETCH ? at.slot * kSums : 0) + (4 * q + lane) * 2 + 0] = s1[q];
                    red[wave][(STRETCH ? at.slot * kSums : 0) + (4 * q + lane) * 2 + 1] = s2[q];
                }
            }
            if (last) {
                if (STRETCH && ahead) at = piece_of(nxt, wave);
                break;
            }
            if (STRETCH) at = piece_of(cur, t_idx);   // (an item of its own has one piece)
            begin_piece();
        }
        if (wave == kLister && nxt.n_tiles > 0) {   // the item after the next (behind the last one nothing is waited for: 1 us of small calls)
            if (spent(rest)) {
                id = own_next() ? id + (int)gridDim.x : 2 * (int)gridDim.x + __builtin_amdgcn_readfirstlane(later_item);
                rest = start_of(id);
            }
            list_item(rest, id, cur.buf == 0 ? 2 : cur.buf - 1);
        }
        __syncthreads();   // nobody reads this item's tables any more
        if (tid < 2 * G * cur.n_pieces) {   // the waves' sums of a piece, in their order
            const int *const o = lds_piece[cur.buf][tid / (2 * G)];
            const int64_t to = ((int64_t)instance_of((uint32_t)o[0], o[1]) * a.n_tiles + o[3]) * (2 * G) + tid % (2 * G);
            const int e = tid % (2 * G), g = e % G, which = e / G;
            double v = 0.0;
            for (int w_ = 0; w_ < W; ++w_) v += red[w_][tid / (2 * G) * kSums + g * 2 + which];
            a.partials[to] = v;
        }
        if (nxt.n_tiles == 0) break;
        cur = nxt;
        store_tables(cur);
        __syncthreads();
    }
}

template <int G>
tri_status launch_lane_g(const ScoreArgs &sa, bool half_split, hipStream_t st)
{
    const bool paged = sa.c.block_shift >= 0, rotated = sa.c.k_rotated != 0;
    const bool stretch = sa.stretches != nullptr;
    auto pick = [&](auto half, auto str) {
        constexpr bool H = decltype(half)::value, S = decltype(str)::value;
        return rotated ? (paged ? score_lane_kernel<G, true, true, H, S> : score_lane_kernel<G, false, true, H, S>)
                       : (paged ? score_lane_kernel<G, true, false, H, S> : score_lane_kernel<G, false, false, H, S>);
    };
    using std::true_type, std::false_type;
    auto kern = stretch ? (half_split ? pick(true_type{}, true_type{}) : pick(false_type{}, true_type{}))
                        : (half_split ? pick(true_type{}, false_type{}) : pick(false_type{}, false_type{}));
    const int lds = lane_lds_bytes(G, paged, rotated, half_split, stretch), threads = lane_waves(G, paged, rotated, half_split) * 64;
    if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
        return hip_status("hipFuncSetAttribute(score_lane_kernel)");
    static std::atomic<int> resident[2][2][2][2][kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        set_error("score: no current device below %d", kMaxDevices);
        return TRI_ERR_HIP;
    }
    std::atomic<int> &cached = resident[stretch ? 1 : 0][half_split ? 1 : 0][rotated ? 1 : 0][paged ? 1 : 0][dev];
    int slots = cached.load(std::memory_order_relaxed);
    if (slots == 0) {
        int n_cu = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, threads, lds) != hipSuccess ||
            n_cu <= 0 || per_cu <= 0) {
            (void)hipGetLastError();
            set_error("score: occupancy query failed");
            return TRI_ERR_HIP;
        }
        slots = n_cu * per_cu;
        cached.store(slots, std::memory_order_relaxed);
    }
    const int64_t max_items = (int64_t)sa.n_tiles * sa.c.n_seqs * sa.c.n_kv_heads * sa.n_layers;
    if (max_items > (int64_t)0x7fff0000) {
        set_error("score: %lld chunks of %d keys exceed the 32-bit work counter", (long long)max_items, sa.chunk_keys);
        return TRI_ERR_UNSUPPORTED;
    }
    const int grid = stretch ? std::min(slots, sa.n_stretches) : (int)std::min<int64_t>((int64_t)slots, max_items);
    ScoreArgs sb = sa;
    sb.first_mult = 1;
    for (int p : {197, 199, 211, 223})
        if (grid % p != 0) {
            sb.first_mult = p;
            break;
        }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, st, sb);
    return hip_status("score_lane_kernel");
}

}  // namespace

// (compiled once per group size: TRI_LANE_GROUP)
template <>
tri_status launch_score_lane<TRI_LANE_GROUP>(const ScoreArgs &sa, bool half_split, hipStream_t st)
{
    return launch_lane_g<TRI_LANE_GROUP>(sa, half_split, st);
}

}  // namespace tri
