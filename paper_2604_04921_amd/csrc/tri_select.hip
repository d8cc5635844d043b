// Top-B selection per head-instance (Section 4.3): an exact select on an order-preserving integer
// image of the float score, then an ordered emit so that the kept slots come out ascending and equal
// scores at the threshold go to the lower slots.
//
// Final scores (tri_select_topk) or, in the fused step, the raw per-head scores and their per-chunk moments are the input; the
// statistics and S_final = max_g (S~(g) - mu_g) / sigma_g are then formed here (neither travels through memory).
// One workgroup selects among a head-instance's keys (select_kernel): up to 32768 keys lie in its LDS, those of longer
// sequences stay in memory.  Where one workgroup per head-instance would read the raw scores too slowly -- long
// sequences, batches of few head-instances -- many workgroups turn them into integer keys and histograms first
// (keys_kernel).
#include <algorithm>

#include "tri_bins.h"
#include "tri_fill.h"

namespace tri {

namespace {

// 16 bytes wherever floats may lie: the hardware asks for no more than a dword's alignment
typedef float float4v __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t word4v __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kSelThreads = 1024;       // threads per workgroup, or
constexpr int kSelSmallThreads = 256;   // many short sequences
constexpr int kSelHeldKeys = 32768;     // keys held in LDS at most
constexpr int kSelBins = 2048;          // linear score bins of the histogram pass

// A score as the selection ranks it, before its key and its bin are formed: -0.0 is folded onto +0.0, and one that is no number counts as
// +inf (its key alone would lie above every number's, its bin below: passes that disagree about a score leave entries of the kept set
// unwritten).
__device__ __forceinline__ float ranked(float score) { return fminf(score + 0.0f, __builtin_inff()); }
// Monotone map float -> uint32 (larger float <=> larger key) of a ranked score.
__device__ __forceinline__ uint32_t order_key(float x)
{
    const uint32_t b = __float_as_uint(x);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}

struct SelectArgs {
    const float *final_;   // [inst][Nmax] final scores, or NULL when raw scores and their moments are given
    float *raw;            // [inst][G][Nmax]; keys_kernel leaves a head-instance's integer keys in its first row
    const double *partials;   // [inst][n_tiles][2G] per-tile sum and sum of squares of the raw scores
    int32_t n_tiles, tile_keys;
    uint32_t *hist;        // [inst][n_chunks][kSelBins / 2]: histograms of the keys' chunks, two 16-bit counts per word
    const int32_t *seq_len;
    int32_t *kept_idx;     // [inst][B]
    int32_t *kept_cnt;     // [inst]
    int32_t n_seqs, n_kv_heads, max_seq_len, budget;
    int32_t chunk_keys, n_chunks;   // keys_kernel: keys per workgroup, workgroups per head-instance
    const int32_t *head_budgets;   // [L][Hkv] or NULL: budget of each (layer, KV head), at most `budget`
    // fill != 0: the workgroup goes on to evict its head-instance in place (fill_block)
    FillArgs fa;
    int32_t fill;
};

// The budget of head-instance `inst`: the common one, or the head's own (read into [0, budget]).
__device__ __forceinline__ int instance_budget(const SelectArgs &a, int inst)
{
    if (!a.head_budgets) return a.budget;
    const int h = inst % a.n_kv_heads, l = inst / (a.n_kv_heads * a.n_seqs);
    return min(max(a.head_budgets[l * a.n_kv_heads + h], 0), a.budget);
}

__device__ __forceinline__ float key_to_float(uint32_t u)
{
    return __uint_as_float(u ^ ((uint32_t)((int32_t)~u >> 31) | 0x80000000u));
}
// 2048 bins over [-4, 12): where a score lies in them, and its bin (scores beyond go to the first and the last one)
__device__ __forceinline__ float bin_place(float score) { return fmaf(score, (float)kBinsPerUnit, (float)kBinOfZero); }
__device__ __forceinline__ int linear_bin(float score) { return (int)__builtin_amdgcn_fmed3f(bin_place(score), 0.0f, 2047.0f); }
__device__ __forceinline__ int linear_bin(uint32_t u) { return linear_bin(key_to_float(u)); }

// The least key of bin `bin` (1 to 2047) and those above it: bins are ranges of keys, since places rise with keys.
__device__ __forceinline__ uint32_t first_key(int bin)
{
    const double edge = bin_edge(bin);
    const float f = (float)edge;
    return order_key(f) + ((double)f < edge ? 1u : 0u);
}

// Mean and 1/sigma of a head-instance's heads from the moments (block_stats; every thread of the workgroup calls).
template <int G>
__device__ __forceinline__ Moments load_moments(const SelectArgs &a, int inst, int tid)
{
    return moments_ahead<G>(a.partials + (int64_t)inst * a.n_tiles * (2 * G), a.n_tiles, tid);
}
template <int G>
__device__ __forceinline__ void load_zparams(const SelectArgs &a, const Moments &ahead, int inst, int N, int tid, double *zpart, double *zst,
                                             ZParams (&zp)[G])
{
    block_stats<G>(ahead, a.partials + (int64_t)inst * a.n_tiles * (2 * G), moment_entries(a.n_tiles, a.tile_keys, N), N, tid, zpart, zst);
#pragma unroll
    for (int g = 0; g < G; ++g) zp[g] = z_params(zst[2 * g], zst[2 * g + 1]);
}

// The threshold among the m candidates (keys of the bin that holds the B-th largest, zeros behind them up to
// the next multiple of 32): the key of which fewer than `need` are larger and at least `need` as large.  sh[3] = that key,
// sh[4] = how many are larger.  Eight neighbouring threads share a candidate and read the list 16 bytes at a time: the phase
// is a chain of LDS latencies (one thread per candidate, one key per read: 40 candidates cost 3 us).  Barriers are the
// caller's.
template <int THREADS>
__device__ __forceinline__ void rank_candidates(const uint32_t *cand_key, uint32_t m, uint32_t need, int tid, uint32_t *sh)
{
    const uint4 *quad = reinterpret_cast<const uint4 *>(cand_key);
    const int part = tid & 7;
    for (uint32_t c0 = 0; c0 < m; c0 += THREADS / 8) {   // uniform: every lane takes part in the shuffles
        const uint32_t c = c0 + (uint32_t)(tid >> 3);
        const uint32_t kc = c < m ? cand_key[c] : 0u;
        uint32_t gt = 0u, ge = 0u;
#pragma unroll 2
        for (uint32_t q = part; 4u * q < m; q += 8u) {
            const uint4 k = quad[q];
            gt += (k.x > kc ? 1u : 0u) + (k.y > kc ? 1u : 0u) + (k.z > kc ? 1u : 0u) + (k.w > kc ? 1u : 0u);
            ge += (k.x >= kc ? 1u : 0u) + (k.y >= kc ? 1u : 0u) + (k.z >= kc ? 1u : 0u) + (k.w >= kc ? 1u : 0u);
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            gt += __shfl_xor(gt, o, 64);
            ge += __shfl_xor(ge, o, 64);
        }
        if (c < m && gt < need && need <= ge) {   // candidates of equal key write the same values
            sh[3] = kc;
            sh[4] = gt;
        }
    }
}

// `add` and how many lanes below this one are set in the mask
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask, uint32_t add)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, add));
}

// Sum of the first `wave` of W counts (the loads do not wait for one another).
template <int W>
__device__ __forceinline__ uint32_t sum_before(const uint32_t *counts, int wave)
{
    uint32_t sum = 0u;
#pragma unroll
    for (int w = 0; w < W; ++w) sum += w < wave ? counts[w] : 0u;
    return sum;
}

// Raw scores -> integer keys (written over the head-instance's first raw row: every key's scores are read by the thread that
// writes it) and the histogram of each chunk's linear bins.  grid (instances * n_chunks), block 256.  A streaming kernel:
// 4 G bytes read and 4 written per key, the next keys' loads issued before a key's arithmetic.  (Four keys per thread and load, whatever the
// rows' alignment: what a load brings from behind a row's end lies in the workspace too and is not used.)
constexpr int kKeysThreads = 256;
template <int G>
__global__ __launch_bounds__(kKeysThreads) void keys_kernel(SelectArgs a)
{
    __shared__ uint32_t hist[kSelBins];
    __shared__ double zst[2 * G], zpart[32 * G];
    const int tid = threadIdx.x;
    const int inst = blockIdx.x / a.n_chunks, chunk = blockIdx.x - inst * a.n_chunks;
    const int s = (inst / a.n_kv_heads) % a.n_seqs;
    const Moments ahead = load_moments<G>(a, inst, tid);
    const int N = clamp_len(a.seq_len[s], a.max_seq_len);
    const int c0 = chunk * a.chunk_keys, c1 = min(N, c0 + a.chunk_keys);
    const int B = instance_budget(a, inst);
    if (c0 >= N || N <= B || B == 0) return;   // (uniform over the workgroup; select_kernel reads nothing of it either)
    for (int k = tid; k < kSelBins; k += kKeysThreads) hist[k] = 0u;
    ZParams zp[G];
    load_zparams<G>(a, ahead, inst, N, tid, zpart, zst, zp);
    __syncthreads();
    float *rw = a.raw + (int64_t)inst * G * a.max_seq_len;
    constexpr int kStep = 4 * kKeysThreads;   // keys per iteration
    // thread's key i of the iteration at n0
    auto slot = [&](int n0, int i) { return n0 + 4 * tid + i; };
    auto load = [&](int n0, float (&v)[G][4]) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float *row = rw + (int64_t)g * a.max_seq_len;
            const float4v t = __builtin_nontemporal_load(reinterpret_cast<const float4v *>(row + min(slot(n0, 0), (N - 1) & ~3)));
#pragma unroll
            for (int i = 0; i < 4; ++i) v[g][i] = t[i];
        }
    };
    auto finish = [&](int n0, const float (&v)[G][4]) {
        uint32_t u[4];
        int bin[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float f = z_score(v[0][i], zp[0]);
#pragma unroll
            for (int g = 1; g < G; ++g) f = fmaxf(f, z_score(v[g][i], zp[g]));
            f = ranked(f);
            u[i] = order_key(f);
            bin[i] = linear_bin(f);
        }
        uint32_t *ks = reinterpret_cast<uint32_t *>(rw);
        if (slot(n0, 3) < c1) {
            *reinterpret_cast<word4v *>(ks + slot(n0, 0)) = word4v{u[0], u[1], u[2], u[3]};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (slot(n0, i) < c1) ks[slot(n0, i)] = u[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (slot(n0, i) < c1) atomicAdd(&hist[bin[i]], 1u);
    };
    // A clamped load of the iteration past the end may read what another thread has already replaced by keys: its values
    // are not used.
    float cur[G][4], nxt[G][4];
    load(c0, cur);
    for (int n0 = c0; n0 < c1; n0 += kStep) {
        load(n0 + kStep, nxt);
        finish(n0, cur);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i) cur[g][i] = nxt[g][i];
    }
    __syncthreads();
    uint32_t *out = a.hist + ((int64_t)inst * a.n_chunks + chunk) * (kSelBins / 2);
    for (int k = tid; k < kSelBins / 2; k += kKeysThreads) out[k] = hist[2 * k] | (hist[2 * k + 1] << 16);
}

// One workgroup selects among a head-instance's keys.  grid (instances).
//   SRC     G > 0: raw scores of G query heads; 0: final scores; kFromKeys: what keys_kernel left (integer keys, chunk
//           histograms; not HELD)
//   HELD    the keys lie in LDS (dynamic, four bytes per key, whole rows of 256) from the first pass on; else every pass reads
//           them from memory
//   VEC     16-byte loads of the source: always of the workspace's rows (see keys_kernel); of final scores, which are the caller's, where
//           four entries from a slot below N on exist (rows of a multiple of four)
// Steps:
//   1. Histogram over 2048 *linear* bins of the score on [-4, 12) (monotone in the score, so a valid coarse partition; z-scores
//      spread over hundreds of bins, whereas the top bits of their float image share a handful of values and would
//      serialise the LDS atomics).
//   2. One scan finds the bin that holds the B-th largest score; its few keys are gathered and ranked exactly, which gives the
//      threshold key and the number of threshold ties to keep.  A bin with more keys than the list holds (many equal
//      scores) is resolved one bit at a time instead.
//   3. Ordered emit: every wave owns a contiguous stretch of the slots and knows from the gathering pass how many it keeps.
// Between the passes there are half a dozen barriers, so the kernel is a chain of latencies wherever the batch does not
// keep several workgroups per CU busy -- that of fetching its instructions among them: code that unrolled the rows to
// hold the keys in registers was 27 to 40 KB and ran once through; these loops are 7 to 8 KB (the
// fill's included, 16), and leave two to three times the registers free.  Measured against that variant: 4608 head-instances of 8000 keys,
// the whole step 3773 -> 3725 us; 2304 of 32768, this launch 342 -> 302 us; one of 4096, 11.4 -> 8.3 us; a step on eight of
// 32768 70 -> 66 us.
constexpr int kFromKeys = -1;
template <int SRC, bool VEC, bool HELD, int THREADS>
__global__ __launch_bounds__(THREADS, HELD ? (THREADS == kSelThreads ? 4 : 5) : 8) void select_kernel(SelectArgs a, int64_t key_row)
{
    static_assert(VEC || SRC == 0, "the workspace's rows allow 16-byte loads whatever their length");
    constexpr int kWaves = THREADS / 64;
    constexpr int kBinsPerThread = kSelBins / THREADS;
    constexpr int kHeads = SRC > 0 ? SRC : 1;
    constexpr int kCand = kSelBins / 2;             // keys of the threshold bin ranked in LDS
    extern __shared__ __align__(16) uint32_t keys[];   // HELD: the keys; later the fill's move list
    __shared__ __align__(16) uint32_t bins[kSelBins];   // the histogram, then candidates (first half keys, second half slots)
    __shared__ uint32_t scan_tot[kWaves];
    __shared__ uint32_t wave_gt[kWaves], wave_eq[kWaves];
    __shared__ uint32_t sh[36];   // 0: selected bin, 1: need inside it, 2: candidate count, 3: threshold key, 4..35: bit counters / larger candidates
    uint32_t *const cand_key = bins, *const cand_idx = bins + kCand;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int inst = blockIdx.x;
    const int s = (inst / a.n_kv_heads) % a.n_seqs;
    Moments ahead{};
    if constexpr (SRC > 0) ahead = load_moments<kHeads>(a, inst, tid);
    const int N = clamp_len(a.seq_len[s], a.max_seq_len);
    const int B = instance_budget(a, inst);
    int32_t *out = a.kept_idx + (int64_t)inst * a.budget;
    if (tid == 0) a.kept_cnt[inst] = N < B ? N : B;
    // the eviction in place that may follow: keys and histogram are free by then
    auto fill_tail = [&](int cnt) {
        if constexpr (HELD && SRC > 0) {
            if (a.fill) {
                __syncthreads();   // out[] is complete and nobody reads the LDS any more
                fill_block<THREADS>(a.fa, inst, cnt, out, reinterpret_cast<int32_t *>(keys), bins, scan_tot,
                                    reinterpret_cast<int32_t *>(&sh[0]));
            }
        }
    };
    if (B == 0) {   // a head whose own budget is 0 keeps nothing
        fill_tail(0);
        return;
    }
    if (N <= B) {  // nothing to evict: keep every slot
        for (int n = tid; n < N; n += THREADS) out[n] = n;
        fill_tail(N);
        return;
    }
    const float *src = SRC > 0 ? a.raw + (int64_t)inst * kHeads * a.max_seq_len
                               : SRC == 0 ? a.final_ + (int64_t)inst * a.max_seq_len : nullptr;
    const uint32_t *ks = SRC == kFromKeys ? reinterpret_cast<const uint32_t *>(a.raw) + inst * key_row : nullptr;

    // ---- HELD, scores: the first loads go out ahead of the statistics, which are a chain of loads and barriers of their own
    constexpr int kStep = 4 * THREADS;   // keys per iteration of the loading loop
    auto src_slot = [&](int n0, int i) { return VEC ? n0 + 4 * tid + i : n0 + i * THREADS + tid; };
    auto load = [&](int n0, float (&v)[kHeads][4]) {
#pragma unroll
        for (int g = 0; g < kHeads; ++g) {
            const float *row = src + (int64_t)g * a.max_seq_len;
            if constexpr (VEC) {
                const float4v t = __builtin_nontemporal_load(reinterpret_cast<const float4v *>(row + min(src_slot(n0, 0), (N - 1) & ~3)));
#pragma unroll
                for (int i = 0; i < 4; ++i) v[g][i] = t[i];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[g][i] = __builtin_nontemporal_load(row + min(src_slot(n0, i), N - 1));
            }
        }
    };
    float cur[kHeads][4];
    if constexpr (HELD) load(0, cur);
    for (int k = tid; k < kSelBins; k += THREADS) bins[k] = 0u;
    if (tid < 36) sh[tid] = 0u;
    if (tid < kWaves) wave_gt[tid] = wave_eq[tid] = 0u;
    ZParams zp[kHeads];
    if constexpr (SRC > 0) {
        __shared__ double zst[2 * kHeads], zpart[32 * kHeads];
        load_zparams<kHeads>(a, ahead, inst, N, tid, zpart, zst, zp);
    }
    __syncthreads();

    // ---- keys into LDS (a slot past the end, up to the row's, holds key 0, which no score maps to and which lies below
    // every threshold), histogram of their bins
    if constexpr (HELD) {
        for (int n0 = 0; n0 < N; n0 += kStep) {
            float nxt[kHeads][4];
            load(n0 + kStep, nxt);   // (past the end: the last key again)
            uint32_t u[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float f = cur[0][i];
                if constexpr (SRC > 0) {
                    f = z_score(f, zp[0]);
#pragma unroll
                    for (int g = 1; g < kHeads; ++g) f = fmaxf(f, z_score(cur[g][i], zp[g]));
                }
                f = ranked(f);
                u[i] = src_slot(n0, i) < N ? order_key(f) : 0u;
                if (src_slot(n0, i) < N) atomicAdd(&bins[linear_bin(f)], 1u);
            }
            const int end = (N + 255) & ~255;
            if constexpr (VEC) {
                if (src_slot(n0, 0) < end) *reinterpret_cast<uint4 *>(keys + src_slot(n0, 0)) = make_uint4(u[0], u[1], u[2], u[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (src_slot(n0, i) < end) keys[src_slot(n0, i)] = u[i];
            }
#pragma unroll
            for (int g = 0; g < kHeads; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) cur[g][i] = nxt[g][i];
        }
    }
    // The wave's stretch [w0, w1) in rows of 256 slots.  f(n0, u): slot n0 + 4 lane + i holds key u[i]; rows in ascending order.
    constexpr int kRow = 256;
    const int seg = ((N + kWaves - 1) / kWaves + kRow - 1) / kRow * kRow;
    const int w0 = min(N, wave * seg), w1 = min(N, w0 + seg);
    auto load_row = [&](int n0, uint32_t (&u)[4]) {
        if constexpr (VEC) {
            const int n = min(n0 + 4 * lane, (N - 1) & ~3);
            if constexpr (SRC == 0) {
                const float4v t = *reinterpret_cast<const float4v *>(src + n);
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = order_key(ranked(t[i]));
            } else {
                const word4v t = *reinterpret_cast<const word4v *>(ks + n);
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = t[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = min(n0 + 4 * lane + i, N - 1);
                u[i] = order_key(ranked(src[n]));
            }
        }
    };
    auto for_rows = [&](auto f) {
        if constexpr (HELD) {
#pragma unroll 1
            for (int n0 = w0; n0 < w1; n0 += kRow) {
                const uint4 t = *reinterpret_cast<const uint4 *>(keys + n0 + 4 * lane);
                const uint32_t u[4] = {t.x, t.y, t.z, t.w};
                f(n0, u);
            }
        } else {
            uint32_t u[4], nxt[4];
            if (w0 < w1) load_row(w0, u);
#pragma unroll 1
            for (int n0 = w0; n0 < w1; n0 += kRow) {
                load_row(n0 + kRow, nxt);   // the next row is on its way while this one is looked at
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n0 + 4 * lane + i >= w1) u[i] = 0u;
                f(n0, u);
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = nxt[i];
            }
        }
    };

    // ---- the bin holding the B-th largest: thread t owns bins 2047 - t * kBinsPerThread and the ones just below
    uint32_t v[kBinsPerThread];
    if constexpr (SRC == kFromKeys) {
        static_assert(THREADS == kSelThreads, "one thread per word of a chunk's histogram");
        v[0] = v[1] = 0u;
        const int chunks = (N + a.chunk_keys - 1) / a.chunk_keys;
        const uint32_t *h = a.hist + (int64_t)inst * a.n_chunks * (kSelBins / 2) + (kSelBins / 2 - 1 - tid);
        for (int c0 = 0; c0 < chunks; c0 += 8) {   // eight loads in flight
            uint32_t t[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) t[c] = h[(int64_t)min(c0 + c, chunks - 1) * (kSelBins / 2)];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if (c0 + c >= chunks) t[c] = 0u;
                v[0] += t[c] >> 16;
                v[1] += t[c] & 0xffffu;
            }
        }
    } else {
        if constexpr (!HELD)
            for_rows([&](int, const uint32_t (&u)[4]) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (u[i] != 0u) atomicAdd(&bins[linear_bin(u[i])], 1u);
            });
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kBinsPerThread; ++k) v[k] = bins[kSelBins - 1 - kBinsPerThread * tid - k];
    }
    {
        uint32_t own = 0u;
#pragma unroll
        for (int k = 0; k < kBinsPerThread; ++k) own += v[k];
        uint32_t cum = own;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_up(cum, o, 64);
            if (lane >= o) cum += t;
        }
        if (lane == 63) scan_tot[wave] = cum;
        __syncthreads();   // (the histogram has been read: its place now takes the candidates)
        for (int k = tid; k < kCand; k += THREADS) cand_key[k] = 0u;
        uint32_t excl = cum - own + sum_before<kWaves>(scan_tot, wave);
        const uint32_t want = (uint32_t)B;
#pragma unroll
        for (int k = 0; k < kBinsPerThread; ++k) {   // exactly one thread and bin holds the B-th key
            if (excl < want && want <= excl + v[k]) {
                sh[0] = (uint32_t)(kSelBins - 1 - kBinsPerThread * tid - k);
                sh[1] = want - excl;
            }
            excl += v[k];
        }
    }
    __syncthreads();
    const int sel_bin = (int)sh[0];
    uint32_t need = sh[1];   // how many keys of the selected bin are kept (>= 1)

    // ---- gather the selected bin's keys (any order; the ranks below do not depend on it), count the keys above it
    uint32_t above_bin = 0u;
    // (places below the first bin and beyond the last one belong to them; a slot past the end, key 0, is no number and no score's)
    auto gather_bin = [&](auto above, auto inside) {
        for_rows([&](int n0, const uint32_t (&u)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                above_bin += above(u[i]) ? 1u : 0u;
                if (inside(u[i])) {
                    const uint32_t pos = atomicAdd(&sh[2], 1u);
                    if (pos < (uint32_t)kCand) {
                        cand_key[pos] = u[i];
                        cand_idx[pos] = (uint32_t)(n0 + 4 * lane + i);
                    }
                }
            }
        });
    };
    const bool last_bin = sel_bin == kSelBins - 1;
    if constexpr (HELD) {
        const float bin_lo = sel_bin == 0 ? -__builtin_inff() : (float)sel_bin, bin_hi = last_bin ? __builtin_inff() : (float)(sel_bin + 1);
        gather_bin([&](uint32_t u) { return bin_place(key_to_float(u)) >= bin_hi && !last_bin; },
                   [&](uint32_t u) { const float place = bin_place(key_to_float(u)); return place >= bin_lo && (place < bin_hi || last_bin); });
    } else {
        // Long rows: compared as keys, with the bin's ends worked out once, and not key by key as places.  With the single comparison of the emit
        // below, a selection of 8 rows of 131072 keys 54.1 -> 45.8 us.  (Ends that the wave searches for in twelve rounds: 47.2, and 8 sequences of 2176
        // keys in rows of 131072 7.0 instead of 6.3, where the places take 6.2.)
        const uint32_t first = sel_bin == 0 ? 1u : first_key(sel_bin), end = last_bin ? ~0u : first_key(sel_bin + 1);
        gather_bin([&](uint32_t u) { return u >= end; }, [&](uint32_t u) { return u - first < end - first; });
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) above_bin += __shfl_xor(above_bin, o, 64);
    if (lane == 0) wave_gt[wave] = above_bin;
    __syncthreads();
    const uint32_t m = sh[2];
    uint32_t thr;
    if (m <= (uint32_t)kCand) {
        rank_candidates<THREADS>(cand_key, m, need, tid, sh);
        __syncthreads();
        thr = sh[3];
        need -= sh[4];   // threshold ties kept
        for (uint32_t c = tid; c < m; c += THREADS) {   // the waves' own counts
            const int owner = (int)cand_idx[c] / seg;
            if (cand_key[c] > thr) atomicAdd(&wave_gt[owner], 1u);
            else if (cand_key[c] == thr) atomicAdd(&wave_eq[owner], 1u);
        }
        __syncthreads();
    } else {
        // too many keys in one bin (many equal scores): one bit at a time, keys of the bin only
        uint32_t prefix = 0u, mask = 0u;
#pragma unroll 1
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t bm = 1u << bit;
            uint32_t c = 0u;
            for_rows([&](int, const uint32_t (&u)[4]) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool in = u[i] != 0u && linear_bin(u[i]) == sel_bin;
                    c += (uint32_t)__popcll(__ballot(in && (u[i] & mask) == prefix && (u[i] & bm) != 0u));
                }
            });
            if (lane == 0 && c) atomicAdd(&sh[4 + bit], c);
            __syncthreads();
            const uint32_t ones = sh[4 + bit];
            if (ones >= need) prefix |= bm;
            else need -= ones;
            mask |= bm;
        }
        thr = prefix;
        uint32_t cg = 0u, ce = 0u;
        for_rows([&](int, const uint32_t (&u)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                cg += (uint32_t)__popcll(__ballot(u[i] > thr));
                ce += (uint32_t)__popcll(__ballot(u[i] == thr));
            }
        });
        if (lane == 0) {
            wave_gt[wave] = cg;
            wave_eq[wave] = ce;
        }
        __syncthreads();
    }
    // keys > thr are kept; of the keys == thr the first `need` slots

    // ---- ordered emit: the wave starts behind the kept slots of the waves before it
    uint32_t g_run = sum_before<kWaves>(wave_gt, wave), e_run = sum_before<kWaves>(wave_eq, wave);
    // Every threshold tie is kept (mostly there is one): one comparison per key (8 rows of 32768 keys, this launch, 21.7 -> 20.4 us, 576 of them
    // 90 -> 86, 8 of 12289 11.9 -> 11.5; short ones 0.2 us either way).
    if (sum_before<kWaves>(wave_eq, kWaves) == need) {
        uint32_t run = g_run + e_run;
        for_rows([&](int n0, const uint32_t (&u)[4]) {
            uint32_t at = run;   // kept keys before the lane's first slot
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint64_t m = __ballot(u[i] >= thr);
                at = lanes_below(m, at);
                run += (uint32_t)__popcll(m);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool kept = u[i] >= thr;
                if (kept && at < (uint32_t)B) out[at] = n0 + 4 * lane + i;
                at += kept ? 1u : 0u;
            }
        });
        fill_tail(B);
        return;
    }
    for_rows([&](int n0, const uint32_t (&u)[4]) {
        uint32_t g_at = g_run, e_at = e_run;   // kept / threshold keys before the lane's first slot
        uint64_t eq_any = 0ull;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t gm = __ballot(u[i] > thr);
            g_at = lanes_below(gm, g_at);
            g_run += (uint32_t)__popcll(gm);
            eq_any |= __ballot(u[i] == thr);
        }
        if (eq_any) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint64_t em = __ballot(u[i] == thr);
                e_at = lanes_below(em, e_at);
                e_run += (uint32_t)__popcll(em);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool gt = u[i] > thr, eq = u[i] == thr;
            const uint32_t dst = g_at + min(e_at, need);
            if ((gt || (eq && e_at < need)) && dst < (uint32_t)B) out[dst] = n0 + 4 * lane + i;
            g_at += gt ? 1u : 0u;
            e_at += eq ? 1u : 0u;
        }
    });
    fill_tail(B);
}

template <int SRC>
tri_status launch_held(const SelectArgs &sa, int n_inst, bool small, bool vec, hipStream_t st)
{
    auto kern = small ? select_kernel<SRC, true, true, kSelSmallThreads> : select_kernel<SRC, true, true, kSelThreads>;
    if constexpr (SRC == 0)
        if (!vec) kern = small ? select_kernel<SRC, false, true, kSelSmallThreads> : select_kernel<SRC, false, true, kSelThreads>;
    size_t lds = (size_t)((sa.max_seq_len + 255) / 256 * 256) * sizeof(uint32_t);
    if (sa.fill) lds = std::max(lds, (size_t)sa.budget * 2 * sizeof(int32_t));
    // (the most any call asks for, not this call's share: the limit belongs to the process, and another thread may set it between)
    constexpr int kLdsLimit = kSelHeldKeys * (int)sizeof(uint32_t);
    if (lds > 48 * 1024 && hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit) != hipSuccess)
        return hip_status("hipFuncSetAttribute(select_kernel)");
    hipLaunchKernelGGL(kern, dim3(n_inst), dim3(small ? kSelSmallThreads : kSelThreads), lds, st, sa, (int64_t)0);
    return hip_status("select_kernel");
}

template <int G>
tri_status launch_select_g(const SelectArgs &sa, int n_inst, int n_cu, hipStream_t st)
{
    const bool vec = G > 0 || (sa.max_seq_len & 3) == 0;
    if (sa.max_seq_len <= kSelHeldKeys) {
        // Short sequences: small workgroups, cheap barriers, several per CU -- unless there are so few that a CU has one
        // anyway (one head-instance of 4096 keys, whole step: 32.1 us with 1024 threads, 33.4 with 256; 288 of 2176, score and
        // selection: 92.4 and 91.7; 1152: equal; 2304: 385.6 and 384.5).
        const bool small = sa.max_seq_len <= 4096 && n_inst > n_cu / 2;
        return launch_held<G>(sa, n_inst, small, vec, st);
    }
    if constexpr (G > 0) {
        // Longer ones through keys_kernel: 512 head-instances of 131072 keys, eight heads, 744 us in one launch that kept the
        // keys in memory -> 486 + 125 us; 768 of 4096 to 65536 keys, four heads, 486 us in two launches split by length -> 152 +
        // 80 us.  (Up to 32768 keys the extra launch and the keys' way through memory cost what the wider grid
        // gains: eight head-instances of 32768 keys, whole step, 64.9 us against 66.2; of 8192, 41.7 against 38.5; 512 of
        // 32768, 1202 against 1153.)
        SelectArgs sk = sa;
        sk.chunk_keys = 2048;   // about sixteen chunks per head-instance; a chunk's counts fit 16 bits
        while (sk.chunk_keys < 32768 && sk.max_seq_len > 16 * sk.chunk_keys) sk.chunk_keys *= 2;
        sk.n_chunks = (sk.max_seq_len + sk.chunk_keys - 1) / sk.chunk_keys;
        const dim3 grid((uint32_t)((int64_t)n_inst * sk.n_chunks));
        hipLaunchKernelGGL(keys_kernel<G>, grid, dim3(kKeysThreads), 0, st, sk);
        tri_status rc = hip_status("keys_kernel");
        if (rc != TRI_OK) return rc;
        const int64_t key_row = (int64_t)G * sk.max_seq_len;
        hipLaunchKernelGGL((select_kernel<kFromKeys, true, false, kSelThreads>), dim3(n_inst), dim3(kSelThreads), 0, st, sk, key_row);
        return hip_status("select_kernel");
    }
    if constexpr (G == 0) {
        auto kern = vec ? select_kernel<0, true, false, kSelThreads> : select_kernel<0, false, false, kSelThreads>;
        hipLaunchKernelGGL(kern, dim3(n_inst), dim3(kSelThreads), 0, st, sa, (int64_t)0);
    }
    return hip_status("select_kernel");
}

}  // namespace

tri_status launch_select(const tri_model &m, const float *final_scores, float *raw, MomentLayout moments, uint32_t *hist,
                         const tri_cache &c, int32_t budget, int32_t *kept_idx, int32_t *kept_cnt, hipStream_t st, const FillTail *fill,
                         bool *fill_taken)
{
    if (fill_taken) *fill_taken = false;
    const int n_inst = m.n_layers * c.n_seqs * m.n_kv_heads;
    if (n_inst <= 0) return TRI_OK;
    SelectArgs sa{final_scores, raw, moments.partials, moments.n_tiles, moments.tile_keys, hist, c.seq_len, kept_idx,
                  kept_cnt, c.n_seqs, m.n_kv_heads, c.max_seq_len, budget, 1, 1, m.head_budgets};
    sa.fill = 0;
    // Short sequences: the eviction in place rides along (its move list takes the keys' place in LDS) -- on small batches, whose
    // workgroups are all resident at once (eight of 256 threads per CU): there the launch saved counts (one sequence of 288
    // head-instances: 0.147 -> 0.142 ms per step, four: 0.299 -> 0.291), whereas 18432 head-instances take 0.74 ms this way
    // against 0.21 + 0.44 ms as two launches.
    int n_cu = 0;
    const tri_status rcu = device_cus(&n_cu);
    if (rcu != TRI_OK) return rcu;
    // (not where the new lengths are written over the old ones, which other workgroups of the launch still read)
    const bool aliased = fill && fill->new_seq_len && fill->new_seq_len < c.seq_len + c.n_seqs && c.seq_len < fill->new_seq_len + c.n_seqs;
    if (!final_scores && fill && fill_taken && !aliased && c.max_seq_len <= 4096 && budget <= 2048 && n_inst <= 8 * n_cu) {
        sa.fa = FillArgs{make_view(m, c), fill->new_seq_len, budget, c.dtype == TRI_BF16 ? 2 : 4,
                         kHeadDim * (c.dtype == TRI_BF16 ? 2 : 4) / 16};
        sa.fill = 1;
        *fill_taken = true;
    }
    if (final_scores) return launch_select_g<0>(sa, n_inst, n_cu, st);
    switch (m.n_q_heads / m.n_kv_heads) {
        case 1: return launch_select_g<1>(sa, n_inst, n_cu, st);
        case 2: return launch_select_g<2>(sa, n_inst, n_cu, st);
        case 3: return launch_select_g<3>(sa, n_inst, n_cu, st);
        case 4: return launch_select_g<4>(sa, n_inst, n_cu, st);
        case 5: return launch_select_g<5>(sa, n_inst, n_cu, st);
        case 6: return launch_select_g<6>(sa, n_inst, n_cu, st);
        case 7: return launch_select_g<7>(sa, n_inst, n_cu, st);
        case 8: return launch_select_g<8>(sa, n_inst, n_cu, st);
    }
    set_error("group size not built (1 to 8)");
    return TRI_ERR_UNSUPPORTED;
}

}  // namespace tri
