// Declarations shared by the two score kernels (generic and MFMA).
#pragma once
#include "tri_internal.h"
#include "tri_items.h"

namespace tri {

struct ScoreArgs {
    CacheView c;
    const float *table;      // [L][S][Hkv][F][3][G]: folded centre table
    const double *band_rev;  // [F]: omega_f / 2pi
    const uint4 *phasors;    // relative-position phasor table (MFMA kernel only)
    float *raw;              // [L][S][Hq][Nmax]
    double *partials;        // [L][S][Hkv][n_tiles][2G]: per-tile sum and sum of squares
    int32_t n_tiles;         // tiles per head-instance in `partials`
    int32_t n_layers;
    int32_t first_mult;      // MFMA kernel only: workgroup b starts on item (b * first_mult) mod grid size
    int32_t *work;           // MFMA kernel only: item counter and work list (fast_work_ints(S, Nmax) ints)
    int32_t chunk_keys;      // MFMA kernels only: keys per work item (= keys per entry of `partials`)
    const int32_t *stretches;   // general MFMA kernel: a StretchPlan instead of a work list, or NULL
    int32_t n_stretches, n_first;   // at most; how many of them the plan has
};

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Relative positions covered by the sixteen-lane kernel's phasor table.
constexpr int kPhasorRange = 128;
constexpr int kPhasorBlockStride = kPhasorRange * 16 + 64;      // bytes per 4-band chunk (64 B skew)
constexpr int kPhasorHalfStride = 16 * kPhasorBlockStride;      // bytes per half (bands 0-1 / 2-3 of a chunk)
constexpr int kPhasorBytes = 2 * kPhasorHalfStride;

// Work list of the MFMA score kernels, built on the device from the sequence lengths by one workgroup of a multiple of
// 64 threads: [0] the kernel's shared item counter (zeroed here), [1] entries per (layer, KV head), from
// kWorkHeader on one (sequence, chunk) pair per chunk of chunk_keys keys that exists.  The first wave finds where each of
// 64 runs of sequences starts with a shuffle scan (one thread adding 64 LDS entries one after the other took 3 us),
// then every run's pairs are written by one lane of each wave.
constexpr int kWorkHeader = 4;
__device__ __forceinline__ void build_work_list(const int32_t *seq_len, int n_seqs, int max_seq_len, int chunk_keys,
                                                int32_t *work)
{
    __shared__ int start[64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int seg = (n_seqs + 63) / 64, s0 = min(n_seqs, lane * seg), s1 = min(n_seqs, s0 + seg);
    auto chunks = [&](int s) { return (clamp_len(seq_len[s], max_seq_len) + chunk_keys - 1) / chunk_keys; };
    if (wave == 0) {
        int cnt = 0;
        for (int s = s0; s < s1; ++s) cnt += chunks(s);
        int cum = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(cum, o, 64);
            if (lane >= o) cum += t;
        }
        start[lane] = cum - cnt;
        if (lane == 63) {
            work[0] = 0;
            work[1] = cum;
        }
    }
    __syncthreads();
    int o = start[lane];
    for (int s = s0; s < s1; ++s) {
        const int n = chunks(s);
        for (int ch = wave; ch < n; ch += n_waves) {
            work[kWorkHeader + 2 * (o + ch)] = s;
            work[kWorkHeader + 2 * (o + ch) + 1] = ch;
        }
        o += n;
    }
}

// The stretches of a batch (tri_items.h): how many tiles a (layer, KV head) has, how many of them lie ahead of each sequence, and where the
// first `first` stretches begin, worked out by one workgroup of kStretchSeqs / 2 threads.
struct StretchStart {
    int32_t lh, s, off, entry, tiles;   // layer << 16 | KV head; from tile off of sequence s on; which of its head-instance's moments; length
};
constexpr int kStretchInts = 5;
struct StretchPlan {   // in the phasor table's area, behind the table
    int32_t before[kStretchSeqs];
    StretchStart start[1];
};
constexpr size_t kStretchPlanAt = 48 * 1024;
// where stretch i begins
template <typename Ints>
__device__ __forceinline__ StretchStart stretch_start(uint32_t i, const Stretches &st, uint32_t per_lh, int n_seqs, uint32_t n_kv_heads, Ints before)
{
    const uint32_t begin = stretch_begin(st, i), lh = begin / per_lh, l = lh / n_kv_heads;
    const int r = (int)(begin - lh * per_lh);
    int s = 0;   // the last sequence with no more than r tiles ahead of it: r lies in it (those behind an empty one have as many)
    for (int step = n_seqs > 1 ? 1 << (31 - __builtin_clz(n_seqs - 1)) : 0; step > 0; step >>= 1)
        if (s + step < n_seqs && before[s + step] <= r) s += step;
    const int off = r - before[s];
    return StretchStart{(int32_t)(l << 16 | (lh - l * n_kv_heads)), s, off, (int32_t)(i - stretch_of(st, begin - off)), (int32_t)(st.least + (i < st.longer ? 1 : 0))};
}
__device__ __forceinline__ void plan_stretches(const int32_t *seq_len, int n_seqs, int max_seq_len, int n_layers, int n_kv_heads, int entries, int most,
                                               int first, int waves, int32_t *work, StretchPlan *plan)
{
    __shared__ int before[kStretchSeqs], wave_sum[kStretchSeqs / 128], wave_most[kStretchSeqs / 128];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto tiles = [&](int s) { return s < n_seqs ? (clamp_len(seq_len[s], max_seq_len) + kStretchTile - 1) / kStretchTile : 0; };
    const int t0 = tiles(2 * tid), t1 = tiles(2 * tid + 1);
    int cum = t0 + t1, longest = max(t0, t1);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(cum, o, 64);
        if (lane >= o) cum += t;
        longest = max(longest, __shfl_xor(longest, o, 64));
    }
    if (lane == 63) wave_sum[wave] = cum, wave_most[wave] = longest;
    __syncthreads();
    int per_lh = 0;
#pragma unroll
    for (int w = 0; w < kStretchSeqs / 128; ++w) {
        if (w < wave) cum += wave_sum[w];
        per_lh += wave_sum[w];
        longest = max(longest, wave_most[w]);
    }
    before[2 * tid] = cum - t0 - t1;
    before[2 * tid + 1] = cum - t1;
    if (2 * tid < n_seqs) plan->before[2 * tid] = cum - t0 - t1;
    if (2 * tid + 1 < n_seqs) plan->before[2 * tid + 1] = cum - t1;
    const uint32_t total = (uint32_t)per_lh * (uint32_t)(n_layers * n_kv_heads);
    const Stretches st = stretches_of(total, 1, stretches_wanted(total, longest, entries, most, first, waves));
    if (tid == 0) work[0] = 0, work[1] = per_lh, work[2] = (int)st.count;
    __syncthreads();
    for (int i = tid; i < first; i += kStretchSeqs / 2)
        plan->start[i] = i < (int)st.count ? stretch_start(i, st, per_lh, n_seqs, n_kv_heads, before) : StretchStart{};
}

// (cos, sin) of band f at relative position r, in double
__device__ __forceinline__ void relative_phasor(double theta, int f, int r, float *c, float *s)
{
    constexpr double kTwoPiD = 6.283185307179586476925286766559;
    double x = (double)r * (pow(theta, -2.0 * (double)f / (double)kHeadDim) / kTwoPiD);
    x -= floor(x);
    double sd, cd;
    sincospi(2.0 * x, &sd, &cd);
    *c = (float)cd;
    *s = (float)sd;
}
// Entry t of the sixteen-lane kernel's table, (half hf, chunk b, r) = (cos, sin) of bands 4b+2hf, 4b+2hf+1 at relative position
// r, at byte hf * kPhasorHalfStride + b * kPhasorBlockStride + 16 r.  The fold kernel writes it with kFastTablePhasors extra
// threads (a launch of its own took 4.6 us), a phasor each (neighbouring bands in neighbouring threads).
constexpr int kFastTablePhasors = 4 * 16 * kPhasorRange;
__device__ __forceinline__ void fast_phasor(double theta, int t, float2 *out)
{
    const int e = t / 2, r = e % kPhasorRange, b = (e / kPhasorRange) % 16, hf = e / (kPhasorRange * 16), f = 4 * b + 2 * hf + t % 2;
    float2 v;
    relative_phasor(theta, f, r, &v.x, &v.y);
    out[((hf * kPhasorHalfStride + b * kPhasorBlockStride) / 16 + r) * 2 + t % 2] = v;
}
// bf16 keys; G in 1..8.  launch_score_lane (tri_score_lane.hip): the general one; launch_score_fast (tri_score_mfma.hip): paged,
// interleaved pairs, pre-RoPE.  Each has its own phasor table layout.
tri_status launch_score_fast(int G, const ScoreArgs &sa, hipStream_t st);
template <int G>
tri_status launch_score_lane(const ScoreArgs &sa, bool half_split, hipStream_t st);
// (each group size is a compilation of its own)
template <>
tri_status launch_score_lane<1>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<2>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<3>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<4>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<5>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<6>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<7>(const ScoreArgs &sa, bool half_split, hipStream_t st);
template <>
tri_status launch_score_lane<8>(const ScoreArgs &sa, bool half_split, hipStream_t st);
// The general kernel's table of e^{i w r}: entry (band pair bp, r) = (cos, sin) of bands 2bp and 2bp+1 at relative position r, at byte
// bp * kLanePairStride + 16 r.  The fold kernel writes it with kLaneTablePhasors extra threads.
constexpr int kLaneRange = 88;                                  // relative positions 0 .. 87: what LDS has room for
constexpr int kLanePairStride = kLaneRange * 16 + 16;           // bytes per band pair (16 bytes of skew)
constexpr int kLanePhasorBytes = (kBands / 2) * kLanePairStride;
constexpr int kLaneTablePhasors = kBands * kLaneRange;
__device__ __forceinline__ void lane_phasor(double theta, int t, float2 *out)
{
    const int e = t / 2, r = e % kLaneRange, bp = e / kLaneRange;
    float2 v;
    relative_phasor(theta, 2 * bp + t % 2, r, &v.x, &v.y);
    out[(bp * (kLanePairStride / 16) + r) * 2 + t % 2] = v;
}
// ints the MFMA kernel's work list takes: a header and one (sequence, chunk) pair per possible chunk
inline size_t fast_work_ints(int64_t n_seqs, int64_t max_seq_len)
{
    return kWorkHeader + 2 * (size_t)n_seqs * (size_t)((max_seq_len + kMinChunk - 1) / kMinChunk);
}

}  // namespace tri
