// Scoring kernels: table fold, per-key score, moments, z-score + max over the GQA group.
//
// Algebra (Sections 4.1-4.2, Appendix B.2).  With q = E[q_f], k = k_f complex, x = p_q + delta - p_k:
//   ||q|| ||k|| cos(omega x + arg q - arg k) = Re( q conj(k) e^{i omega x} )
// and the average over the offsets delta in D is linear, so
//   S~_trig(k) = Re sum_f  Qhat_f * conj( k_f e^{i omega_f p_k} ),
//   Qhat_f = E[q_f] * (1/|D|) sum_delta e^{i omega_f delta} * e^{i omega_f p_q}.
// The norm term does not depend on the offset: S_norm(k) = sum_f c_f |k_f|, c_f = E||q_f|| - ||E[q_f]||.
// The fold kernel builds (Re Qhat, Im Qhat, c) per (layer, sequence, query head, band) in double;
// the score kernel then needs, per key and band, one rotation of the key by its own position,
// one modulus, and three FMAs per query head -- independent of |D|.
#include <algorithm>
#include <atomic>

#include "tri_score_common.h"

namespace tri {

namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;

struct FoldArgs {
    const float *centers;   // [L][Hq][F][3]
    float *table;           // [L][S][Hkv][F][3][G]
    double *band_rev;       // [F]
    const int32_t *cur_pos; // [S]
    double theta;
    int32_t n_off;
    int32_t variant;        // tri_score_variant
    int32_t S, Hq, Hkv, G;
    int32_t fold_seqs;      // sequences per workgroup
    int32_t seq_blocks;     // workgroups per (layer, KV head)
    int32_t band_shift;     // each once per 64 >> band_shift parts of 1 << band_shift bands
    int32_t extra, extra_each;   // workgroups for everything but the tables, and how many of them a layer's row holds
    int32_t lane_kernel;    // layout of the phasor table: that of tri_score_lane.hip or the sixteen-lane kernel's
    float4 *phasors;        // relative-position phasor table of the MFMA score kernel, filled in by extra workgroups
    StretchPlan *stretches; // stretches of the general MFMA kernel, or NULL; its moments are cleared here
    int64_t offsets[kMaxOffsets];
    const int32_t *seq_len; // [S]
    int32_t *work;          // work list of the MFMA score kernels, or NULL when the generic kernel runs
    double *partials;       // [L][S][Hkv][n_entries][2G]
    int32_t chunk_keys;     // keys per entry of that list
    int32_t n_stretches, n_first, n_entries, stretch_waves;
    int32_t L;
    int32_t max_seq_len;
};

// exp(2 pi i * frac(t * rev)) in double; t * rev is exact enough for |t| < 2^62 * 2^-53 relative
__device__ __forceinline__ void unit_phasor(double t, double rev, double *c, double *s)
{
    double x = t * rev;
    x -= floor(x);
    sincospi(2.0 * x, s, c);   // (no reduction of large arguments, which the general function carries along)
}

constexpr int kFoldSeqs = 8;      // sequences per workgroup, more where workgroups abound,
constexpr int kFoldSeqsMost = 32; // at most this many
constexpr int kFoldThreads = 512;
constexpr int kBandShift = 6;
static_assert(kBands == 1 << kBandShift, "bands");

// The folded tables of one (layer, KV head), fold_seqs sequences and 1 << band_shift bands per workgroup: grid (Hkv * seq_blocks *
// (64 >> band_shift) + extra_each, L), block 512.  The phasors a fold needs depend on the band and on the offsets or the query position only, and every
// workgroup evaluates them for itself: (offset or sequence, band) pairs spread over its threads, three double-precision
// sincos per thread for 16 offsets and 8 sequences and all bands, the offsets then added in their order by one thread per band.  The
// kernel is bound by that chain of software sincos and pow, not by its work: a launch of its own for the phasors, in which one
// thread per band went through the offsets one after the other, and a second one for the tables took 5.8 + 4.6 us (10.6 + 5.1
// with 32 offsets); with this one a step on one head's 4096 keys takes 35.6 us instead of 39.5, on one layer of eight heads
// x 32768 keys 74.3 instead of 78.4.  Where workgroups are few the bands of each go to two or four (launch_score), a sincos per thread: the
// same steps 22.6 -> 22.2 and 47.4 -> 46.9 us, 32 x 2176 keys, scores and selection, 26.4 -> 26.0.  SPLIT: only there are the
// bands of a workgroup a variable (a constant saves the others 0.15 us: scores of 36 x 8 x 300 fp32 keys 28.2 -> 28.0, bf16 25.35 -> 25.2).
// The extra workgroups have nothing to do with the tables: the first writes the band frequencies, the second lists the stretches or
// chunks of the MFMA score kernels (a launch of its own would cost more than the list; behind the first one's pow it cost small
// calls 0.5 us), those after it fill the MFMA score kernel's phasor table when it needs one, an entry per thread.  They are spread over the
// layers' rows.  (All of them in every row, where only the first row's had work, is a grid of 528 workgroups instead of 165 for 33 x 4
// head-instances: scores of 64 keys each 17.4 us instead of 14.7, 64 x 1000 keys 19.3 / 17.3, 40 x 2 x 568 at G = 8 22.8 / 20.6.)
template <bool SPLIT>
__global__ __launch_bounds__(kFoldThreads) void fold_kernel(FoldArgs a)
{
    extern __shared__ __align__(16) double fold_lds[];
    double (*const off_ph)[2] = reinterpret_cast<double (*)[2]>(fold_lds);   // e^{i w delta_j}: entry (j, band); row 0 then holds their mean
    const int tid = threadIdx.x, band_shift = SPLIT ? a.band_shift : kBandShift, bands = 1 << band_shift, parts = kBands >> band_shift;
    double (*const cur_ph)[2] = off_ph + a.n_off * bands;                    // e^{i w cur_pos[s]}
    const int n_fold = a.Hkv * a.seq_blocks * parts, l = blockIdx.y;
    // Section 2.1: omega_f = theta^(-2f/d); kept as revolutions per position.  (kFoldThreads is a multiple of the
    // workgroup's bands: a thread's band is the same in every loop below)
    const bool folds = (int)blockIdx.x < n_fold;   // (uniform over the workgroup)
    const int extra = folds ? -1 : l * a.extra_each + (int)blockIdx.x - n_fold;
    if (extra >= a.extra) return;
    if (extra == 1) {
        if (a.stretches) plan_stretches(a.seq_len, a.S, a.max_seq_len, a.L, a.Hkv, a.n_entries, a.n_stretches, a.n_first, a.stretch_waves, a.work, a.stretches);
        else if (a.work) build_work_list(a.seq_len, a.S, a.max_seq_len, a.chunk_keys, a.work);
        return;
    }
    if (extra > 1) {
        const int t = (extra - 2) * kFoldThreads + tid;   // (an entry holds two bands: a thread each)
        if (a.lane_kernel) lane_phasor(a.theta, t, reinterpret_cast<float2 *>(a.phasors));
        else fast_phasor(a.theta, t, reinterpret_cast<float2 *>(a.phasors));
        return;
    }
    const int f0 = extra == 0 ? 0 : (blockIdx.x & (parts - 1)) << band_shift, f = extra == 0 ? tid % kBands : f0 + (tid & (bands - 1));
    const double rev = pow(a.theta, -2.0 * (double)f / (double)kHeadDim) / kTwoPi;
    if (extra == 0) {
        if (tid < kBands) a.band_rev[f] = rev;
        return;
    }
    const int x = blockIdx.x >> (kBandShift - band_shift), h = x / a.seq_blocks, sb = x - h * a.seq_blocks;
    // the thread's (band, query head) pair, the head fastest: neighbouring threads write neighbouring entries of [F][3][G].  Its
    // statistics are asked for ahead of the phasors.
    static_assert(kBands * kMaxGroup <= kFoldThreads, "a pair per thread");
    const int fl = min(tid / a.G, bands - 1), fb = f0 + fl, g = tid - tid / a.G * a.G;
    const float *ct = a.centers + (((int64_t)l * a.Hq + h * a.G + g) * kBands + fb) * 3;
    const float c0 = ct[0], c1 = ct[1], c2 = ct[2];
    const int s0 = sb * a.fold_seqs, n_seq = min(a.S - s0, a.fold_seqs);
    if (a.stretches)   // an entry that no stretch of the head-instance's writes counts as nothing
        for (int j = f0 >> band_shift; j < n_seq; j += parts) {
            double *const m = a.partials + (((int64_t)l * a.S + s0 + j) * a.Hkv + h) * a.n_entries * (2 * a.G);
            for (int k = tid; k < a.n_entries * 2 * a.G; k += kFoldThreads) m[k] = 0.0;
        }
    for (int k = tid; k < (a.n_off + n_seq) * bands; k += kFoldThreads) {   // (the sequences' phasors lie behind the offsets')
        const int j = k >> band_shift;
        double c, s;
        unit_phasor(j < a.n_off ? (double)a.offsets[j] : (double)a.cur_pos[s0 + j - a.n_off], rev, &c, &s);
        off_ph[k][0] = c;
        off_ph[k][1] = s;
    }
    __syncthreads();
    if (tid < bands) {   // mean over the offsets, in their order
        double er = 0.0, ei = 0.0;
#pragma unroll 8
        for (int j = 0; j < a.n_off; ++j) {
            er += off_ph[j * bands + tid][0];
            ei += off_ph[j * bands + tid][1];
        }
        off_ph[tid][0] = er / (double)a.n_off;
        off_ph[tid][1] = ei / (double)a.n_off;
    }
    __syncthreads();
    // the ablation variants (Section 5) only change the table: no trig part, no norm part, or the norm
    // part without its (1 - R_f) weight, i.e. S_norm^(0) of Section 4.1
    const bool trig_on = a.variant != TRI_SCORE_NORM_ONLY, norm_on = a.variant != TRI_SCORE_TRIG_ONLY;
    if (tid < bands * a.G) {
        const double er = off_ph[fl][0], ei = off_ph[fl][1];
        const double qr = (double)c0, qi = (double)c1, qa = (double)c2;
        const double ar = trig_on ? qr * er - qi * ei : 0.0, ai = trig_on ? qr * ei + qi * er : 0.0;
        const double cn = !norm_on ? 0.0 : a.variant == TRI_SCORE_NORM_UNWEIGHTED ? qa : qa - hypot(qr, qi);
        for (int j = 0; j < n_seq; ++j) {
            const double c = cur_ph[j * bands + fl][0], sn = cur_ph[j * bands + fl][1];
            float *t = a.table + (((((int64_t)l * a.S + s0 + j) * a.Hkv + h) * kBands + fb) * 3) * a.G;
            t[0 * a.G + g] = (float)(ar * c - ai * sn);
            t[1 * a.G + g] = (float)(ar * sn + ai * c);
            t[2 * a.G + g] = (float)cn;
        }
    }
}

template <typename T>
struct Elem;
template <>
struct Elem<float> {
    static constexpr int kRow16 = 32;  // 16-byte chunks per key row
};
template <>
struct Elem<uint16_t> {
    static constexpr int kRow16 = 16;
};

// One band of one key: rotate the key by its own position, take its modulus, and add the
// three products per query head.  tb: this band's [3][G] table entries, in LDS.
template <int G>
__device__ __forceinline__ void band_update(float (&acc)[G], const float *tb, double pd,
                                            double rev, float re, float im)
{
    double xr = pd * rev;
    float x = (float)__builtin_amdgcn_fract(xr);   // phase in revolutions, [0, 1]
    float sn = __builtin_amdgcn_sinf(x);           // v_sin_f32 / v_cos_f32 take revolutions
    float cs = __builtin_amdgcn_cosf(x);
    float kr = re * cs - im * sn;
    float ki = re * sn + im * cs;
    float m = __builtin_amdgcn_sqrtf(re * re + im * im);
#pragma unroll
    for (int g = 0; g < G; ++g)
        acc[g] = fmaf(tb[0 * G + g], kr, fmaf(tb[1 * G + g], ki, fmaf(tb[2 * G + g], m, acc[g])));
}

// grid (n_tiles, S*Hkv, L), block 512: a tile of one or two parts of 128 keys, four threads per key (a quarter of the bands each, the
// quarter the same for a whole wave, so that the table entries, in LDS, are read by a wave at one address).  Keys are staged through
// LDS so that global loads are coalesced 16-byte accesses while each thread ends up with its quarter of one key.  The 68 KB that 128
// fp32 keys take let two workgroups share a CU: one's loads overlap the other's arithmetic, and the second part's loads go out ahead of the
// first part's arithmetic.
// Against 256 keys in one workgroup of 1024 threads, alone on its CU, with the table as scalar operands (whose loads a wave waited for every
// other band): fp32, whole steps, 192 heads of 32768 keys 1252 -> 838 us at G = 4, 1044 -> 697 at G = 1, 1600 -> 998 at G = 8; scores and selection
// of 288 heads of 2176 146 -> 96; scores of 320 ragged ones up to 20011 865 -> 535; bf16 in blocks of 8, scores of 288 heads of 2176 101 -> 70 at G = 4,
// 55 -> 55 at G = 1, of 16384 669 -> 410 and 332 -> 311.  (That one: one thread per key, one wave per SIMD, 3595 us for 288 heads of 32768 keys;
// four 1730.)  128 registers, none spilled.
constexpr int kScoreSplit = 4, kPartKeys = 128, kScoreThreads = kPartKeys * kScoreSplit;
template <int G, typename T, int PAIRS>
__global__ __launch_bounds__(kScoreThreads, 4) void score_kernel(ScoreArgs a)
{
    constexpr int ROW16 = Elem<T>::kRow16, kLoads = kPartKeys * ROW16 / kScoreThreads;
    constexpr int STRIDE16 = ROW16 + 1;   // odd number of 16-byte units: conflict-free row reads
    extern __shared__ uint4 lds[];        // a part's keys; later its quarters' sums
    __shared__ __align__(16) float tab[kBands * 3 * G];
    __shared__ double rev[kBands];
    __shared__ int64_t k_at[kScoreTile], p_at[kScoreTile];   // paged: where the tile's keys and positions are
    __shared__ double red[kPartKeys / 64][2 * G];

    const CacheView &c = a.c;
    const int tid = threadIdx.x, key = tid % kPartKeys;
    const int quarter = __builtin_amdgcn_readfirstlane(tid / kPartKeys);
    const int tile = blockIdx.x;
    const int s = blockIdx.y / c.n_kv_heads, h = blockIdx.y % c.n_kv_heads;
    const int l = blockIdx.z;
    const int N = clamp_len(c.seq_len[s], c.max_seq_len);
    const int n0 = tile * a.chunk_keys, n1 = min(N, n0 + a.chunk_keys);
    if (n0 >= N) return;
    const int64_t inst = ((int64_t)l * c.n_seqs + s) * c.n_kv_heads + h;

    const T *kbase = (const T *)c.k;
    // Contiguous keys are a product away from the first; paged ones are looked up by one thread each.  (A lookup and two 64-bit products
    // by each of the sixteen or thirty-two threads that load a row: 288 heads of 16384 bf16 keys in blocks of 8, scores, 430 us at G = 1
    // against 311 now, 525 / 410 at G = 4; fp32 ones 676 / 528 and 785 / 597.)
    const bool paged = c.block_shift >= 0;
    const int64_t k_base = (int64_t)l * c.stride_layer + (int64_t)h * c.stride_head + (paged ? 0 : (int64_t)s * c.stride_sb);
    const int64_t p_base = (int64_t)l * c.pos_stride_layer + (int64_t)h * c.pos_stride_head + (paged ? 0 : (int64_t)s * c.pos_stride_sb);
    if (paged) {
        const int n = n0 + tid;
        if (tid < kScoreTile && n < n1) {
            const int b = c.block_table[(int64_t)s * c.max_blocks + (n >> c.block_shift)], in = n & ((1 << c.block_shift) - 1);
            k_at[tid] = (int64_t)b * c.stride_sb + slot_offset(c, in);
            p_at[tid] = (int64_t)b * c.pos_stride_sb + in;
        }
        __syncthreads();
    }
    uint4 kd[kLoads];
    int p_next = 0;
    auto load = [&](int m0) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int ci = i * kScoreThreads + tid, n = m0 + ci / ROW16;
            kd[i] = make_uint4(0u, 0u, 0u, 0u);
            if (n < N) kd[i] = reinterpret_cast<const uint4 *>(kbase + k_base + (paged ? k_at[n - n0] : slot_offset(c, n)))[ci % ROW16];
        }
        const int n = m0 + key;
        if (n < N && !c.k_rotated) p_next = c.pos[p_base + (paged ? p_at[n - n0] : n)];   // a post-RoPE key needs no rotation
    };
    load(n0);
    {
        const float *src = a.table + inst * (kBands * 3 * G);
        for (int k = tid; k < kBands * 3 * G; k += kScoreThreads) tab[k] = src[k];
        if (tid < kBands) rev[tid] = a.band_rev[tid];
    }
    // Quarter 0: the key's scores of the part and of the part before, for the moments.  (The sums themselves, held as doubles in every
    // thread, took four times the registers: 4 to 24 spilled with six and more query heads, 64 heads of 8192 fp32 keys, half-split, scores, 93.5,
    // 111.9 and 112.9 us at G = 6, 7, 8 against 76.6, 80.8 and 86.2.)
    static_assert(kScoreTile <= 2 * kPartKeys, "two parts at most");
    float last[G], before[G];
#pragma unroll
    for (int g = 0; g < G; ++g) last[g] = before[g] = 0.f;
    const int Hq = c.n_kv_heads * G;
    float *rw = a.raw + (((int64_t)l * c.n_seqs + s) * Hq + (int64_t)h * G) * c.max_seq_len;
    const float *const tb = tab;
    for (int m0 = n0; m0 < n1; m0 += kPartKeys) {
        if (m0 > n0) __syncthreads();   // the sums of the part before have been read
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int ci = i * kScoreThreads + tid;
            lds[ci / ROW16 * STRIDE16 + ci % ROW16] = kd[i];
        }
        const double pd = (double)p_next;
        __syncthreads();
        if (m0 + kPartKeys < n1) load(m0 + kPartKeys);   // on its way during this part's arithmetic
        const int n = m0 + key;
        const bool valid = n < N;
        float acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = 0.f;
        const uint4 *row = lds + key * STRIDE16;
        constexpr int kBandsEach = kBands / kScoreSplit;

        if constexpr (sizeof(T) == 2 && PAIRS == TRI_PAIR_INTERLEAVED) {
#pragma unroll 2
            for (int j = quarter * (kBandsEach / 4); j < (quarter + 1) * (kBandsEach / 4); ++j) {
                uint4 q = row[j];
                const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int f = 4 * j + i;
                    band_update<G>(acc, tb + f * 3 * G, pd, rev[f], bf16_lo(w[i]), bf16_hi(w[i]));
                }
            }
        } else if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int j = quarter * (kBandsEach / 8); j < (quarter + 1) * (kBandsEach / 8); ++j) {
                uint4 qr = row[j], qi = row[j + 8];
                const uint32_t wr[4] = {qr.x, qr.y, qr.z, qr.w}, wi[4] = {qi.x, qi.y, qi.z, qi.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int f = 8 * j + 2 * i;
                    band_update<G>(acc, tb + f * 3 * G, pd, rev[f], bf16_lo(wr[i]), bf16_lo(wi[i]));
                    band_update<G>(acc, tb + (f + 1) * 3 * G, pd, rev[f + 1], bf16_hi(wr[i]), bf16_hi(wi[i]));
                }
            }
        } else if constexpr (PAIRS == TRI_PAIR_INTERLEAVED) {
#pragma unroll 2
            for (int j = quarter * (kBandsEach / 2); j < (quarter + 1) * (kBandsEach / 2); ++j) {
                uint4 q = row[j];
                int f = 2 * j;
                band_update<G>(acc, tb + f * 3 * G, pd, rev[f], __uint_as_float(q.x), __uint_as_float(q.y));
                band_update<G>(acc, tb + (f + 1) * 3 * G, pd, rev[f + 1], __uint_as_float(q.z), __uint_as_float(q.w));
            }
        } else {
#pragma unroll 2
            for (int j = quarter * (kBandsEach / 4); j < (quarter + 1) * (kBandsEach / 4); ++j) {
                uint4 qr = row[j], qi = row[j + 16];
                const uint32_t wr[4] = {qr.x, qr.y, qr.z, qr.w}, wi[4] = {qi.x, qi.y, qi.z, qi.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int f = 4 * j + i;
                    band_update<G>(acc, tb + f * 3 * G, pd, rev[f], __uint_as_float(wr[i]), __uint_as_float(wi[i]));
                }
            }
        }

        // the quarters' sums together, in their order
        __syncthreads();   // nobody reads the keys any more
        float *const sums = reinterpret_cast<float *>(lds);   // [quarter - 1][head][key]
        if (quarter > 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) sums[((quarter - 1) * G + g) * kPartKeys + key] = acc[g];
        }
        __syncthreads();
        if (quarter == 0) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
#pragma unroll
                for (int q = 1; q < kScoreSplit; ++q) acc[g] += sums[((q - 1) * G + g) * kPartKeys + key];
                before[g] = last[g];
                last[g] = valid ? acc[g] : 0.f;
                if (valid) rw[(int64_t)g * c.max_seq_len + n] = acc[g];
            }
        }
    }
    // the tile's sum and sum of squares per query head (double, fixed order)
    if (quarter == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const double x0 = (double)before[g], x1 = (double)last[g];
            double v1 = x0 + x1, v2 = x0 * x0 + x1 * x1;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                v1 += __shfl_xor(v1, o, 64);
                v2 += __shfl_xor(v2, o, 64);
            }
            if ((tid & 63) == 0) {
                red[tid >> 6][g] = v1;
                red[tid >> 6][G + g] = v2;
            }
        }
    }
    __syncthreads();
    if (tid < 2 * G) a.partials[(inst * a.n_tiles + tile) * (2 * G) + tid] = red[0][tid] + red[1][tid];
}

struct FinalArgs {
    const float *raw;     // [inst][G][Nmax]  (instance-major because Hq = Hkv * G)
    float *final_;        // [inst][Nmax]
    const int32_t *seq_len;
    int32_t n_seqs, n_kv_heads, max_seq_len;
    int32_t key_blocks;   // workgroups per head-instance
    const double *partials;   // [inst][n_tiles][2G]: moments of tile_keys keys each
    int32_t n_tiles, tile_keys;
};

// grid (instances * ceil(Nmax/1024)), block 256: Section 4.3, mu_g and sigma_g over the N keys (population sigma) from the moments, which
// every workgroup adds up for itself, and S_final(k) = max_g (S~(g)(k) - mu_g) / sigma_g.  Four keys per thread, all their scores
// and the moments loaded before the first is used: rows of an odd length read one score at a time took 24 x 5 x 8 head-instances of
// up to 20011 keys, scores, 834 us against 806.  The statistics in a launch of their own ahead of this one: scores and selection of
// 288 x 2176 interleaved keys 77.4 us against 75.5, 32 x 2176 28.1 / 26.3, 2304 x 2176 344.7 / 339.1, 9216 1305 / 1289, half-split 1335.0 / 1334.4.
template <int G>
__global__ __launch_bounds__(256) void final_kernel(FinalArgs a)
{
    __shared__ double zst[2 * G], zpart[32 * G];
    const int inst = blockIdx.x / a.key_blocks, kb = blockIdx.x - inst * a.key_blocks;
    const int s = (inst / a.n_kv_heads) % a.n_seqs;
    const double *pt = a.partials + (int64_t)inst * a.n_tiles * (2 * G);
    const Moments ahead = moments_ahead<G>(pt, a.n_tiles, threadIdx.x);
    const int N = clamp_len(a.seq_len[s], a.max_seq_len);
    if (kb * 1024 >= N) return;
    const int n0 = (kb * 256 + threadIdx.x) * 4, n = min(n0, N - 1);   // (every thread takes part in block_stats)
    // 16-byte accesses within a row (both arrays may be the caller's, who owes floats' alignment only: the hardware asks for no more)
    typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
    const bool vec = n + 3 < a.max_seq_len;
    const float *rw = a.raw + (int64_t)inst * G * a.max_seq_len;
    float v[G][4];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float *row = rw + (int64_t)g * a.max_seq_len;
        if (vec) {
            const float4u t = *reinterpret_cast<const float4u *>(row + n);
            v[g][0] = t[0], v[g][1] = t[1], v[g][2] = t[2], v[g][3] = t[3];
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[g][k] = row[min(n + k, N - 1)];
        }
    }
    block_stats<G>(ahead, pt, moment_entries(a.n_tiles, a.tile_keys, N), N, threadIdx.x, zpart, zst);
    if (n0 >= N) return;
    float best[4];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const ZParams zp = z_params(zst[2 * g], zst[2 * g + 1]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float z = z_score(v[g][k], zp);
            best[k] = (g == 0) ? z : fmaxf(best[k], z);
        }
    }
    float *out = a.final_ + (int64_t)inst * a.max_seq_len + n;
    if (n + 3 < N) {
        *reinterpret_cast<float4u *>(out) = float4u{best[0], best[1], best[2], best[3]};
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (n + k < N) out[k] = best[k];
    }
}

template <int G, typename T>
tri_status launch_score_kernel(const tri_model &m, const ScoreArgs &sa, dim3 grid, hipStream_t st)
{
    const size_t lds = (size_t)kPartKeys * (Elem<T>::kRow16 + 1) * 16;
    if (m.pairs == TRI_PAIR_INTERLEAVED) {
        auto kern = score_kernel<G, T, TRI_PAIR_INTERLEAVED>;
        if (lds > 48 * 1024 &&
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return hip_status("hipFuncSetAttribute(score_kernel)");
        hipLaunchKernelGGL(kern, grid, dim3(kScoreThreads), lds, st, sa);
    } else {
        auto kern = score_kernel<G, T, TRI_PAIR_HALF>;
        if (lds > 48 * 1024 &&
            hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
            return hip_status("hipFuncSetAttribute(score_kernel)");
        hipLaunchKernelGGL(kern, grid, dim3(kScoreThreads), lds, st, sa);
    }
    return hip_status("score_kernel");
}

// MFMA kernels: bf16, a group of 16 slots never straddling a block, 32-bit offsets of the rows of such a group, or of a whole tile where there
// are no blocks.  (Those with 64-bit products or a base per 32 rows, for contiguous slots 64 to 128 MB apart: 0.3 us, 1 - 3 %, on every
// small call whose tiles are not all whole.)
bool mfma_path(const tri_cache &c, int G)
{
    return c.dtype == TRI_BF16 && (c.block_size == 0 || c.block_size >= 16) &&
           c.stride_slot * 2 * (c.block_size == 0 ? 32 : 16) < ((int64_t)1 << 31) &&
           ((int64_t)G * c.max_seq_len + 16) * 4 < ((int64_t)1 << 32);
}

template <int G>
tri_status launch_score_g(const tri_model &m, const tri_cache &c, ScoreArgs sa, const FinalArgs &fa,
                          float *final_out, MomentLayout *moments, bool lane_kernel, int n_cu, hipStream_t st)
{
    const int n_inst = m.n_layers * c.n_seqs * m.n_kv_heads;
    const bool fast = mfma_path(c, G);
    // Generic kernel: one part per workgroup where tiles of two would leave CUs without any or give a few twice the others' (scores: 8
    // heads of 8192 fp32 keys, a tile per CU, 19.4 us in tiles of two parts, 18.4 in tiles of one; one of 4096, a step, 26.2 / 22.9; 9 / 8 of
    // a tile: 32 bf16 heads of 2176 in blocks of 8, a step, 30.4 / 29.5, one of 80000 23.4 / 22.7, fp32 ones at G = 1 18.8 / 18.2, at G = 8 28.3 /
    // 29.8; with one or two query heads, which leave the CU more to wait for than to do, up to 3 / 2: 48 of 1900 at G = 2 22.6 / 21.6, 40 of
    // 2176 at G = 1 20.4 / 19.5, at G = 4 24.3 / 24.6), or need a longer last round of the two workgroups that a CU holds (128 of 1100 keys at
    // G = 4, 640 tiles of two or 1152 of one, 33.6 / 31.7, bf16 31.0 / 28.4; 48 of 2934 32.1 / 31.6).  Elsewhere there are only more moments to
    // add up and more workgroups (8 fp32 heads of 12288 23.9 / 24.9, of 16384 26.6 / 29.2, at G = 8 29.5 / 31.8 and 32.1 / 36.7; 56 of 2176 at
    // G = 8 31.9 / 35.5; bf16 27.7 / 30.7).  The moments of so many tiles lie in the area of the phasor table, which is not needed then: the
    // workspace's own has an entry per 256 keys.
    tri_status rc = TRI_OK;
    int tile_keys = fast ? sa.chunk_keys : kScoreTile;
    if (!fast) {
        const int64_t parts = (int64_t)n_inst * ((c.max_seq_len + kPartKeys - 1) / kPartKeys);
        const int64_t tiles = (int64_t)n_inst * ((c.max_seq_len + kScoreTile - 1) / kScoreTile);
        const int64_t slots = 2 * n_cu, part_rounds = (parts + slots - 1) / slots, tile_rounds = (tiles + slots - 1) / slots;
        const bool one = tiles * 4 <= (int64_t)n_cu * (G <= 2 ? 6 : 5) || part_rounds < 2 * tile_rounds;
        if (one && parts * 2 * G * (int64_t)sizeof(double) <= kPhasorAreaBytes) {
            tile_keys = kPartKeys;
            sa.partials = reinterpret_cast<double *>(const_cast<uint4 *>(sa.phasors));
        }
        sa.chunk_keys = tile_keys;
    }
    if (sa.stretches) tile_keys = 0;   // (sa.n_tiles: launch_score)
    else sa.n_tiles = (c.max_seq_len + tile_keys - 1) / tile_keys;
    hipEvent_t ev0, ev1;
    const bool timed = timing_next(&ev0, &ev1);
    if (timed) (void)hipEventRecord(ev0, st);
    if (lane_kernel) {
        rc = launch_score_lane<G>(sa, m.pairs == TRI_PAIR_HALF, st);
    } else if (fast) {
        rc = launch_score_fast(G, sa, st);
    } else {
        dim3 grid(sa.n_tiles, c.n_seqs * m.n_kv_heads, m.n_layers);
        rc = (c.dtype == TRI_BF16) ? launch_score_kernel<G, uint16_t>(m, sa, grid, st)
                                   : launch_score_kernel<G, float>(m, sa, grid, st);
    }
    if (timed) (void)hipEventRecord(ev1, st);
    if (rc != TRI_OK) return rc;
    if (moments) {
        moments->n_tiles = sa.n_tiles;
        moments->tile_keys = tile_keys;
        moments->partials = sa.partials;
    }
    if (!final_out) return rc;   // fused step: the selection forms the statistics from the moments itself
    FinalArgs fb = fa;
    fb.key_blocks = (c.max_seq_len + 1023) / 1024;
    if ((int64_t)fb.key_blocks * n_inst > (int64_t)0x7fffffff) {
        set_error("tri_score: %d head-instances x %d key blocks exceed the grid", n_inst, fb.key_blocks);
        return TRI_ERR_UNSUPPORTED;
    }
    const dim3 final_grid((uint32_t)((int64_t)fb.key_blocks * n_inst));
    fb.partials = sa.partials;
    fb.n_tiles = sa.n_tiles;
    fb.tile_keys = tile_keys;
    hipLaunchKernelGGL(final_kernel<G>, final_grid, dim3(256), 0, st, fb);
    rc = hip_status("final_kernel");
    return rc;
}

}  // namespace

// Compute units of the current GPU (asked once per GPU).
tri_status device_cus(int *n_cu)
{
    constexpr int kDevices = 64;
    static std::atomic<int> cached[kDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) {
        (void)hipGetLastError();
        set_error("score: no current device below %d", kDevices);
        return TRI_ERR_HIP;
    }
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            set_error("score: compute-unit count not available");
            return TRI_ERR_HIP;
        }
        cached[dev].store(n, std::memory_order_relaxed);
    }
    *n_cu = n;
    return TRI_OK;
}

tri_status launch_score(const tri_model &m, const float *centers, const tri_cache &c, float *final_out,
                        float *raw_out, char *ws, const Workspace &wl, MomentLayout *moments, hipStream_t st)
{
    const int G = m.n_q_heads / m.n_kv_heads;
    if (moments) *moments = MomentLayout{1, 1, reinterpret_cast<const double *>(ws + wl.partials)};
    if (c.max_seq_len <= 0 || c.n_seqs <= 0) return TRI_OK;
    FoldArgs fo{};
    fo.centers = centers;
    fo.table = reinterpret_cast<float *>(ws + wl.table);
    fo.band_rev = reinterpret_cast<double *>(ws + wl.band_rev);
    fo.cur_pos = c.cur_pos;
    fo.seq_len = c.seq_len;
    fo.work = mfma_path(c, G) ? reinterpret_cast<int32_t *>(ws + wl.work) : nullptr;
    // keys per work item: small batches are cut finer
    int n_cu = 0;
    tri_status rc = device_cus(&n_cu);
    if (rc != TRI_OK) return rc;
    int chunk_keys = kFastChunk;
    if (fo.work) {
        chunk_keys = item_keys((int64_t)m.n_layers * c.n_seqs * m.n_kv_heads, c.max_seq_len, n_cu);
    }
    fo.chunk_keys = chunk_keys;
    fo.max_seq_len = c.max_seq_len;
    fo.S = c.n_seqs;
    fo.fold_seqs = kFoldSeqs;
    while (fo.fold_seqs < kFoldSeqsMost && (int64_t)m.n_layers * m.n_kv_heads * ((c.n_seqs + 2 * fo.fold_seqs - 1) / (2 * fo.fold_seqs)) >= 2 * n_cu)
        fo.fold_seqs *= 2;
    fo.seq_blocks = (c.n_seqs + fo.fold_seqs - 1) / fo.fold_seqs;
    fo.band_shift = kBandShift;   // (half as many workgroups as CUs at most: 64 head-instances of 2176 keys, scores and selection, 29.5 -> 29.3 us with two parts)
    const int64_t n_fold = (int64_t)m.n_layers * m.n_kv_heads * fo.seq_blocks;
    while (fo.band_shift > 4 && n_fold * (kBands >> fo.band_shift) * 2 <= n_cu / 2) --fo.band_shift;
    fo.Hq = m.n_q_heads;
    fo.Hkv = m.n_kv_heads;
    fo.G = G;
    fo.theta = m.rope_theta;
    fo.n_off = m.n_offsets;
    fo.variant = m.score_variant;
    for (int j = 0; j < m.n_offsets; ++j) fo.offsets[j] = m.offsets[j];
    const bool sixteen = sixteen_lane_kernel(G, chunk_keys, (int64_t)m.n_layers * c.n_seqs * m.n_kv_heads, c.max_seq_len, n_cu,
                                             m.pairs == TRI_PAIR_HALF, c.block_size != 0, c.k_rotated != 0);
    const bool lane_kernel = fo.work && !sixteen;
    const int table_entries = !fo.work || c.k_rotated ? 0 : lane_kernel ? kLaneTablePhasors : kFastTablePhasors;
    fo.phasors = reinterpret_cast<float4 *>(ws + wl.phasors);
    const int64_t n_inst = (int64_t)m.n_layers * c.n_seqs * m.n_kv_heads;
    const int rounds = lane_kernel && c.n_seqs <= kStretchSeqs ? stretch_rounds(G, n_inst, c.max_seq_len, n_cu) : 0;
    if (rounds > 0) {
        const int count = rounds * n_cu, least = stretch_least(n_inst, c.max_seq_len, count), entries = stretch_entries(c.max_seq_len, least);
        if ((size_t)n_inst * entries * 2 * G * sizeof(double) <= wl.raw - wl.partials &&
            kStretchPlanAt + sizeof(StretchPlan) + (size_t)n_cu * sizeof(StretchStart) <= (size_t)kPhasorAreaBytes) {
            fo.stretches = reinterpret_cast<StretchPlan *>(ws + wl.phasors + kStretchPlanAt);
            fo.n_stretches = count;
            fo.n_first = n_cu;
            fo.stretch_waves = lane_waves(G, c.block_size != 0, c.k_rotated != 0, m.pairs == TRI_PAIR_HALF);
            fo.n_entries = entries;
            fo.partials = reinterpret_cast<double *>(ws + wl.partials);
            fo.L = m.n_layers;
        }
    }
    fo.lane_kernel = lane_kernel;
    const size_t fold_lds = (size_t)(m.n_offsets + std::min(fo.fold_seqs, c.n_seqs)) * kBands * 2 * sizeof(double);
    constexpr int kFoldLdsLimit = (kMaxOffsets + kFoldSeqsMost) * kBands * 2 * (int)sizeof(double);   // the most any call asks for
    auto fold = fo.band_shift < kBandShift ? fold_kernel<true> : fold_kernel<false>;
    if (fold_lds > 48 * 1024 &&
        hipFuncSetAttribute((const void *)fold, hipFuncAttributeMaxDynamicSharedMemorySize, kFoldLdsLimit) != hipSuccess)
        return hip_status("hipFuncSetAttribute(fold_kernel)");
    fo.extra = (fo.work ? 2 : 1) + table_entries / kFoldThreads;
    fo.extra_each = (fo.extra + m.n_layers - 1) / m.n_layers;
    hipLaunchKernelGGL(fold, dim3(m.n_kv_heads * fo.seq_blocks * (kBands >> fo.band_shift) + fo.extra_each, m.n_layers),
                       dim3(kFoldThreads), fold_lds, st, fo);
    if ((rc = hip_status("fold_kernel")) != TRI_OK) return rc;

    ScoreArgs sa{};
    sa.c = make_view(m, c);
    sa.table = fo.table;
    sa.band_rev = fo.band_rev;
    sa.raw = raw_out ? raw_out : reinterpret_cast<float *>(ws + wl.raw);
    sa.partials = reinterpret_cast<double *>(ws + wl.partials);
    sa.phasors = reinterpret_cast<const uint4 *>(ws + wl.phasors);
    sa.work = reinterpret_cast<int32_t *>(ws + wl.work);
    sa.n_layers = m.n_layers;
    sa.chunk_keys = chunk_keys;
    sa.stretches = reinterpret_cast<const int32_t *>(fo.stretches);
    sa.n_stretches = fo.n_stretches;
    sa.n_first = fo.n_first;
    sa.n_tiles = fo.n_entries;
    FinalArgs fa{};
    fa.raw = sa.raw;
    fa.final_ = final_out;
    fa.seq_len = c.seq_len;
    fa.n_seqs = c.n_seqs;
    fa.n_kv_heads = m.n_kv_heads;
    fa.max_seq_len = c.max_seq_len;
    switch (G) {
        case 1: return launch_score_g<1>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 2: return launch_score_g<2>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 3: return launch_score_g<3>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 4: return launch_score_g<4>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 5: return launch_score_g<5>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 6: return launch_score_g<6>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 7: return launch_score_g<7>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
        case 8: return launch_score_g<8>(m, c, sa, fa, final_out, moments, lane_kernel, n_cu, st);
    }
    set_error("group size %d not built (1 to 8)", G);
    return TRI_ERR_UNSUPPORTED;
}

}  // namespace tri
