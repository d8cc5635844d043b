// Offline calibration (Section 4.1; Appendix B.5): per (layer, query head, band) the complex mean
// of the pre-RoPE query samples and the mean of their moduli.
#include <algorithm>

#include "tri_internal.h"

namespace tri {

namespace {

struct CentersArgs {
    const void *q;  // [T][L][Hq][d]
    float *out;     // [L][Hq][F][3], or NULL: leave the sums in `sums`
    double *sums;   // [L][Hq][F][3] running sums (streaming calibration), or NULL
    int64_t T;
    int64_t heads;      // L * Hq
    int64_t first_head; // of this launch
    int32_t first;  // sums: 1 = overwrite, 0 = add to what is there
};

constexpr int kCenterThreads = 256;
constexpr int kCenterWaves = kCenterThreads / 64;

// (re, im) of eight bands of a head vector in 16-byte pieces, two (bf16) or four (fp32): with interleaved pairs one run of pieces, with
// half-split ones a run of real and one of imaginary parts.  The O lanes that share 8 O bands (from octet q0 on) take the pieces of a run in
// turn, so that a load instruction reads O neighbouring ones.  (A lane with its pieces side by side read every line by two or four
// instructions, some of them from memory again: 4096 tokens x 36 x 32 heads in bf16, interleaved, 298 -> 230 us, half-split equal; 18 x 32 in fp32
// 455 -> 204, half-split 278 -> 203.)
template <bool BF16, bool HALF, int O>
struct Octet {
    static constexpr int kPieces = BF16 ? 2 : 4, kPer = BF16 ? 8 : 4;   // pieces, elements per piece
    static constexpr int kRun = HALF ? kPieces / 2 : kPieces, kPieceBands = HALF ? kPer : kPer / 2;
    uint4 p[kPieces];
    // which of the O lanes' bands is the k-th of lane q
    static __device__ __forceinline__ int band(int q, int k) { return (k / kPieceBands * O + q) * kPieceBands + k % kPieceBands; }
    // ONCE: nobody else reads these bytes
    template <bool ONCE>
    __device__ __forceinline__ void load(const void *base, int64_t row, int q0, int q)
    {
#pragma unroll
        for (int k = 0; k < kPieces; ++k) {
            const int e = k / kRun * kBands + (q0 * kRun + k % kRun * O + q) * kPer;
            const char *at = (const char *)base + (row + e) * (BF16 ? 2 : 4);
            p[k] = ONCE ? load_stream16(at) : *reinterpret_cast<const uint4 *>(at);
        }
    }
    // element e of the 16 in load order
    __device__ __forceinline__ float at(int e) const
    {
        const int k = BF16 ? e >> 3 : e >> 2, r = BF16 ? (e & 7) >> 1 : e & 3;
        const uint32_t w = r == 0 ? p[k].x : r == 1 ? p[k].y : r == 2 ? p[k].z : p[k].w;
        if constexpr (!BF16) return __uint_as_float(w);
        return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
    }
    __device__ __forceinline__ float re(int k) const { return at(HALF ? k : 2 * k); }
    __device__ __forceinline__ float im(int k) const { return at(HALF ? 8 + k : 2 * k + 1); }
};

// sqrt of a sum of two squares of fp32 values, to within a unit in the last place of a double: one coupled Newton
// step and one correction by the residual on the hardware's reciprocal root (squares of fp32 values lie well inside
// double's range, so the scaling of the library's square root -- half of the kernel's time -- is not needed).
__device__ __forceinline__ double root(double s)
{
    const double r = __builtin_amdgcn_rsq(s);
    double g = s * r, h = 0.5 * r;
    const double d = fma(-h, g, 0.5);
    g = fma(g, d, g);
    h = fma(h, d, h);
    g = fma(fma(-g, g, s), h, g);
    return s > 0.0 && s < __builtin_inf() ? g : s;   // 0, infinity and NaN are their own
}

// The same for a sum that is not infinite, and NaN for one that is: one step of third order, and zero's root through a finite reciprocal
// instead of a comparison (a quarter of the clocks of a sample and band: 4096 tokens x 36 x 32 heads in bf16 262 -> 235 us half-split, 271 -> 230 interleaved).
__device__ __forceinline__ double finite_root(double s)
{
    const double r = __builtin_amdgcn_rsq(fmax(s, 1e-300));   // (the least square of an fp32 value other than 0 is 2e-90)
    const double g = s * r, e = fma(-g, r, 1.0);
    return fma(g * e, fma(0.375, e, 0.5), g);
}

// Block 256: thread = (band octet of the workgroup's O, token residue); O neighbouring threads read O/8 of a head vector with
// 16-byte loads, the next token's on their way while one is summed.  Grid: 8 / O workgroups per (layer, head), eight apart in the
// launch, so that those that share cache lines run on one XCD, side by side (workgroups go to the eight XCDs in turn).  Double sums in a fixed order: per thread
// over its tokens, then a butterfly over the residues of a wave, then the waves in order.
// Bound by its double arithmetic in bf16 (4096 tokens x 36 x 32 heads, 1.2 GB: 235 us half-split, 230 interleaved, 5.2 TB/s, where 271 both stood before
// finite_root and the order of the pieces) and by the memory stream in fp32 (18 x 32 heads, as many bytes: 203, 6.0 TB/s).
template <bool BF16, bool HALF, int O>
__global__ __launch_bounds__(kCenterThreads) void centers_kernel(CentersArgs a)
{
    constexpr int kResidues = kCenterThreads / O;
    __shared__ double part[kCenterWaves][8 * O][3];
    const int q = threadIdx.x % O, r = threadIdx.x / O, wave = threadIdx.x >> 6;
    constexpr int kParts = 8 / O;
    const int64_t lh = a.first_head + (int64_t)(blockIdx.x / (8 * kParts)) * 8 + blockIdx.x % 8;   // layer * Hq + head
    const int q0 = (int)(blockIdx.x / 8) % kParts * O;
    if (lh >= a.heads) return;
    double sre[8], sim[8], sab[8];
    auto row = [&](int64_t t) { return (t * a.heads + lh) * kHeadDim; };
    auto sum_up = [&](auto root_of) {
#pragma unroll
        for (int k = 0; k < 8; ++k) sre[k] = sim[k] = sab[k] = 0.0;
        Octet<BF16, HALF, O> cur, nxt;
        if (r < a.T) cur.template load<O == 8>(a.q, row(r), q0, q);
        for (int64_t t = r; t < a.T; t += kResidues) {
            nxt.template load<O == 8>(a.q, row(t + kResidues < a.T ? t + kResidues : t), q0, q);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const double x = (double)cur.re(k), y = (double)cur.im(k);
                sre[k] += x;
                sim[k] += y;
                sab[k] += root_of(fma(x, x, y * y));
                __builtin_amdgcn_sched_barrier(0);   // one band after the other: 84 registers instead of 116 (bf16, half-split)
            }
            cur = nxt;
        }
    };
    sum_up([](double v) { return finite_root(v); });
    bool finite = true;
#pragma unroll
    for (int k = 0; k < 8; ++k) finite = finite && sab[k] == sab[k];
    if (!finite) sum_up([](double v) { return root(v); });   // an infinite or not a numerical sample among the thread's
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
        for (int o = O; o < 64; o <<= 1) {   // lanes that differ in the residue only
            sre[k] += __shfl_xor(sre[k], o, 64);
            sim[k] += __shfl_xor(sim[k], o, 64);
            sab[k] += __shfl_xor(sab[k], o, 64);
        }
        if ((threadIdx.x & 63) < O) {
            const int f = Octet<BF16, HALF, O>::band(q, k);
            part[wave][f][0] = sre[k];
            part[wave][f][1] = sim[k];
            part[wave][f][2] = sab[k];
        }
    }
    __syncthreads();
    if (threadIdx.x < 8 * O) {
        const int f = threadIdx.x;
        double t0 = 0.0, t1 = 0.0, t2 = 0.0;
        for (int k = 0; k < kCenterWaves; ++k) {
            t0 += part[k][f][0];
            t1 += part[k][f][1];
            t2 += part[k][f][2];
        }
        const int64_t e = (lh * kBands + 8 * q0 + f) * 3;
        if (a.sums) {   // one thread owns the entry: a plain read-modify-write, chunks arrive in stream order
            double *o = a.sums + e;
            o[0] = a.first ? t0 : o[0] + t0;
            o[1] = a.first ? t1 : o[1] + t1;
            o[2] = a.first ? t2 : o[2] + t2;
        } else {
            float *o = a.out + e;
            o[0] = (float)(t0 / (double)a.T);
            o[1] = (float)(t1 / (double)a.T);
            o[2] = (float)(t2 / (double)a.T);
        }
    }
}

template <bool BF16, bool HALF>
tri_status launch_centers_t(CentersArgs a, int n_cu, hipStream_t st)
{
    // A workgroup per (layer, head) where that gives every CU two; else the bands are split over two, four or eight, which
    // read the same cache lines.  4096 tokens: 32 heads 89 -> 16 us with eight, 128 heads 91 -> 36 with four, 256 heads 102 ->
    // 65 with two; four per CU instead of two would take 128 heads to 46, 384 heads from 100 to 138.
    int parts = 1;
    while (parts < 8 && a.heads * parts < 2 * (int64_t)n_cu) parts *= 2;
    auto kern = parts == 1 ? centers_kernel<BF16, HALF, 8> : parts == 2 ? centers_kernel<BF16, HALF, 4>
                : parts == 4 ? centers_kernel<BF16, HALF, 2> : centers_kernel<BF16, HALF, 1>;
    // (a launch takes fewer than 2^32 threads along x: more heads than that, in turn)
    constexpr int64_t kMostHeads = (int64_t)1 << 23;
    for (a.first_head = 0; a.first_head < a.heads; a.first_head += kMostHeads) {
        const int64_t heads = std::min(a.heads - a.first_head, kMostHeads);
        hipLaunchKernelGGL(kern, dim3((uint32_t)((heads + 7) / 8 * 8 * parts)), dim3(kCenterThreads), 0, st, a);
        const tri_status rc = hip_status("centers_kernel");
        if (rc != TRI_OK) return rc;
    }
    return TRI_OK;
}

// sums / total tokens -> the statistics table
__global__ __launch_bounds__(256) void centers_finalize_kernel(const double *sums, double total, int64_t n, float *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = (float)(sums[i] / total);
}

struct DiagArgs {
    const float *q;      // [L][Hq][F][3]
    const float *k;      // [L][Hkv][F][3] or NULL
    float *mrl;          // [L][Hq][F]
    float *contrib;      // [L][Hq][F] or NULL
    int32_t *top;        // [L][Hq][K] or NULL
    int32_t Hq, Hkv, K;
};

// Appendix B.5: R_f = ||E[q_f]|| / E||q_f||.  Appendix B.7: C_f = E||q_f|| E||k_f|| and the K bands with the
// largest C_f (equal contributions: the lower band first).  grid (Hq, L), block F: thread = band.
__global__ __launch_bounds__(kBands) void diagnostics_kernel(DiagArgs a)
{
    __shared__ float cf[kBands];
    const int f = threadIdx.x, h = blockIdx.x, l = blockIdx.y;
    const int64_t e = ((int64_t)l * a.Hq + h) * kBands + f;
    const float *q = a.q + e * 3;
    const double ab = (double)q[2];
    a.mrl[e] = ab > 0.0 ? (float)(hypot((double)q[0], (double)q[1]) / ab) : 0.f;
    if (!a.k) return;
    const int G = a.Hq / a.Hkv;
    const float *k = a.k + (((int64_t)l * a.Hkv + h / G) * kBands + f) * 3;
    const float c = (float)(ab * (double)k[2]);
    if (a.contrib) a.contrib[e] = c;
    if (!a.top) return;
    cf[f] = c;
    __syncthreads();
    int rank = 0;
    for (int o = 0; o < kBands; ++o) rank += (cf[o] > c || (cf[o] == c && o < f)) ? 1 : 0;
    if (rank < a.K) a.top[((int64_t)l * a.Hq + h) * a.K + rank] = f;
}

}  // namespace

tri_status launch_centers(const tri_model &m, const void *q, int32_t q_dtype, int64_t n_tokens, float *out,
                          double *sums, int32_t first, hipStream_t st)
{
    int n_cu = 0;
    const tri_status rc = device_cus(&n_cu);
    if (rc != TRI_OK) return rc;
    const CentersArgs a{q, out, sums, n_tokens, (int64_t)m.n_layers * m.n_q_heads, 0, first};
    const bool half = m.pairs == TRI_PAIR_HALF;
    if (q_dtype == TRI_BF16) return half ? launch_centers_t<true, true>(a, n_cu, st) : launch_centers_t<true, false>(a, n_cu, st);
    return half ? launch_centers_t<false, true>(a, n_cu, st) : launch_centers_t<false, false>(a, n_cu, st);
}

tri_status launch_centers_finalize(const tri_model &m, const double *sums, int64_t total_tokens, float *out,
                                   hipStream_t st)
{
    const int64_t n = (int64_t)m.n_layers * m.n_q_heads * kBands * 3;
    hipLaunchKernelGGL(centers_finalize_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sums,
                       (double)total_tokens, n, out);
    return hip_status("centers_finalize_kernel");
}

tri_status launch_diagnostics(const tri_model &m, const float *q_centers, const float *k_centers, float *mrl,
                              float *contrib, int32_t top_k, int32_t *top, hipStream_t st)
{
    DiagArgs a{q_centers, k_centers, mrl, contrib, top, m.n_q_heads, m.n_kv_heads, top_k};
    hipLaunchKernelGGL(diagnostics_kernel, dim3(m.n_q_heads, m.n_layers), dim3(kBands), 0, st, a);
    return hip_status("diagnostics_kernel");
}

}  // namespace tri
