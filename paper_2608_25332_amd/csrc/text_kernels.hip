// Critical text tokens (Sec. 4.2, equations for r and T).
//
//   r[j] = (1/Nt) sum_i softmax_j(e_i . e_j)      (E E^T without scaling)
//   T    = { j : r[j] > mean(r) }, every token when that is empty
//
// The self-similarity E E^T is formed on the upper triangle of its tiles and
// written in full (text_gram split over k, or the streaming form, in
// dedup_kernels.hip).  text_rows takes each row's maximum and normaliser; since
// G is its own transpose, r[j] then needs row j of G only, so every later step
// is spread over rows too: text_cols (a wave per token) and text_mark, or both
// in text_rank, one workgroup per sample, for up to kRankFuse tokens.
#include "provip.h"
#include "pv_launch.h"
#include "pv_device.h"

#include <math.h>

namespace pv {

constexpr int kRankNT = 1024;
constexpr int kRankW = kRankNT / 64;  // waves
constexpr int kRankFuse = 256;        // tokens up to which one workgroup ranks a sample
constexpr int kTextU = 4;             // rows, or k slices, loaded together

// Sum of one value per thread over the workgroup, in a fixed order: the
// wave's lanes in the order of a butterfly, then the waves in index order.
__device__ __forceinline__ float block_sum_fixed(float v, float *wsum) {
    v = wave_sum64(v);
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wsum[wave] = v;
    __syncthreads();
    float t = 0.f;
    for (int w = 0; w < kRankW; ++w) t += wsum[w];
    return t;
}

// text_rows: grid (ceil(Nt / 4), B), a wave per row i: G[b][i] = the k slices
// added in slice order (KS == 0: G is complete already), and the row's
// (maximum, 1 / sum of exponentials) -> stats[b][i].  PER * 64 >= Nt.
template <int PER>
__global__ __launch_bounds__(256) void text_rows_kernel(const float *__restrict__ part, int B,
                                                        int Nt, int KS, float *__restrict__ G,
                                                        float2 *__restrict__ stats) {
    const int lane = threadIdx.x & 63, b = blockIdx.y;
    const int i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (i >= Nt) return;
    float *row = G + ((size_t)b * Nt + i) * Nt;
    float g[PER];
    if (KS == 0) {
#pragma unroll
        for (int t = 0; t < PER; ++t) g[t] = row[min(lane + 64 * t, Nt - 1)];
    } else {
        const size_t ks_stride = (size_t)B * Nt * Nt;
        const float *prow = part + ((size_t)b * Nt + i) * Nt;
#pragma unroll
        for (int t = 0; t < PER; ++t) g[t] = 0.f;
        for (int k0 = 0; k0 < KS; k0 += kTextU) {
            float v[kTextU][PER];
#pragma unroll
            for (int u = 0; u < kTextU; ++u)
#pragma unroll
                for (int t = 0; t < PER; ++t)
                    v[u][t] = prow[(size_t)min(k0 + u, KS - 1) * ks_stride + min(lane + 64 * t, Nt - 1)];
#pragma unroll
            for (int u = 0; u < kTextU; ++u)
                if (k0 + u < KS) {
#pragma unroll
                    for (int t = 0; t < PER; ++t) g[t] += v[u][t];
                }
        }
#pragma unroll
        for (int t = 0; t < PER; ++t)
            if (lane + 64 * t < Nt) row[lane + 64 * t] = g[t];
    }
    float m = -INFINITY;
#pragma unroll
    for (int t = 0; t < PER; ++t) m = fmaxf(m, g[t]);  // past the end: the last element again
    m = wave_max_f32(m);
    float l = 0.f;
#pragma unroll
    for (int t = 0; t < PER; ++t)
        if (lane + 64 * t < Nt) l += expf(g[t] - m);
    l = wave_sum64(l);
    if (lane == 0) stats[(size_t)b * Nt + i] = make_float2(m, 1.0f / l);
}

// r[j] = (1/Nt) sum_i exp(G[j][i] - m_i) / l_i of a wave's row j (in g), the
// statistics of the rows in st.
template <int PER>
__device__ __forceinline__ float text_col(const float (&g)[PER], const float2 *st, int Nt, int lane) {
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int i = lane + 64 * t;
        const float2 q = st[min(i, Nt - 1)];
        if (i < Nt) s += expf(g[t] - q.x) * q.y;
    }
    return wave_sum64(s) / (float)Nt;
}

// text_cols: grid (ceil(Nt / 4), B), a wave per token j: r[b][j].
template <int PER>
__global__ __launch_bounds__(256) void text_cols_kernel(const float *__restrict__ G,
                                                        const float2 *__restrict__ stats, int Nt,
                                                        float *__restrict__ r) {
    const int lane = threadIdx.x & 63, b = blockIdx.y;
    const int j = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (j >= Nt) return;
    float g[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t) g[t] = G[((size_t)b * Nt + j) * Nt + min(lane + 64 * t, Nt - 1)];
    const float v = text_col<PER>(g, stats + (size_t)b * Nt, Nt, lane);
    if (lane == 0) r[(size_t)b * Nt + j] = v;
}

// One workgroup of kRankNT threads: mean of r over the tokens, the mask of
// those strictly above it (every token when there is none) and their count.
__device__ __forceinline__ void text_mark(const float *rr, int b, int Nt, float *wsum,
                                          int32_t *__restrict__ mask, int32_t *__restrict__ count) {
    const int tid = threadIdx.x;
    float own = 0.f;
    for (int j = tid; j < Nt; j += kRankNT) own += rr[j];
    const float mean = block_sum_fixed(own, wsum) / (float)Nt;
    int above = 0;
    for (int j = tid; j < Nt; j += kRankNT) above += rr[j] > mean ? 1 : 0;
    const int n_above = (int)block_sum_fixed((float)above, wsum);
    // none strictly above the mean: every token is kept
    for (int j = tid; j < Nt; j += kRankNT)
        mask[(size_t)b * Nt + j] = (n_above == 0 || rr[j] > mean) ? 1 : 0;
    if (tid == 0) count[b] = n_above == 0 ? Nt : n_above;
}

__global__ __launch_bounds__(kRankNT) void text_mark_kernel(const float *__restrict__ r, int Nt,
                                                            int32_t *__restrict__ mask,
                                                            int32_t *__restrict__ count) {
    __shared__ float wsum[kRankW];
    text_mark(r + (size_t)blockIdx.x * Nt, blockIdx.x, Nt, wsum, mask, count);
}

// text_rank: text_cols and text_mark of one sample in one workgroup (two
// launches' work: 4 + 3 us as launches of their own, 5 us here at 64 tokens).
// Wave w takes tokens w, w + kRankW, ..., the rows of kTextU loaded together.
template <int PER>
__global__ __launch_bounds__(kRankNT) void text_rank_kernel(const float *__restrict__ G,
                                                            const float2 *__restrict__ stats, int Nt,
                                                            float *__restrict__ r_out,
                                                            int32_t *__restrict__ mask,
                                                            int32_t *__restrict__ count) {
    __shared__ float2 st[kRankFuse];
    __shared__ float rr[kRankFuse];
    __shared__ float wsum[kRankW];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *Gb = G + (size_t)b * Nt * Nt;
    if (tid < Nt) st[tid] = stats[(size_t)b * Nt + tid];
    __syncthreads();
    for (int j0 = wave; j0 < Nt; j0 += kTextU * kRankW) {
        float g[kTextU][PER];
#pragma unroll
        for (int u = 0; u < kTextU; ++u)
#pragma unroll
            for (int t = 0; t < PER; ++t)
                g[u][t] = Gb[(size_t)min(j0 + u * kRankW, Nt - 1) * Nt + min(lane + 64 * t, Nt - 1)];
#pragma unroll
        for (int u = 0; u < kTextU; ++u) {
            const int j = j0 + u * kRankW;
            if (j >= Nt) break;  // uniform over the wave
            const float v = text_col<PER>(g[u], st, Nt, lane);
            if (lane == 0) {
                rr[j] = v;
                if (r_out) r_out[(size_t)b * Nt + j] = v;
            }
        }
    }
    __syncthreads();
    text_mark(rr, b, Nt, wsum, mask, count);
}

#define PV_PER_CASES(call)                \
    if (Nt <= 64) call(1);                \
    else if (Nt <= 128) call(2);          \
    else if (Nt <= 256) call(4);          \
    else if (Nt <= 512) call(8);          \
    else call(PV_MAX_TEXT / 64);

hipError_t launch_text_rows(const float *part, int B, int Nt, int KS, float *G, float *stats,
                            hipStream_t st) {
    if (Nt > PV_MAX_TEXT) return hipErrorInvalidValue;
#define PV_ROWS_CASE(per)                                                                     \
    hipLaunchKernelGGL(text_rows_kernel<per>, dim3((Nt + 3) / 4, B), dim3(256), 0, st, part, B, \
                       Nt, KS, G, reinterpret_cast<float2 *>(stats))
    PV_PER_CASES(PV_ROWS_CASE)
#undef PV_ROWS_CASE
    return hipGetLastError();
}

bool text_rank_fused(int Nt) { return Nt <= kRankFuse; }

hipError_t launch_text_rank(const float *G, const float *stats, int B, int Nt, float *r,
                            int32_t *mask, int32_t *count, hipStream_t st) {
    if (!text_rank_fused(Nt)) return hipErrorInvalidValue;
    const float2 *s2 = reinterpret_cast<const float2 *>(stats);
#define PV_RANK_CASE(per)                                                                          \
    hipLaunchKernelGGL(text_rank_kernel<per>, dim3(B), dim3(kRankNT), 0, st, G, s2, Nt, r, mask, \
                       count)
    if (Nt <= 64) PV_RANK_CASE(1);
    else if (Nt <= 128) PV_RANK_CASE(2);
    else PV_RANK_CASE(kRankFuse / 64);
#undef PV_RANK_CASE
    return hipGetLastError();
}

hipError_t launch_text_cols(const float *G, const float *stats, int B, int Nt, float *r,
                            hipStream_t st) {
    if (Nt > PV_MAX_TEXT) return hipErrorInvalidValue;
#define PV_COLS_CASE(per)                                                                     \
    hipLaunchKernelGGL(text_cols_kernel<per>, dim3((Nt + 3) / 4, B), dim3(256), 0, st, G,     \
                       reinterpret_cast<const float2 *>(stats), Nt, r)
    PV_PER_CASES(PV_COLS_CASE)
#undef PV_COLS_CASE
    return hipGetLastError();
}

hipError_t launch_text_mark(const float *r, int B, int Nt, int32_t *mask, int32_t *count,
                            hipStream_t st) {
    hipLaunchKernelGGL(text_mark_kernel, dim3(B), dim3(kRankNT), 0, st, r, Nt, mask, count);
    return hipGetLastError();
}
#undef PV_PER_CASES

}  // namespace pv
