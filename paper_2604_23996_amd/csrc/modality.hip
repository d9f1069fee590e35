// Gaussian-statistics modality score (Sec. 3.2.2).
//
//  update (optional): per-modality batch count, mean and centred sum of
//     squares, folded into the caller's EMA-Welford state (Eq. 5-7).
//     gauss_partial: 4 waves share 512 columns (8 per lane) and split a
//       64-token chunk (rows loaded eight at a time); fp64 sums of
//       (x - shift) and (x - shift)^2, where the shift is the previous mean
//       (rounded to float32: any constant near the mean will do), then a
//       fixed-order LDS tree, lanes adjacent (bank-conflict free).
//     gauss_merge: 32 columns per block; for each modality sixteen thread groups
//       add their share of the chunk partials in chunk order, then the groups
//       in order; the EMA update; and, since both modalities' new statistics
//       are at hand, the score coefficients of gauss_prep.
//     At 16384 x 2048 bf16 (67 MB) an update and a score take 22 + 8 + 16 us
//     (27 + 14 with both modalities' sums live, which left two waves a SIMD,
//     and 64 columns per merge block);
//     with an LDS tree that had all lanes on one bank, a merge of 64 one-wave
//     blocks that walked 256 chunks with 16 loads in flight, a gauss_prep of
//     its own and one stripe of the score in flight, 40 + 32 + 5 + 22 us.
//  score: gauss_prep (score without update) turns the state into per-column
//     mu_m and 1 / sigma^2_m (fp64 division, stored fp32) and the fp64 constant
//     sum_d log(s2_v / s2_t) as per-block parts;
//     modality_score evaluates, per token,
//       Delta = sum_d [log s2_v - log s2_t + (x - mu_v)^2 / s2_v - (x - mu_t)^2 / s2_t]
//     (each column's two squared terms in fp32, accumulated in fp64);
//     M_vision = sigmoid(-Delta / (2 tau)), M_text = 1 - M_vision (Eq. 8-9).
//     The two squared terms are kept apart rather than expanded around a
//     common centre: with very different variances the expansion cancels
//     terms ~1/sigma^2 times larger than the result.
#include "common.h"
#include "kernels.h"

namespace smoes {

namespace {

constexpr int kChunkRows = 64;    // tokens per gauss_partial block (16 per wave)
constexpr int kColsPerBlock = 512; // 64 lanes x 8 columns
constexpr int kScoreTokPerWave = 2;
constexpr int kScoreThreads = 256;
constexpr int kPrepThreads = 256;   // columns per gauss_prep block
constexpr int kMergeCols = 32;      // columns per gauss_merge block
constexpr int kMergeGroups = 16;    // chunk groups per column and modality
constexpr int kCstMax = 512;        // SMOES_D_MAX / kMergeCols: parts of the score constant

struct ModalityWs {
    float* coef;       // [4][d]: mu_v, 1/s2_v, mu_t, 1/s2_t
    double* cst;       // per block of 32 (gauss_merge) or 256 (gauss_prep) columns: sum (log s2_v - log s2_t)
    double* n_old;     // [2]: state counts before the update
    int32_t* counts;   // [nchunk][2]
    double* s1;        // [nchunk][2][d]
    double* s2;        // [nchunk][2][d]
};

ModalityWs carve(void* ws, int64_t T, int d) {
    char* p = static_cast<char*>(ws);
    ModalityWs w;
    const int64_t nchunk = ceil_div(T, kChunkRows);
    w.coef = reinterpret_cast<float*>(p);
    p += align_up(sizeof(float) * 4 * d, 256);
    w.cst = reinterpret_cast<double*>(p);
    p += sizeof(double) * kCstMax;
    w.n_old = reinterpret_cast<double*>(p);
    p += 256;
    w.counts = reinterpret_cast<int32_t*>(p);
    p += align_up(sizeof(int32_t) * 2 * nchunk, 256);
    w.s1 = reinterpret_cast<double*>(p);
    p += align_up(sizeof(double) * 2 * nchunk * d, 256);
    w.s2 = reinterpret_cast<double*>(p);
    return w;
}

// The constant subtracted from modality m's column before it is summed: its
// previous mean, rounded to float32 (gauss_partial and gauss_merge agree on it).
__device__ __forceinline__ float shift_of(double smu, double n) {
    return n > 0.0 ? static_cast<float>(smu / n) : 0.0f;
}

template <bool BF16>
__global__ void __launch_bounds__(256)
gauss_partial_kernel(const void* __restrict__ x, int64_t T, int d, const uint8_t* __restrict__ mid,
                     const float* __restrict__ gauss_n, const float* __restrict__ gauss_smu,
                     int32_t* __restrict__ counts, double* __restrict__ s1g, double* __restrict__ s2g,
                     double* __restrict__ n_old) {
    __shared__ double red[2][16][kWave];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = lane_id();
    const int64_t chunk = blockIdx.x;
    const int col0 = blockIdx.y * kColsPerBlock + lane * 8;
    const bool active = col0 < d;
    const int c0 = active ? col0 : 0;  // lanes past d read column 0 and write nothing
    if (chunk == 0 && blockIdx.y == 0 && threadIdx.x < 2) n_old[threadIdx.x] = gauss_n[threadIdx.x];
    const int64_t r0 = chunk * kChunkRows;
    const int nr = static_cast<int>(T - r0 < kChunkRows ? T - r0 : kChunkRows);
    // labels of the chunk's rows as one bit each
    static_assert(kChunkRows == kWave, "one label per lane");
    const uint64_t text = __ballot(lane < nr && mid[r0 + (lane < nr ? lane : 0)] != 0);

    // One modality after the other, so that one set of sums is live: this wave's
    // rows (wave, wave + 4, ...) of the modality in groups of U, whose loads go
    // out together and are then added in row order.
    constexpr int U = 8;
    constexpr int Q = BF16 ? 1 : 2;
    const uint64_t mine = (0x1111111111111111ull << wave) & (nr == kChunkRows ? ~0ull : (1ull << nr) - 1);
    const double n_prev[2] = {gauss_n[0], gauss_n[1]};
#pragma unroll 1
    for (int m = 0; m < 2; ++m) {
        uint64_t left = mine & (m ? text : ~text);
        float sh[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) sh[i] = shift_of(gauss_smu[static_cast<int64_t>(m) * d + c0 + i], n_prev[m]);
        double s1[8], s2[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s1[i] = s2[i] = 0.0;
        while (left != 0) {  // uniform
            uint4 v[U][Q];
            int n = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (left == 0) break;
                const int r = __builtin_ctzll(left);
                left &= left - 1;
                ++n;
                const int64_t e = (r0 + r) * d + c0;
                const uint4* q = BF16 ? reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(x) + e)
                                      : reinterpret_cast<const uint4*>(static_cast<const float*>(x) + e);
#pragma unroll
                for (int i = 0; i < Q; ++i) v[u][i] = q[i];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u >= n) break;
                const uint32_t* w = reinterpret_cast<const uint32_t*>(&v[u][0]);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float xv = BF16 ? __uint_as_float(i & 1 ? w[i / 2] & 0xffff0000u : w[i / 2] << 16)
                                          : __uint_as_float(w[i]);
                    const double y = static_cast<double>(xv) - static_cast<double>(sh[i]);
                    s1[i] += y;
                    s2[i] = fma(y, y, s2[i]);
                }
            }
        }
        // fixed-order tree over the waves: (w0 + w2) + (w1 + w3)
        auto put = [&](int slot) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                red[slot][i][lane] = s1[i];
                red[slot][8 + i][lane] = s2[i];
            }
        };
        auto add = [&](int slot) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                s1[i] += red[slot][i][lane];
                s2[i] += red[slot][8 + i][lane];
            }
        };
        if (wave >= 2) put(wave - 2);
        __syncthreads();
        if (wave < 2) add(wave);
        __syncthreads();
        if (wave == 1) put(0);
        __syncthreads();
        if (wave == 0) {
            add(0);
            if (active) {
                const int64_t o = (chunk * 2 + m) * d + col0;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    s1g[o + i] = s1[i];
                    s2g[o + i] = s2[i];
                }
            }
        }
        __syncthreads();
    }
    if (blockIdx.y == 0 && threadIdx.x == 0) {
        const int nt = __popcll(text);
        counts[chunk * 2] = nr - nt;
        counts[chunk * 2 + 1] = nt;
    }
}

// One modality's column of the score: mean and floored variance of a state
// (mean 0, variance 1 without a count).
__device__ __forceinline__ void mean_var(double n, double smu, double ssig, double var_floor, double& mu, double& var) {
    mu = 0.0;
    var = 1.0;
    if (n > 0.0) {
        mu = smu / n;
        var = fmax(ssig / n, var_floor);
    }
}

__global__ void __launch_bounds__(kMergeCols * 2 * kMergeGroups)
gauss_merge_kernel(int d, int64_t nchunk, const int32_t* __restrict__ counts,
                   const double* __restrict__ s1g, const double* __restrict__ s2g,
                   const double* __restrict__ n_old, float beta, float var_floor,
                   float* __restrict__ gauss_n, float* __restrict__ gauss_smu,
                   float* __restrict__ gauss_ssig, float* __restrict__ coef, double* __restrict__ cst_part) {
    __shared__ double red[2][kMergeGroups][2][kMergeCols];
    __shared__ int32_t nred[kMergeGroups][2];
    __shared__ double mv[2][2][kMergeCols];
    const int cl = threadIdx.x % kMergeCols, m = (threadIdx.x / kMergeCols) & 1, grp = threadIdx.x / (2 * kMergeCols);
    const int col = blockIdx.x * kMergeCols + cl;
    const int cr = col < d ? col : d - 1;
    const int64_t len = ceil_div(nchunk, kMergeGroups);
    const int64_t lo = grp * len, hi = lo + len < nchunk ? lo + len : nchunk;
    int32_t n = 0;
    double S1 = 0.0, S2 = 0.0;
    constexpr int B = 16;  // chunk loads in flight; the sums still run in chunk order
    for (int64_t c0 = lo; c0 < hi; c0 += B) {
        int32_t vn[B];
        double v1[B], v2[B];
#pragma unroll
        for (int q = 0; q < B; ++q) {
            const int64_t c = c0 + q < hi ? c0 + q : c0;
            vn[q] = counts[c * 2 + m];
            v1[q] = s1g[(c * 2 + m) * d + cr];
            v2[q] = s2g[(c * 2 + m) * d + cr];
        }
#pragma unroll
        for (int q = 0; q < B; ++q)
            if (c0 + q < hi) {
                n += vn[q];
                S1 += v1[q];
                S2 += v2[q];
            }
    }
    red[0][grp][m][cl] = S1;
    red[1][grp][m][cl] = S2;
    if (cl == 0) nred[grp][m] = n;
    __syncthreads();
    if (grp == 0) {
        int64_t nn = 0;
        S1 = S2 = 0.0;
#pragma unroll
        for (int g = 0; g < kMergeGroups; ++g) {
            nn += nred[g][m];
            S1 += red[0][g][m][cl];
            S2 += red[1][g][m][cl];
        }
        const double nprev = n_old[m];
        const double smu_old = gauss_smu[static_cast<int64_t>(m) * d + cr];
        const double ssig_old = gauss_ssig[static_cast<int64_t>(m) * d + cr];
        const double shift = shift_of(smu_old, nprev);
        const double b = static_cast<double>(beta);
        const double nt = static_cast<double>(nn);
        double mean_T = 0.0, m2_T = 0.0, cross = 0.0;
        if (nn > 0) {
            mean_T = shift + S1 / nt;
            m2_T = S2 - S1 * (S1 / nt);
            if (m2_T < 0.0) m2_T = 0.0;
            if (nprev > 0.0) {
                const double dm = mean_T - smu_old / nprev;
                cross = dm * dm * (b * nprev * nt) / (b * nprev + nt);
            }
        }
        const float n_new = static_cast<float>(b * nprev + nt);
        const float smu_new = static_cast<float>(b * smu_old + nt * mean_T);
        const float ssig_new = static_cast<float>(b * ssig_old + m2_T + cross);
        if (col < d) {
            gauss_smu[static_cast<int64_t>(m) * d + col] = smu_new;
            gauss_ssig[static_cast<int64_t>(m) * d + col] = ssig_new;
            if (col == 0) gauss_n[m] = n_new;
        }
        mean_var(n_new, smu_new, ssig_new, var_floor, mv[0][m][cl], mv[1][m][cl]);
    }
    __syncthreads();
    static_assert(kMergeCols <= kWave, "one wave writes the coefficients");
    if (threadIdx.x < kWave) {  // the coefficients, and their constant's part
        double acc = 0.0;
        if (threadIdx.x < kMergeCols && col < d) {
            coef[col] = static_cast<float>(mv[0][0][cl]);
            coef[d + col] = static_cast<float>(1.0 / mv[1][0][cl]);
            coef[2 * d + col] = static_cast<float>(mv[0][1][cl]);
            coef[3 * d + col] = static_cast<float>(1.0 / mv[1][1][cl]);
            acc = log(mv[1][0][cl]) - log(mv[1][1][cl]);
        }
        acc = wave_sum_u(acc);
        if (threadIdx.x == 0) cst_part[blockIdx.x] = acc;
    }
}

// Per-column score coefficients; each block of 256 columns also writes its
// part of the fp64 constant (a fixed-order LDS tree), summed by modality_score.
__global__ void __launch_bounds__(kPrepThreads)
gauss_prep_kernel(int d, const float* __restrict__ gauss_n, const float* __restrict__ gauss_smu,
                  const float* __restrict__ gauss_ssig, float var_floor, float* __restrict__ coef,
                  double* __restrict__ cst_part) {
    __shared__ double part[kPrepThreads];
    const double nv = gauss_n[0], nt = gauss_n[1];
    const int c = blockIdx.x * kPrepThreads + threadIdx.x;
    double acc = 0.0;
    if (c < d) {
        double mv, vv, mt, vt;
        mean_var(nv, gauss_smu[c], gauss_ssig[c], var_floor, mv, vv);
        mean_var(nt, gauss_smu[d + c], gauss_ssig[d + c], var_floor, mt, vt);
        coef[c] = static_cast<float>(mv);
        coef[d + c] = static_cast<float>(1.0 / vv);
        coef[2 * d + c] = static_cast<float>(mt);
        coef[3 * d + c] = static_cast<float>(1.0 / vt);
        acc = log(vv) - log(vt);
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kPrepThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) cst_part[blockIdx.x] = part[0];
}

// Two tokens per wave. The stripes of 512 columns (8 per lane) run four at a
// time: the loads of a token's next four stripes go out together before any of
// them is used (a loop that left after each stripe kept one stripe in flight:
// 22 against 16 us at 16384 x 2048 bf16).
template <bool BF16>
__global__ void __launch_bounds__(kScoreThreads)
modality_score_kernel(const void* __restrict__ x, int64_t T, int d, const float* __restrict__ coef,
                      const double* __restrict__ cst_part, int n_part, double inv2tau, float* __restrict__ M) {
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int64_t tok0 = (static_cast<int64_t>(blockIdx.x) * (kScoreThreads / kWave) + wave) * kScoreTokPerWave;
    if (tok0 >= T) return;  // whole waves only: the reduction below is wave-local
    constexpr int S = 4;        // stripes in flight
    constexpr int Q = BF16 ? 1 : 2;
    int64_t rows[kScoreTokPerWave];
#pragma unroll
    for (int t = 0; t < kScoreTokPerWave; ++t) rows[t] = (tok0 + t < T ? tok0 + t : T - 1) * d;
    double cst = 0.0;
    for (int b = lane; b < n_part; b += kWave) cst += cst_part[b];
    double acc[kScoreTokPerWave];
#pragma unroll
    for (int t = 0; t < kScoreTokPerWave; ++t) acc[t] = cst;
    for (int g = lane * 8; g < d; g += S * kWave * 8) {
        uint4 v[kScoreTokPerWave][S][Q];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int c0 = g + s * kWave * 8 < d ? g + s * kWave * 8 : 0;
#pragma unroll
            for (int t = 0; t < kScoreTokPerWave; ++t) {
                const uint4* q = BF16 ? reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(x) + rows[t] + c0)
                                      : reinterpret_cast<const uint4*>(static_cast<const float*>(x) + rows[t] + c0);
#pragma unroll
                for (int i = 0; i < Q; ++i) v[t][s][i] = q[i];
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int c0 = g + s * kWave * 8;
            if (c0 >= d) break;
            float mv[8], iv[8], mt[8], it[8];
            const float4* p0 = reinterpret_cast<const float4*>(coef + c0);
            const float4* p1 = reinterpret_cast<const float4*>(coef + d + c0);
            const float4* p2 = reinterpret_cast<const float4*>(coef + 2 * d + c0);
            const float4* p3 = reinterpret_cast<const float4*>(coef + 3 * d + c0);
            *reinterpret_cast<float4*>(&mv[0]) = p0[0];
            *reinterpret_cast<float4*>(&mv[4]) = p0[1];
            *reinterpret_cast<float4*>(&iv[0]) = p1[0];
            *reinterpret_cast<float4*>(&iv[4]) = p1[1];
            *reinterpret_cast<float4*>(&mt[0]) = p2[0];
            *reinterpret_cast<float4*>(&mt[4]) = p2[1];
            *reinterpret_cast<float4*>(&it[0]) = p3[0];
            *reinterpret_cast<float4*>(&it[4]) = p3[1];
#pragma unroll
            for (int t = 0; t < kScoreTokPerWave; ++t) {
                const uint32_t* w = reinterpret_cast<const uint32_t*>(&v[t][s][0]);
                float part = 0.0f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float xv = BF16 ? __uint_as_float(i & 1 ? w[i / 2] & 0xffff0000u : w[i / 2] << 16)
                                          : __uint_as_float(w[i]);
                    const float dv = xv - mv[i];
                    const float dt = xv - mt[i];
                    part += dv * dv * iv[i] - dt * dt * it[i];
                }
                acc[t] += static_cast<double>(part);
            }
        }
    }
    // per token: the lane partials (with the constant's parts) by a fixed butterfly
#pragma unroll
    for (int t = 0; t < kScoreTokPerWave; ++t) acc[t] = wave_sum_u(acc[t]);
    if (lane < kScoreTokPerWave) {
        static_assert(kScoreTokPerWave == 2, "the token select below assumes two tokens per wave");
        const int t = lane;
        const double delta = t == 0 ? acc[0] : acc[1];
        if (tok0 + t < T) {
            const double s = -delta * inv2tau;
            double mv, mt;
            if (s >= 0.0) {
                const double e = exp(-s);
                mv = 1.0 / (1.0 + e);
                mt = e / (1.0 + e);
            } else {
                const double e = exp(s);
                mv = e / (1.0 + e);
                mt = 1.0 / (1.0 + e);
            }
            M[(tok0 + t) * 2] = static_cast<float>(mv);
            M[(tok0 + t) * 2 + 1] = static_cast<float>(mt);
        }
    }
}

}  // namespace

size_t modality_workspace_bytes(int64_t T, int d) {
    const int64_t nchunk = ceil_div(T, kChunkRows);
    return align_up(sizeof(float) * 4 * d, 256) + sizeof(double) * kCstMax + 256 +
           align_up(sizeof(int32_t) * 2 * nchunk, 256) +
           2 * align_up(sizeof(double) * 2 * nchunk * d, 256);
}

hipError_t launch_modality(const void* x, int x_dtype, int64_t T, int d, const uint8_t* modality_id,
                           float* gauss_n, float* gauss_smu, float* gauss_ssig, int update,
                           float beta, float tau, float var_floor, float* M, void* ws,
                           hipStream_t stream) {
    ModalityWs w = carve(ws, T, d);
    const bool bf16 = x_dtype == 1;
    hipError_t err;
    if (update) {
        const int64_t nchunk = ceil_div(T, kChunkRows);
        const dim3 grid(static_cast<unsigned>(nchunk), static_cast<unsigned>(ceil_div(d, kColsPerBlock)));
        if (bf16)
            hipLaunchKernelGGL(gauss_partial_kernel<true>, grid, dim3(256), 0, stream, x, T, d,
                               modality_id, gauss_n, gauss_smu, w.counts, w.s1, w.s2, w.n_old);
        else
            hipLaunchKernelGGL(gauss_partial_kernel<false>, grid, dim3(256), 0, stream, x, T, d,
                               modality_id, gauss_n, gauss_smu, w.counts, w.s1, w.s2, w.n_old);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        hipLaunchKernelGGL(gauss_merge_kernel, dim3(static_cast<unsigned>(ceil_div(d, kMergeCols))),
                           dim3(kMergeCols * 2 * kMergeGroups), 0, stream, d, nchunk, w.counts, w.s1, w.s2, w.n_old,
                           beta, var_floor, gauss_n, gauss_smu, gauss_ssig, w.coef, w.cst);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    } else {
        hipLaunchKernelGGL(gauss_prep_kernel, dim3(static_cast<unsigned>(ceil_div(d, kPrepThreads))),
                           dim3(kPrepThreads), 0, stream, d, gauss_n, gauss_smu, gauss_ssig, var_floor, w.coef, w.cst);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    const int n_part = static_cast<int>(ceil_div(d, update ? kMergeCols : kPrepThreads));
    const double t = tau > 0.0f ? static_cast<double>(tau) : 0.5 * d;
    const double inv2tau = 1.0 / (2.0 * t);
    const int64_t tok_per_block = static_cast<int64_t>(kScoreThreads / kWave) * kScoreTokPerWave;
    const dim3 grid(static_cast<unsigned>(ceil_div(T, tok_per_block)));
    if (bf16)
        hipLaunchKernelGGL(modality_score_kernel<true>, grid, dim3(kScoreThreads), 0, stream, x, T,
                           d, w.coef, w.cst, n_part, inv2tau, M);
    else
        hipLaunchKernelGGL(modality_score_kernel<false>, grid, dim3(kScoreThreads), 0, stream, x,
                           T, d, w.coef, w.cst, n_part, inv2tau, M);
    return hipGetLastError();
}

}  // namespace smoes
