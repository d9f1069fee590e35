// GMM estimator: a K-component diagonal Gaussian mixture per modality in
// place of the single Gaussian of Sec. 3.2.2 (the supplementary GMM ablation,
// K in {2, 4}). The state per modality m and component c is (N, S_mu, S_sigma2)
// as in Eq. 5-7; pi_mc = N_mc / sum_c N_mc.
//
//  gmm_prep: state -> per (m, c, column) mu and 1 / sigma^2 (fp64 division,
//     stored fp32) and per column block the fp64 parts of sum_d log sigma^2.
//  gmm_loglik: per token and (m, c), q = sum_d (x - mu)^2 / sigma^2 (fp32 per
//     8-column stripe, accumulated in fp64, reduced by a fixed butterfly), the
//     component log-likelihood log pi - (sum log sigma^2 + q) / 2, then either
//     the score (Eq. 9 over the per-modality log-sum-exp) or the
//     responsibilities of the token's own modality (the E-step).
//  update (stepwise EM): gmm_partial sums r (x - shift), r (x - shift)^2 and r
//     per chunk of 64 tokens in fp64 (shift = the component's previous mean,
//     rounded to float32: any constant near the mean will do), gmm_merge adds
//     the chunks in a fixed order, applies Eq. 5-7 with the weighted batch
//     count, mean and centred sum of squares, and writes the score's
//     coefficients of the new state, as gmm_prep does for the old one.
// At 8192 x 2048 bf16 and K = 2 (33.6 MB) an update and a score take 4 + 15 + 18
// + 10 + 17 us, bound by latency and by the address unit (the coefficients come
// through L1 once per wave, so a wave takes four tokens, from 4096 tokens on).
// Before, 5 + 27 + 42 + 21 + 5 + 25: gmm_partial read every row's label before it loaded the row, once
// per modality, and its LDS tree had all lanes on one bank; gmm_merge walked
// 128 chunks with 8 loads in flight; gmm_loglik kept one 512-column stripe of
// two rows in flight and ran its float64 logarithms once per wave.
#include "common.h"
#include "kernels.h"

namespace smoes {

namespace {

constexpr int kGChunk = 64;         // tokens per gmm_partial block
constexpr int kGPrepThreads = 256;  // columns per gmm_prep block
constexpr int kGMergeCols = 64;     // columns per gmm_merge block
constexpr int kGMergeGroups = 8;    // chunk groups per column
constexpr int kGMaxParts = 256;     // SMOES_D_MAX / kGMergeCols: parts of a log-variance sum
// tokens per gmm_loglik wave: 4, or 1 where those would not give every CU a
// block: a wave's chain of columns is then shorter. EM step and score with K = 2, four /
// one per wave in us: 64 tokens x 2048 37.7 / 31.8, 3072 48.4 / 45.1, 4095 50.6 / 51.0,
// 6000 57.5 / 64.3; x 4096: 2048 tokens 58.0 / 49.7, 3072 61.5 / 62.7, 6000 81.0 / 104.9
constexpr int kGTokPerWave = 4;
constexpr int64_t kGTokFill = 256 * 4 * kGTokPerWave;
constexpr int kGThreads = 256;
// columns per lane of gmm_partial: 4, or 2 where the sums of 3 or 4 components would not leave four waves a SIMD
constexpr int gmm_part_cols(int K) { return K <= 2 ? 4 : 2; }

struct GmmWs {
    float* coef;      // [2K][2][d]: mu, 1 / sigma^2
    double* cst;      // [2K][kGMaxParts]: per block of 256 (gmm_prep) or 64 (gmm_merge) columns, sum log sigma^2
    double* n_old;    // [2K]
    float* resp;      // [T][K] (when the caller passes none)
    double* wsum;     // [nchunk][2K]
    double* s1;       // [nchunk][2K][d]
    double* s2;       // [nchunk][2K][d]
};

GmmWs gmm_carve(void* ws, int64_t T, int d, int K) {
    char* p = static_cast<char*>(ws);
    const int64_t nchunk = ceil_div(T, kGChunk);
    GmmWs w;
    w.coef = reinterpret_cast<float*>(p);
    p += align_up(sizeof(float) * 2 * K * 2 * d, 256);
    w.cst = reinterpret_cast<double*>(p);
    p += align_up(sizeof(double) * 2 * K * kGMaxParts, 256);
    w.n_old = reinterpret_cast<double*>(p);
    p += 256;
    w.resp = reinterpret_cast<float*>(p);
    p += align_up(sizeof(float) * T * K, 256);
    w.wsum = reinterpret_cast<double*>(p);
    p += align_up(sizeof(double) * nchunk * 2 * K, 256);
    w.s1 = reinterpret_cast<double*>(p);
    p += align_up(sizeof(double) * nchunk * 2 * K * d, 256);
    w.s2 = reinterpret_cast<double*>(p);
    return w;
}

// Score coefficients of one component's column (mean 0, variance 1 without a
// count); returns log sigma^2.
__device__ __forceinline__ double gmm_coef(double n, double smu, double ssig, double var_floor, int d, int mc, int col,
                                           float* __restrict__ coef) {
    double mu = 0.0, var = 1.0;
    if (n > 0.0) {
        mu = smu / n;
        var = fmax(ssig / n, var_floor);
    }
    coef[(static_cast<int64_t>(mc) * 2) * d + col] = static_cast<float>(mu);
    coef[(static_cast<int64_t>(mc) * 2 + 1) * d + col] = static_cast<float>(1.0 / var);
    return log(var);
}

__global__ void __launch_bounds__(kGPrepThreads)
gmm_prep_kernel(int d, int K, const float* __restrict__ gn, const float* __restrict__ gsmu,
                const float* __restrict__ gssig, float var_floor, float* __restrict__ coef,
                double* __restrict__ cst) {
    __shared__ double part[kGPrepThreads];
    const int mc = blockIdx.y;  // m * K + c
    const double n = gn[mc];
    const int col = blockIdx.x * kGPrepThreads + threadIdx.x;
    double acc = 0.0;
    if (col < d)
        acc = gmm_coef(n, gsmu[static_cast<int64_t>(mc) * d + col], gssig[static_cast<int64_t>(mc) * d + col], var_floor,
                       d, mc, col, coef);
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kGPrepThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) cst[mc * kGMaxParts + blockIdx.x] = part[0];
}

// mode 0: scores M[T][2]; mode 1: responsibilities resp[T][K] of each token's own modality.
template <bool BF16, int K, int NT>
__global__ void __launch_bounds__(kGThreads)
gmm_loglik_kernel(const void* __restrict__ x, int64_t T, int d, const uint8_t* __restrict__ mid,
                  const float* __restrict__ coef, const double* __restrict__ cst, int n_part,
                  const float* __restrict__ gn, double inv_tau, int mode, float* __restrict__ M,
                  float* __restrict__ resp) {
    constexpr int MC = 2 * K;
    __shared__ double q_s[kGThreads / kWave][NT][MC];
    __shared__ double c_s[MC];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = lane_id();
    const int64_t blk0 = static_cast<int64_t>(blockIdx.x) * (kGThreads / kWave) * NT;
    const int64_t tok0 = blk0 + wave * NT;
    int64_t rows[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) rows[t] = tok0 + t < T ? tok0 + t : T - 1;
    // sum log sigma^2 - 2 log pi of each component, by the first wave; added to a token's sum over
    // the columns at the end, in the same order whatever the call's length. Loaded after the
    // columns in a short call, which would wait for these loads first, and before them in a long
    // one, whose other waves hide that.
    // lane j < MC: -2 log pi_mc, pi_mc = N_mc / sum_c N_mc (uniform when the modality has no count)
    auto log_pi = [&] {
        double lp = 0.0;
        if (lane < MC) {
            double tot = 0.0;
#pragma unroll
            for (int c = 0; c < K; ++c) tot += static_cast<double>(gn[lane / K * K + c]);
            lp = -2.0 * (tot > 0.0 ? log(static_cast<double>(gn[lane]) / tot) : -log(static_cast<double>(K)));
        }
        return lp;
    };
    auto constant = [&](int j, double lp) {
        double slv = lane == j ? lp : 0.0;
        for (int b = lane; b < n_part; b += kWave) slv += cst[j * kGMaxParts + b];
        return slv;
    };
    auto constants = [&] {
        if (wave != 0) return;
        const double lp = log_pi();
#pragma unroll
        for (int j = 0; j < MC; ++j) {
            const double v = wave_sum_u(constant(j, lp));
            if (lane == 0) c_s[j] = v;
        }
    };
    if constexpr (NT > 1) constants();
    double acc[NT][MC];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < MC; ++j) acc[t][j] = 0.0;
    // the rows' next S stripes of 512 columns (8 per lane) are loaded before any is used
    constexpr int S = BF16 ? 4 : 2;
    constexpr int Q = BF16 ? 1 : 2;
    for (int g = lane * 8; g < d; g += S * kWave * 8) {
        uint4 raw[NT][S][Q];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int c0 = g + s * kWave * 8 < d ? g + s * kWave * 8 : 0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int64_t e = rows[t] * d + c0;
                const uint4* q = BF16 ? reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(x) + e)
                                      : reinterpret_cast<const uint4*>(static_cast<const float*>(x) + e);
#pragma unroll
                for (int i = 0; i < Q; ++i) raw[t][s][i] = q[i];
            }
        }
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int c0 = g + s * kWave * 8;
        if (c0 >= d) break;
        float v[NT][8];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const uint32_t* w = reinterpret_cast<const uint32_t*>(&raw[t][s][0]);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                v[t][i] = BF16 ? __uint_as_float(i & 1 ? w[i / 2] & 0xffff0000u : w[i / 2] << 16) : __uint_as_float(w[i]);
        }
#pragma unroll
        for (int j = 0; j < MC; ++j) {
            float mu[8], iv[8];
            const float4* pm = reinterpret_cast<const float4*>(coef + (static_cast<int64_t>(j) * 2) * d + c0);
            const float4* pi = reinterpret_cast<const float4*>(coef + (static_cast<int64_t>(j) * 2 + 1) * d + c0);
            *reinterpret_cast<float4*>(&mu[0]) = pm[0];
            *reinterpret_cast<float4*>(&mu[4]) = pm[1];
            *reinterpret_cast<float4*>(&iv[0]) = pi[0];
            *reinterpret_cast<float4*>(&iv[4]) = pi[1];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float part = 0.0f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float dv = v[t][i] - mu[i];
                    part += dv * dv * iv[i];
                }
                acc[t][j] += static_cast<double>(part);
            }
        }
      }
    }
    if constexpr (NT == 1) constants();
    // lane partials -> per (token, component) sums by a fixed butterfly; then one
    // lane per token of the block turns them into its result (the float64
    // logarithms and exponentials cost a wave the same for one token as for 64)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < MC; ++j) {
            const double v = wave_sum_u(acc[t][j]);
            if (lane == 0) q_s[wave][t][j] = v;
        }
    __syncthreads();
    const int64_t j = blk0 + threadIdx.x;
    if (threadIdx.x >= (kGThreads / kWave) * NT || j >= T) return;
    double ll[MC];
#pragma unroll
    for (int c = 0; c < MC; ++c) ll[c] = -0.5 * (q_s[threadIdx.x / NT][threadIdx.x % NT][c] + c_s[c]);
    if (mode == 0) {
        double lse[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            double mx = -INFINITY;
#pragma unroll
            for (int c = 0; c < K; ++c) mx = fmax(mx, ll[m * K + c]);
            double s = 0.0;
#pragma unroll
            for (int c = 0; c < K; ++c) s += exp(ll[m * K + c] - mx);
            lse[m] = mx + log(s);
        }
        const double sgn = (lse[0] - lse[1]) * inv_tau;  // M_vision = sigmoid(sgn)
        double mv, mt;
        if (sgn >= 0.0) {
            const double e = exp(-sgn);
            mv = 1.0 / (1.0 + e);
            mt = e / (1.0 + e);
        } else {
            const double e = exp(sgn);
            mv = e / (1.0 + e);
            mt = 1.0 / (1.0 + e);
        }
        M[j * 2] = static_cast<float>(mv);
        M[j * 2 + 1] = static_cast<float>(mt);
    } else {
        const int m = mid[j] ? 1 : 0;
        double mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < K; ++c) mx = fmax(mx, ll[m * K + c]);
        double e[K], s = 0.0;
#pragma unroll
        for (int c = 0; c < K; ++c) {
            e[c] = exp(ll[m * K + c] - mx);
            s += e[c];
        }
#pragma unroll
        for (int c = 0; c < K; ++c) resp[j * K + c] = static_cast<float>(e[c] / s);
    }
}

// The constant subtracted from a component's column before it is summed: its
// previous mean, rounded to float32 (gmm_partial and gmm_merge agree on it).
__device__ __forceinline__ float gmm_shift(double smu, double n) { return n > 0.0 ? static_cast<float>(smu / n) : 0.0f; }

// Weighted sums over a chunk of tokens: 4 waves split the rows, each lane owns
// CPL columns. One modality after the other (the labels are one bit each), so
// that one modality's sums are live: the wave's rows of the modality in groups
// of eight, loaded together, then added in row order. Fixed-order tree over
// the waves, lanes adjacent.
template <bool BF16, int K>
__global__ void __launch_bounds__(256)
gmm_partial_kernel(const void* __restrict__ x, int64_t T, int d, const uint8_t* __restrict__ mid,
                   const float* __restrict__ resp, const float* __restrict__ gn, const float* __restrict__ gsmu,
                   double* __restrict__ wsum, double* __restrict__ s1g, double* __restrict__ s2g,
                   double* __restrict__ n_old) {
    constexpr int MC = 2 * K;
    constexpr int CPL = gmm_part_cols(K);
    constexpr int NV = K * CPL * 2;  // sums of one modality
    __shared__ double red[2][NV][kWave];
    __shared__ double wred[4][MC];
    __shared__ float resp_s[kGChunk][K];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = lane_id();
    const int64_t chunk = blockIdx.x;
    const int col0 = (blockIdx.y * kWave + lane) * CPL;
    const bool active = col0 < d;
    const int c0 = active ? col0 : 0;  // lanes past d read column 0 and write nothing
    if (chunk == 0 && blockIdx.y == 0 && threadIdx.x < MC) n_old[threadIdx.x] = gn[threadIdx.x];
    const int64_t r0 = chunk * kGChunk;
    const int nr = static_cast<int>(T - r0 < kGChunk ? T - r0 : kGChunk);
    static_assert(kGChunk == kWave, "one label per lane");
    const uint64_t text = __ballot(lane < nr && mid[r0 + (lane < nr ? lane : 0)] != 0);
    for (int i = threadIdx.x; i < nr * K; i += 256) resp_s[i / K][i % K] = resp[r0 * K + i];
    __syncthreads();

    constexpr int U = 8;
    constexpr int NW = BF16 ? CPL / 2 : CPL;
    const uint64_t mine = (0x1111111111111111ull << wave) & (nr == kGChunk ? ~0ull : (1ull << nr) - 1);
#pragma unroll 1
    for (int m = 0; m < 2; ++m) {
        uint64_t left = mine & (m ? text : ~text);
        float sh[K][CPL];
        double s1[K][CPL], s2[K][CPL], ws[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const double n = gn[m * K + c];
            ws[c] = 0.0;
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                sh[c][i] = gmm_shift(gsmu[static_cast<int64_t>(m * K + c) * d + c0 + i], n);
                s1[c][i] = s2[c][i] = 0.0;
            }
        }
        while (left != 0) {  // uniform
            uint32_t v[U][NW];
            int row[U];
            int n = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (left == 0) break;
                row[u] = __builtin_ctzll(left);
                left &= left - 1;
                ++n;
                const int64_t e = (r0 + row[u]) * d + c0;
                const uint32_t* q = BF16 ? reinterpret_cast<const uint32_t*>(static_cast<const uint16_t*>(x) + e)
                                         : reinterpret_cast<const uint32_t*>(static_cast<const float*>(x) + e);
                if constexpr (NW == 1) {
                    v[u][0] = q[0];
                } else if constexpr (NW == 2) {
                    const uint2 w = *reinterpret_cast<const uint2*>(q);
                    v[u][0] = w.x;
                    v[u][1] = w.y;
                } else {
                    const uint4 w = *reinterpret_cast<const uint4*>(q);
                    v[u][0] = w.x;
                    v[u][1] = w.y;
                    v[u][2] = w.z;
                    v[u][3] = w.w;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u >= n) break;
                float xv[CPL];
#pragma unroll
                for (int i = 0; i < CPL; ++i)
                    xv[i] = BF16 ? __uint_as_float(i & 1 ? v[u][i / 2] & 0xffff0000u : v[u][i / 2] << 16)
                                 : __uint_as_float(v[u][i]);
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    const double w = static_cast<double>(resp_s[row[u]][c]);
                    ws[c] += w;
#pragma unroll
                    for (int i = 0; i < CPL; ++i) {
                        const double y = static_cast<double>(xv[i]) - static_cast<double>(sh[c][i]);
                        const double wy = w * y;
                        s1[c][i] += wy;
                        s2[c][i] = fma(wy, y, s2[c][i]);
                    }
                }
            }
        }
        // (w0 + w2) + (w1 + w3)
        auto put = [&](int slot) {
#pragma unroll
            for (int c = 0; c < K; ++c)
#pragma unroll
                for (int i = 0; i < CPL; ++i) {
                    red[slot][(c * CPL + i) * 2][lane] = s1[c][i];
                    red[slot][(c * CPL + i) * 2 + 1][lane] = s2[c][i];
                }
        };
        auto add = [&](int slot) {
#pragma unroll
            for (int c = 0; c < K; ++c)
#pragma unroll
                for (int i = 0; i < CPL; ++i) {
                    s1[c][i] += red[slot][(c * CPL + i) * 2][lane];
                    s2[c][i] += red[slot][(c * CPL + i) * 2 + 1][lane];
                }
        };
        // weight sums: every lane of a wave saw the same rows; lane 0 reports
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < K; ++c) wred[wave][m * K + c] = ws[c];
        }
        if (wave >= 2) put(wave - 2);
        __syncthreads();
        if (wave < 2) add(wave);
        __syncthreads();
        if (wave == 1) put(0);
        __syncthreads();
        if (wave == 0) {
            add(0);
            if (active) {
#pragma unroll
                for (int c = 0; c < K; ++c)
#pragma unroll
                    for (int i = 0; i < CPL; ++i) {
                        const int64_t o = (chunk * MC + m * K + c) * d + col0 + i;
                        s1g[o] = s1[c][i];
                        s2g[o] = s2[c][i];
                    }
            }
        }
        __syncthreads();
    }
    if (blockIdx.y == 0 && threadIdx.x < MC)
        wsum[chunk * MC + threadIdx.x] = (wred[0][threadIdx.x] + wred[2][threadIdx.x]) +
                                         (wred[1][threadIdx.x] + wred[3][threadIdx.x]);
}

// One component (blockIdx.y) x 64 columns: eight thread groups add their share
// of the chunks in chunk order, then the groups in order.
__global__ void __launch_bounds__(kGMergeCols * kGMergeGroups)
gmm_merge_kernel(int d, int K, int64_t nchunk, const double* __restrict__ wsum,
                 const double* __restrict__ s1g, const double* __restrict__ s2g,
                 const double* __restrict__ n_old, float beta, float var_floor, float* __restrict__ gn,
                 float* __restrict__ gsmu, float* __restrict__ gssig, float* __restrict__ coef,
                 double* __restrict__ cst) {
    __shared__ double red[3][kGMergeGroups][kGMergeCols];
    const int mc = blockIdx.y;
    const int cl = threadIdx.x % kGMergeCols, grp = threadIdx.x / kGMergeCols;
    const int col = blockIdx.x * kGMergeCols + cl;
    const int cr = col < d ? col : d - 1;
    const int64_t len = ceil_div(nchunk, kGMergeGroups);
    const int64_t lo = grp * len, hi = lo + len < nchunk ? lo + len : nchunk;
    double n = 0.0, S1 = 0.0, S2 = 0.0;
    constexpr int B = 16;  // chunk loads in flight; the sums still run in chunk order
    for (int64_t c0 = lo; c0 < hi; c0 += B) {
        double vn[B], v1[B], v2[B];
#pragma unroll
        for (int q = 0; q < B; ++q) {
            const int64_t ch = c0 + q < hi ? c0 + q : c0;
            vn[q] = wsum[ch * 2 * K + mc];
            v1[q] = s1g[(ch * 2 * K + mc) * d + cr];
            v2[q] = s2g[(ch * 2 * K + mc) * d + cr];
        }
#pragma unroll
        for (int q = 0; q < B; ++q)
            if (c0 + q < hi) {
                n += vn[q];
                S1 += v1[q];
                S2 += v2[q];
            }
    }
    red[0][grp][cl] = n;
    red[1][grp][cl] = S1;
    red[2][grp][cl] = S2;
    __syncthreads();
    if (grp != 0) return;  // whole waves
    n = S1 = S2 = 0.0;
#pragma unroll
    for (int g = 0; g < kGMergeGroups; ++g) {
        n += red[0][g][cl];
        S1 += red[1][g][cl];
        S2 += red[2][g][cl];
    }
    const double nprev = n_old[mc];
    const int64_t o = static_cast<int64_t>(mc) * d + cr;
    const double smu_old = gsmu[o];
    const double ssig_old = gssig[o];
    const double shift = gmm_shift(smu_old, nprev);
    const double b = static_cast<double>(beta);
    double mean_T = 0.0, m2_T = 0.0, cross = 0.0;
    if (n > 0.0) {
        mean_T = shift + S1 / n;
        m2_T = S2 - S1 * (S1 / n);
        if (m2_T < 0.0) m2_T = 0.0;
        if (nprev > 0.0) {
            const double dm = mean_T - smu_old / nprev;
            cross = dm * dm * (b * nprev * n) / (b * nprev + n);
        }
    }
    const float n_new = static_cast<float>(b * nprev + n);
    const float smu_new = static_cast<float>(b * smu_old + n * mean_T);
    const float ssig_new = static_cast<float>(b * ssig_old + m2_T + cross);
    double acc = 0.0;
    if (col < d) {
        gsmu[o] = smu_new;
        gssig[o] = ssig_new;
        if (col == 0) gn[mc] = n_new;
        acc = gmm_coef(n_new, smu_new, ssig_new, var_floor, d, mc, col, coef);
    }
    acc = wave_sum_u(acc);
    if (cl == 0) cst[mc * kGMaxParts + blockIdx.x] = acc;
}

template <bool BF16, int K>
hipError_t gmm_run(const void* x, int64_t T, int d, const uint8_t* mid, float* gn, float* gsmu, float* gssig,
                   int update, float beta, float tau, float var_floor, float* M, float* resp_out, const GmmWs& w,
                   hipStream_t stream) {
    hipError_t err;
    int n_part = static_cast<int>(ceil_div(d, kGPrepThreads));
    const dim3 pgrid(static_cast<unsigned>(n_part), 2 * K);
    const int nt = T >= kGTokFill ? kGTokPerWave : 1;
    const auto loglik = nt == 1 ? gmm_loglik_kernel<BF16, K, 1> : gmm_loglik_kernel<BF16, K, kGTokPerWave>;
    const dim3 lgrid(static_cast<unsigned>(ceil_div(T, kGThreads / kWave * nt)));
    const double t = tau > 0.0f ? static_cast<double>(tau) : 0.5 * d;
    float* resp = resp_out != nullptr ? resp_out : w.resp;
    if (update || resp_out != nullptr) {
        hipLaunchKernelGGL(gmm_prep_kernel, pgrid, dim3(kGPrepThreads), 0, stream, d, K, gn, gsmu, gssig,
                           var_floor, w.coef, w.cst);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        hipLaunchKernelGGL(loglik, lgrid, dim3(kGThreads), 0, stream, x, T, d, mid, w.coef,
                           w.cst, n_part, gn, 1.0 / t, 1, M, resp);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (update) {
        const int64_t nchunk = ceil_div(T, kGChunk);
        const dim3 grid(static_cast<unsigned>(nchunk), static_cast<unsigned>(ceil_div(d, kWave * gmm_part_cols(K))));
        hipLaunchKernelGGL((gmm_partial_kernel<BF16, K>), grid, dim3(256), 0, stream, x, T, d, mid, resp, gn, gsmu,
                           w.wsum, w.s1, w.s2, w.n_old);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        hipLaunchKernelGGL(gmm_merge_kernel, dim3(static_cast<unsigned>(ceil_div(d, kGMergeCols)), 2 * K),
                           dim3(kGMergeCols * kGMergeGroups), 0, stream, d, K, nchunk, w.wsum, w.s1, w.s2, w.n_old,
                           beta, var_floor, gn, gsmu, gssig, w.coef, w.cst);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        n_part = static_cast<int>(ceil_div(d, kGMergeCols));
    } else if (resp_out == nullptr) {  // else the E-step's coefficients are the score's
        hipLaunchKernelGGL(gmm_prep_kernel, pgrid, dim3(kGPrepThreads), 0, stream, d, K, gn, gsmu, gssig, var_floor,
                           w.coef, w.cst);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    hipLaunchKernelGGL(loglik, lgrid, dim3(kGThreads), 0, stream, x, T, d, mid, w.coef, w.cst,
                       n_part, gn, 1.0 / t, 0, M, resp);
    return hipGetLastError();
}

template <bool BF16>
hipError_t gmm_dispatch(int K, const void* x, int64_t T, int d, const uint8_t* mid, float* gn, float* gsmu,
                        float* gssig, int update, float beta, float tau, float var_floor, float* M, float* resp,
                        const GmmWs& w, hipStream_t s) {
    switch (K) {
        case 1: return gmm_run<BF16, 1>(x, T, d, mid, gn, gsmu, gssig, update, beta, tau, var_floor, M, resp, w, s);
        case 2: return gmm_run<BF16, 2>(x, T, d, mid, gn, gsmu, gssig, update, beta, tau, var_floor, M, resp, w, s);
        case 3: return gmm_run<BF16, 3>(x, T, d, mid, gn, gsmu, gssig, update, beta, tau, var_floor, M, resp, w, s);
        default: return gmm_run<BF16, 4>(x, T, d, mid, gn, gsmu, gssig, update, beta, tau, var_floor, M, resp, w, s);
    }
}

}  // namespace

size_t gmm_workspace_bytes(int64_t T, int d, int K) {
    const int64_t nchunk = ceil_div(T, kGChunk);
    return align_up(sizeof(float) * 2 * K * 2 * d, 256) + align_up(sizeof(double) * 2 * K * kGMaxParts, 256) + 256 +
           align_up(sizeof(float) * T * K, 256) + align_up(sizeof(double) * nchunk * 2 * K, 256) +
           2 * align_up(sizeof(double) * nchunk * 2 * K * d, 256);
}

hipError_t launch_gmm(const void* x, int x_dtype, int64_t T, int d, int K, const uint8_t* modality_id, float* gmm_n,
                      float* gmm_smu, float* gmm_ssig, int update, float beta, float tau, float var_floor, float* M,
                      float* resp, void* ws, hipStream_t stream) {
    const GmmWs w = gmm_carve(ws, T, d, K);
    if (x_dtype == 1)
        return gmm_dispatch<true>(K, x, T, d, modality_id, gmm_n, gmm_smu, gmm_ssig, update, beta, tau, var_floor, M,
                                  resp, w, stream);
    return gmm_dispatch<false>(K, x, T, d, modality_id, gmm_n, gmm_smu, gmm_ssig, update, beta, tau, var_floor, M,
                               resp, w, stream);
}

}  // namespace smoes
