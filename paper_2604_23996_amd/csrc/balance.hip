// Momentum-adaptive binning (Sec. 3.3, Eq. 10-11), the bin-level load
// balance loss with its logit gradient (Sec. 3.5, Eq. 16) and the modality
// specialization index (Sec. 4.1, Eq. 18-19) of one layer, from one batch's
// routing.
//
//   bal_partial : per 64-token chunk: per token the bins its top-k reaches
//                 (kept for the gradient), counts C[m][e] of hard label m with
//                 e in the token's top-k and tokens routed to each bin
//                 (popcounts of transposed bit masks: no atomics), and per expert the gate
//                 mass over the tokens routed to its bin (fp64, fixed order).
//                 64 tokens, because the kernel is latency-bound: at 4096
//                 tokens x 64 experts 10 us, with 256 tokens (16 blocks) and a
//                 ballot per expert 32 us; bal_finalize then has four times the
//                 chunks to add (9 -> 12 us).
//   bal_finalize: one block; four thread groups sum their share of the chunk
//                 partials in chunk order, then the groups in order; then
//                 L_bal = sum_e N_B (n_e / T_k)(S_e / T_k), the gradient
//                 coefficients N_B n_e / T_k^2, the EMA of the expert loads
//                 (fp64, products rounded before the sum), f_spec, the stable
//                 ascending rank of f_spec -> next bin map, and MSI.
//   bal_grad    : one wave per token: dz = scale * g * (dg - sum_e g dg) with
//                 dg_e = coef_e for experts whose bin the token was routed to
//                 (the token's bin mask from bal_partial).
// Readings (the paper leaves them open): "tokens in bin B_k" are the tokens
// routed to bin k; f_e = n_e / T_k, P_e = mean gate of e over them; the top-k
// counts are constants for the gradient; f_spec = 1/2 for an expert with no
// load; MSI counts an expert no token reaches as unspecialised.
#include "common.h"
#include "kernels.h"

namespace smoes {

namespace {

constexpr int kBalChunk = 64;     // tokens per partial block: one per lane
constexpr int kBalThreads = 256;  // 4 waves
constexpr int kBalWaves = kBalThreads / kWave;
constexpr int kFinGroups = 4;     // chunk groups of bal_finalize
constexpr int kFinThreads = kFinGroups * 256;
static_assert(kBalWaves == 4, "wave w counts experts 64 w .. 64 w + 63");

struct BalWs {
    int32_t* cnt;    // [nchunk][2][E]
    int32_t* tk;     // [nchunk][n_bins]
    double* mass;    // [nchunk][E]
    double* coef;    // [E]
    uint64_t* mask;  // [T]: bins each token's top-k reaches
};

BalWs carve(void* ws, int64_t nchunk, int E, int n_bins) {
    char* p = static_cast<char*>(ws);
    BalWs w;
    w.cnt = reinterpret_cast<int32_t*>(p);
    p += align_up(sizeof(int32_t) * nchunk * 2 * E, 256);
    w.tk = reinterpret_cast<int32_t*>(p);
    p += align_up(sizeof(int32_t) * nchunk * n_bins, 256);
    w.mass = reinterpret_cast<double*>(p);
    p += align_up(sizeof(double) * nchunk * E, 256);
    w.coef = reinterpret_cast<double*>(p);
    p += align_up(sizeof(double) * E, 256);
    w.mask = reinterpret_cast<uint64_t*>(p);
    return w;
}

// Phase 1, every wave over the chunk's tokens, one per lane: the token's top-k
// row (k loads in flight), the bins it reaches as a bit mask (n_bins <= 64, bin
// map in LDS); wave w counts experts 64 w .. by label, and one wave the tokens
// per bin, as popcounts of the transposed choice bits. Phase 2, one wave per token with lanes over experts: gate
// mass of each expert over the tokens routed to its bin (fp64, fixed order).
__global__ void __launch_bounds__(kBalThreads)
bal_partial_kernel(const float* __restrict__ probs, const int32_t* __restrict__ idx,
                   const uint8_t* __restrict__ mid, int64_t T, int E, int k, const int32_t* __restrict__ e2b,
                   int n_bins, int32_t* __restrict__ cnt_out, int32_t* __restrict__ tk_out,
                   double* __restrict__ mass_out, uint64_t* __restrict__ mask_out) {
    __shared__ int32_t bin_s[256];
    __shared__ double mass[kBalWaves][256];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * kBalChunk;
    const int n = static_cast<int>(T - j0 < kBalChunk ? T - j0 : kBalChunk);
    const int64_t j = j0 + (lane < n ? lane : 0);
    int ex[SMOES_K_MAX_DEV];
#pragma unroll
    for (int s = 0; s < SMOES_K_MAX_DEV; ++s) ex[s] = s < k ? idx[j * k + s] : 0;
    const uint64_t text = __ballot(mid[j] != 0);  // lanes past the chunk chose nothing
    for (int e = threadIdx.x; e < E; e += kBalThreads) bin_s[e] = e2b[e];
    __syncthreads();
    uint64_t m = 0, mine = 0;  // bins reached; experts 64 wave .. chosen
#pragma unroll
    for (int s = 0; s < SMOES_K_MAX_DEV; ++s) {
        if (s < k) {
            m |= 1ull << bin_s[ex[s]];
            mine |= (ex[s] >> 6) == wave ? 1ull << (ex[s] & 63) : 0ull;
        }
    }
    if (lane >= n) m = mine = 0;
    if (wave == 0 && lane < n) mask_out[j] = m;
    if (wave * 64 < E) {
        // lane t: the tokens that chose expert 64 wave + t, by label
        const uint64_t chose = wave_transpose_bits(mine);
        const int c1 = __popcll(chose & text), c0 = __popcll(chose & ~text);
        const int e = wave * 64 + lane;
        if (e < E) {
            cnt_out[static_cast<int64_t>(blockIdx.x) * 2 * E + e] = c0;
            cnt_out[static_cast<int64_t>(blockIdx.x) * 2 * E + E + e] = c1;
        }
    }
    if (wave == kBalWaves - 1) {  // the wave with the fewest experts
        const int cb = __popcll(wave_transpose_bits(m));  // tokens routed to bin `lane`
        if (lane < n_bins) tk_out[static_cast<int64_t>(blockIdx.x) * n_bins + lane] = cb;
    }
    int bin_of[4];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = lane + q * kWave;
        bin_of[q] = e < E ? bin_s[e] : 0;
    }
    // tokens wave, wave + 4, ... four at a time: their rows are loaded before they are added
    constexpr int U = 4;
    for (int r0 = wave; r0 < n; r0 += U * kBalWaves) {
        float g[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * kBalWaves < n ? r0 + u * kBalWaves : r0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = lane + q * kWave;
                g[u][q] = q * kWave < E ? probs[(j0 + r) * E + (e < E ? e : 0)] : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * kBalWaves;
            if (r >= n) break;  // uniform
            const uint64_t bins = (static_cast<uint64_t>(__builtin_amdgcn_readlane(static_cast<int>(m >> 32), r)) << 32) |
                                  static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(m), r));
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q * kWave < E && ((bins >> bin_of[q]) & 1ull)) acc[q] += static_cast<double>(g[u][q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) mass[wave][lane + q * kWave] = acc[q];
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kBalThreads) {
        double sum = 0.0;
        for (int w = 0; w < kBalWaves; ++w) sum += mass[w][e];  // wave order
        mass_out[static_cast<int64_t>(blockIdx.x) * E + e] = sum;
    }
}

// After the counts are summed the three results are independent chains of
// double divisions, so each has a thread group of its own (0: Eq. 16; 1: Eq.
// 10-11; 2: Eq. 18-19) and three barriers serve them all (one after the other
// with a barrier around each of four sums: 12.9 us, now 11.9, at 64 chunks x 64
// experts).
__global__ void __launch_bounds__(kFinThreads)
bal_finalize_kernel(int64_t nchunk, int E, int n_bins, const int32_t* __restrict__ cnt_in,
                    const int32_t* __restrict__ tk_in, const double* __restrict__ mass_in, double beta,
                    double* __restrict__ load_ema, int32_t* __restrict__ counts, double* __restrict__ fspec_out,
                    int32_t* __restrict__ e2b_next, const int32_t* __restrict__ e2b, float* __restrict__ bal_loss,
                    float* __restrict__ msi_out, double* __restrict__ coef) {
    __shared__ int32_t tk_g[kFinGroups][64];
    __shared__ int32_t cnt_g[kFinGroups][2][256];
    __shared__ double mass_g[kFinGroups][256];
    __shared__ int32_t rank_g[kFinGroups][256];
    __shared__ double fs[256];
    __shared__ double red[4][4];  // wave sums of: loss term, vision load, text load, deviation
    const int e = threadIdx.x & 255, grp = threadIdx.x >> 8;  // E <= 256
    const int NB = E / n_bins;
    const int64_t len = ceil_div(nchunk, kFinGroups);
    const int64_t lo = grp * len, hi = lo + len < nchunk ? lo + len : nchunk;
    constexpr int B = 16;  // chunk loads in flight; the sums still run in chunk order
    int32_t cv = 0, ct = 0, tb = 0;
    double S = 0.0;
    const int er = e < E ? e : 0, br = e < n_bins ? e : 0;
    for (int64_t c0 = lo; c0 < hi; c0 += B) {
        int32_t vv[B], vt[B], vb[B];
        double vm[B];
#pragma unroll
        for (int q = 0; q < B; ++q) {
            const int64_t c = c0 + q < hi ? c0 + q : c0;
            vv[q] = cnt_in[c * 2 * E + er];
            vt[q] = cnt_in[c * 2 * E + E + er];
            vm[q] = mass_in[c * E + er];
            vb[q] = tk_in[c * n_bins + br];
        }
#pragma unroll
        for (int q = 0; q < B; ++q) {  // chunks past the last add 0: a branch would pull their loads into it
            const int in = -static_cast<int>(c0 + q < hi);
            cv += vv[q] & in;
            ct += vt[q] & in;
            tb += vb[q] & in;
            S += in ? vm[q] : 0.0;
        }
    }
    // needed after the block's sums: in flight during them
    const int my_bin = e2b[er];
    const double ema_v = load_ema != nullptr ? load_ema[er] : 0.0, ema_t = load_ema != nullptr ? load_ema[E + er] : 0.0;
    cnt_g[grp][0][e] = cv;
    cnt_g[grp][1][e] = ct;
    mass_g[grp][e] = S;
    if (e < 64) tk_g[grp][e] = tb;
    __syncthreads();
    const int wg = __builtin_amdgcn_readfirstlane(e / kWave);  // wave of its group
    const bool head = lane_id() == 0;
    cv = ct = 0;
    if (e < E) {
#pragma unroll
        for (int g = 0; g < kFinGroups; ++g) {
            cv += cnt_g[g][0][e];
            ct += cnt_g[g][1][e];
        }
    }
    if (grp == 0) {
        // Eq. 16 and its gradient coefficients
        double term = 0.0;
        if (e < E) {
            S = 0.0;
#pragma unroll
            for (int g = 0; g < kFinGroups; ++g) S += mass_g[g][e];
            const int32_t Tk = (tk_g[0][my_bin] + tk_g[1][my_bin]) + (tk_g[2][my_bin] + tk_g[3][my_bin]);
            const double n_e = static_cast<double>(cv) + static_cast<double>(ct);
            double c = 0.0;
            if (Tk > 0) {
                const double t = static_cast<double>(Tk);
                term = NB * (n_e / t) * (S / t);
                c = NB * (n_e / t) / t;
            }
            coef[e] = c;
            if (counts != nullptr) {
                counts[e] = cv;
                counts[E + e] = ct;
            }
        }
        const double w = wave_sum_u(term);
        if (head) red[0][wg] = w;
    } else if (grp == 1) {
        // Eq. 10: EMA of the expert loads (rows: vision, text), products rounded before the sum
        if (e < E) {
            double lv = cv, lt = ct, f = 0.5;
            if (load_ema != nullptr) {
                const double a = 1.0 - beta;
                lv = __dadd_rn(__dmul_rn(beta, ema_v), __dmul_rn(a, static_cast<double>(cv)));
                lt = __dadd_rn(__dmul_rn(beta, ema_t), __dmul_rn(a, static_cast<double>(ct)));
                load_ema[e] = lv;
                load_ema[E + e] = lt;
            }
            const double tot = __dadd_rn(lt, lv);
            if (tot > 0.0) f = __ddiv_rn(lt, tot);  // Eq. 11
            fs[e] = f;
            if (fspec_out != nullptr) fspec_out[e] = f;
        }
    } else if (grp == 2) {
        // Eq. 18's totals (integers: exact in any order)
        const double wv = wave_sum_u(static_cast<double>(cv)), wt = wave_sum_u(static_cast<double>(ct));
        if (head) {
            red[1][wg] = wv;
            red[2][wg] = wt;
        }
    }
    __syncthreads();
    auto total = [&](int i) { return (red[i][0] + red[i][1]) + (red[i][2] + red[i][3]); };
    if (threadIdx.x == 0 && bal_loss != nullptr) bal_loss[0] = static_cast<float>(total(0));
    // stable ascending rank -> consecutive bins of N_B; each group ranks a quarter of the pairs
    if (e2b_next != nullptr && e < E) {
        int rank = 0;
        const double fe = fs[e];
        const int q0 = grp * 64, q1 = q0 + 64 < E ? q0 + 64 : E;
        for (int q = q0; q < q1; ++q) rank += (fs[q] < fe || (fs[q] == fe && q < e)) ? 1 : 0;
        rank_g[grp][e] = rank;
    }
    if (grp == 2) {
        // Eq. 18-19 on this batch's counts
        const double tot_v = total(1), tot_t = total(2);
        double dev = 0.0;
        if (e < E) {
            const double nv = tot_v > 0.0 ? cv / tot_v : 0.0;
            const double nt = tot_t > 0.0 ? ct / tot_t : 0.0;
            const double den = nt + nv;
            const double c_text = den > 0.0 ? nt / den : 0.5;
            dev = 2.0 * fabs(c_text - 0.5);
        }
        const double w = wave_sum_u(dev);
        if (head) red[3][wg] = w;
    }
    __syncthreads();
    if (grp == 0 && e < E && e2b_next != nullptr)
        e2b_next[e] = ((rank_g[0][e] + rank_g[1][e]) + (rank_g[2][e] + rank_g[3][e])) / NB;
    if (threadIdx.x == 0 && msi_out != nullptr) msi_out[0] = static_cast<float>(total(3) / E);
}

__global__ void __launch_bounds__(kBalThreads)
bal_grad_kernel(const float* __restrict__ probs, const uint64_t* __restrict__ mask, int64_t T, int E,
                const int32_t* __restrict__ e2b, const double* __restrict__ coef, double scale, int accumulate,
                float* __restrict__ dlogits) {
    const int wave = threadIdx.x / kWave, lane = lane_id();
    double cf[4];
    int bin_of[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = lane + q * kWave;
        cf[q] = e < E ? coef[e] : 0.0;
        bin_of[q] = e < E ? e2b[e] : 0;
    }
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBalWaves;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * kBalWaves + wave; j < T; j += stride) {
        const uint64_t bins = mask[j];
        double g[4], dg[4], part = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = lane + q * kWave;
            g[q] = e < E ? static_cast<double>(probs[j * E + e]) : 0.0;
            dg[q] = (e < E && ((bins >> bin_of[q]) & 1ull)) ? cf[q] : 0.0;
            part += g[q] * dg[q];
        }
        const double s = wave_sum_u(part);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = lane + q * kWave;
            if (e < E) {
                float v = static_cast<float>(scale * g[q] * (dg[q] - s));
                if (accumulate) v += dlogits[j * E + e];
                dlogits[j * E + e] = v;
            }
        }
    }
}

}  // namespace

size_t binning_workspace_bytes(int64_t T, int E, int n_bins) {
    const int64_t nchunk = ceil_div(T, kBalChunk) > 0 ? ceil_div(T, kBalChunk) : 1;
    return align_up(sizeof(int32_t) * nchunk * 2 * E, 256) + align_up(sizeof(int32_t) * nchunk * n_bins, 256) +
           align_up(sizeof(double) * nchunk * E, 256) + align_up(sizeof(double) * E, 256) +
           align_up(sizeof(uint64_t) * (T > 0 ? T : 1), 256);
}

hipError_t launch_binning(const float* probs, const int32_t* topk_idx, const uint8_t* modality_id, int64_t T,
                          int E, int k, const int32_t* expert_to_bin, int n_bins, float beta, double* load_ema,
                          int32_t* counts, double* f_spec, int32_t* expert_to_bin_next, float grad_scale,
                          float* bal_loss, float* dlogits, int accumulate, float* msi, void* ws,
                          hipStream_t stream) {
    const int64_t nchunk = ceil_div(T, kBalChunk);
    BalWs w = carve(ws, nchunk > 0 ? nchunk : 1, E, n_bins);
    hipError_t err;
    if (nchunk > 0) {
        hipLaunchKernelGGL(bal_partial_kernel, dim3(static_cast<unsigned>(nchunk)), dim3(kBalThreads), 0, stream,
                           probs, topk_idx, modality_id, T, E, k, expert_to_bin, n_bins, w.cnt, w.tk, w.mass,
                           w.mask);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    const double b = static_cast<double>(beta);
    hipLaunchKernelGGL(bal_finalize_kernel, dim3(1), dim3(kFinThreads), 0, stream, nchunk, E, n_bins, w.cnt,
                       w.tk, w.mass, b, load_ema, counts, f_spec, expert_to_bin_next, expert_to_bin, bal_loss,
                       msi, w.coef);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if (dlogits != nullptr && T > 0) {
        int64_t blocks = ceil_div(T, kBalWaves);
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL(bal_grad_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kBalThreads), 0, stream,
                           probs, w.mask, T, E, expert_to_bin, w.coef, static_cast<double>(grad_scale),
                           accumulate, dlogits);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    return hipSuccess;
}

}  // namespace smoes
