// Attention-accumulated modality score (Sec. 3.2.1, Eq. 2-4).
//
// attn_fwd_kernel: causal softmax attention inside each sample, one
// workgroup per (128 query rows, query head), with the modality scores of the
// keys carried along as two extra value channels (the supplementary
// implementation note) — here as float32 matrix products next to the bf16
// MFMA product of the values, so the aggregated scores keep fp32 accuracy.
// Outputs: O[T][H][d_head] = Attn_h V (bf16) and m_heads[T][H][2] = Attn_h M
// (Eq. 3 per head). attn_update_kernel averages m_heads over heads (Eq. 3)
// and applies the norm-weighted residual mix (Eq. 4). attn_init_kernel
// writes the one-hot layer-0 scores (Eq. 2).
//
// Layout of the attention (per wave, 32 queries; per key block, 64 keys):
//   S^T = K Q^T with v_mfma_f32_32x32x16_bf16 (A = K rows from LDS, B = the
//   wave's Q rows held in registers): accumulator element v of lane l is key
//   8*(v/4) + 4*(l/32) + v%4 of the 32-key tile and query l%32, so softmax
//   statistics are per lane plus one exchange with lane l ^ 32.
//   O^T += V^T P^T: P^T's B operand is the S^T accumulator itself, read in
//   the order above; V stays row-major in LDS and the A operand (4 keys of one
//   dim per 8 bytes) comes from the transposing LDS read ds_read_b64_tr_b16:
//   within each 16-lane group, lane j supplies the address of key j/4 and
//   dims 4*(j%4) .. + 3 and receives dim j of those four keys.
// The running maximum is rescaled lazily (only when a block's maximum exceeds
// it by more than 8 in log2 units); blocks that every query of a wave sees
// whole skip the mask.
// Logits use exp2 with the scale folded into log2(e).
#include "common.h"
#include "kernels.h"

namespace smoes {

namespace {

constexpr int AT_BQ = 128;  // query rows per workgroup (4 waves x 32)
constexpr int AT_BK = 64;   // keys per block
constexpr int AT_THREADS = 256;
constexpr int AT_MP = AT_BK + 8;  // pitch of the score channels' rows: four rows x two halves on distinct banks

typedef int at_i32x4 __attribute__((ext_vector_type(4)));
typedef int at_i32x4_u __attribute__((ext_vector_type(4), aligned(2)));  // at any element
typedef short at_v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) at_v4i16 at_lds_v4i16;

// Start of the sample that holds token q: offsets[s] for the largest s < n_batch
// with offsets[s] <= q.
__device__ __forceinline__ int sample_start(const int32_t* offsets, int n_batch, int q) {
    int lo = 0, hi = n_batch - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offsets[mid] <= q) lo = mid; else hi = mid - 1;
    }
    return offsets[lo];
}

typedef float at_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 at_bf16x2 __attribute__((ext_vector_type(2)));

// Two floats to two bf16 (round to nearest even; one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(at_f32x2{a, b}, at_bf16x2));
}

// DMA: K and V start on 16-byte boundaries, as the buffer-to-LDS loads want them;
// at any other start the rows go through registers (not pipelined: correct, slower).
// Heads of 64 fit three waves per SIMD. (7000 tokens in five samples, 32 heads of 64
// over 8, with attn_update_kernel: 166 us with rows staged through registers, query
// blocks by half of the heads and two waves, now 115. All times in this file: passes one
// after another, each on other inputs than the last.)
template <int DH, bool DMA>
__global__ void __launch_bounds__(AT_THREADS)
__attribute__((amdgpu_waves_per_eu(DH == 128 ? 2 : 3, DH == 128 ? 2 : 3)))
attn_fwd_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                int64_t T, int H, int Hkv, const int32_t* __restrict__ offsets, int n_batch,
                const float* __restrict__ m_in, float scale_log2, uint16_t* __restrict__ o,
                float* __restrict__ m_heads) {
    constexpr int CPK = DH / 8;           // 16-byte chunks per key row
    constexpr int KC = DH / 16;           // K = 16 slices of the QK^T contraction
    constexpr int DT = DH / 32;           // 32-row tiles of O^T
    // K and V rows come HBM -> LDS by buffer-to-LDS loads (no registers in
    // between) into one of two buffers while the other is read: one barrier per
    // key block. Rows are unpadded and their 16-byte chunks swizzled, so that
    // the fragment reads hit distinct banks: K rows by the key (16-byte reads of
    // consecutive keys), V rows in 64-byte groups of chunks by the key's low bits
    // (the transposing reads take 64 bytes of each of 8 keys). Against rows staged
    // through registers into one padded buffer, two barriers per block: 178 -> 170
    // us for 7000 tokens in five samples, 32 heads of 128 over 8 KV heads, with
    // attn_update_kernel (215 before the score channels became matrix products, 163
    // with the order below).
    constexpr int RB = DH * 2;                    // row bytes
    constexpr int KV_BYTES = AT_BK * RB;
    constexpr int RPI = 1024 / RB;                // rows per load instruction
    constexpr int NI = AT_BK / RPI / (AT_THREADS / kWave);  // load instructions per wave, K and V each
    __shared__ __attribute__((aligned(1024))) uint8_t kv_lds[2][2 * KV_BYTES];
    __shared__ __attribute__((aligned(16))) float mv_lds[2][4 * AT_MP];
    __shared__ int off_s[AT_THREADS], key_s[AT_THREADS], order_s[AT_THREADS];

    const int nqb = static_cast<int>(ceil_div(T, AT_BQ));
    // Heads run fastest; block b runs on XCD b % 8: a multiple of eight
    // heads is dealt so that an XCD gets adjacent heads, which share KV heads.
    const int hi = static_cast<int>(blockIdx.x) % H;
    const int hq = H % 8 == 0 ? (hi % 8) * (H / 8) + hi / 8 : hi;
    const int hk = hq / (H / Hkv);
    // Query blocks run from the last one down: the longest causal ranges of a
    // sample first, and its blocks together, which share its K and V rows in L2.
    // Where several samples make a few rounds of blocks (two per CU at a time),
    // they run longest first over all samples instead, so that the launch ends
    // evenly: every block ranks them for itself from the sample offsets in LDS,
    // one thread per query block. Attention and update in us, heads of 128, from
    // the last down / ranked: 512 blocks of 2 samples 57.6 / 52.1, 1024 of 4 (4096
    // tokens) 92.5 / 85.5, 1760 of 5 164.8 / 161.9, 2048 of 8 164.1 / 162.5; but 128
    // blocks of 2 23.2 / 23.6 and 4096 of 16 314 / 322, without grouped heads 319 / 344.
    const bool ranked = n_batch > 1 && n_batch <= AT_THREADS && nqb <= AT_THREADS && gridDim.x > 256 && gridDim.x <= 2048;
    int qb = static_cast<int>(blockIdx.x) / H;
    if (ranked) {
        const int t = threadIdx.x;
        off_s[t] = t < n_batch ? offsets[t] : 0;
        __syncthreads();
        const int first = t * AT_BQ, last = first + AT_BQ < static_cast<int>(T) ? first + AT_BQ : static_cast<int>(T);
        const int ks = min(max(sample_start(off_s, n_batch, first), 0), first);
        const int key = (last - ks) / AT_BK * AT_THREADS + t;  // distinct; below 2^17
        if (t < nqb) key_s[t] = key;
        __syncthreads();
        int rank = 0;
        for (int j = 0; j < nqb; ++j) rank += key_s[j] > key ? 1 : 0;
        if (t < nqb) order_s[rank] = t;
        __syncthreads();
        qb = __builtin_amdgcn_readfirstlane(order_s[qb]);
    } else {
        qb = nqb - 1 - qb;
    }
    auto start_of = [&](int row) {
        return ranked ? sample_start(off_s, n_batch, row) : sample_start(offsets, n_batch, row);
    };
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave), lane = lane_id();
    const int half = lane >> 5, l32 = lane & 31;
    const int Ti = static_cast<int>(T);
    const int row0 = qb * AT_BQ;
    // first key any row of the block may see (clamped so that malformed offsets cannot run the loop away)
    const int kstart = min(max(start_of(row0), 0), row0);
    const int kend = min(row0 + AT_BQ, Ti);
    const int qi = row0 + wave * 32 + l32;
    const bool q_ok = qi < Ti;
    const int qe = q_ok ? qi : Ti - 1;
    const int qstart = min(max(start_of(qe), 0), qe);
    const int wq0 = row0 + wave * 32;  // first query row of this wave
    // swizzle of a K row's and a V row's chunks
    auto k_swz = [](int key) { return DH == 128 ? key & 15 : (key >> 1) & 7; };
    auto v_swz = [](int key) { return DH == 128 ? (key & 3) << 2 : ((key >> 1) & 1) << 2; };
    // The transposing V reads: 16-lane group g = lane / 16 covers dims
    // 16 (g & 1) .. + 15 of a 32-dim tile and keys 4 (g >> 1) .. + 3 of an
    // 8-key half-slice; lane j of the group points at key j / 4, dims 4 (j % 4) ..
    const int v_key = (lane >> 5) * 4 + ((lane & 15) >> 2);
    const int v_chunk = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);  // of the tile's four
    const int v_byte = v_key * RB + (lane & 1) * 8;
    // sample start of the wave's last query: the largest start of its queries
    const int wq_start_max = __builtin_amdgcn_readlane(qstart, 31);

    const i32x4_t rsK = buf_rsrc(k, static_cast<int>(T * Hkv * DH * 2));
    const i32x4_t rsV = buf_rsrc(v, static_cast<int>(T * Hkv * DH * 2));
    const i32x4_t rsM = buf_rsrc(m_in, static_cast<int>(T * 2 * 4));

    // the wave's Q rows as B fragments held in registers for the whole key
    // loop: slice c = dims 16c + 8*half .. + 7 of query qe
    at_i32x4 qf[KC];
    {
        const uint4* qrow = reinterpret_cast<const uint4*>(q + (static_cast<int64_t>(qe) * H + hq) * DH);
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            const uint4 t = qrow[2 * c + half];
            qf[c] = at_i32x4{static_cast<int>(t.x), static_cast<int>(t.y), static_cast<int>(t.z), static_cast<int>(t.w)};
        }
    }

    // Key block kb0 into buffer `buf`: this wave's share of the K and V rows, and
    // (waves 0 and 1) the keys' vision and text scores. Keys past T read zeros.
    const uint32_t lds_kv = lds_address(kv_lds), lds_mv = lds_address(mv_lds);
    const int ld_row = lane / CPK, ld_slot = lane % CPK;
    auto load_block = [&](int buf, int kb0) {
        const uint32_t dst = lds_kv + static_cast<uint32_t>(buf * 2 * KV_BYTES);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int R = (wave * NI + i) * RPI + ld_row;  // key of the block
            // T * Hkv * RB < 2^31 and a block is far smaller: a key past T stays out of range
            const int row = static_cast<int>((static_cast<uint32_t>(kb0 + R) * Hkv + hk) * static_cast<uint32_t>(RB));
            const uint32_t o = static_cast<uint32_t>((wave * NI + i) * 1024);
            if constexpr (DMA) {
                dma16(rsK, row + ((ld_slot ^ k_swz(R)) * 16), dst + o);
                dma16(rsV, row + ((ld_slot ^ v_swz(R)) * 16), dst + KV_BYTES + o);
            } else {
                uint8_t* l = kv_lds[buf] + o + lane * 16;
                const int64_t e = (static_cast<int64_t>(kb0 + R) * Hkv + hk) * DH;  // elements
                const bool in = kb0 + R < Ti;
                at_i32x4 kv4{}, vv4{};
                if (in) {
                    kv4 = *reinterpret_cast<const at_i32x4_u*>(k + e + (ld_slot ^ k_swz(R)) * 8);
                    vv4 = *reinterpret_cast<const at_i32x4_u*>(v + e + (ld_slot ^ v_swz(R)) * 8);
                }
                *reinterpret_cast<at_i32x4*>(l) = kv4;
                *reinterpret_cast<at_i32x4*>(l + KV_BYTES) = vv4;
            }
        }
        if (wave < 2)
            dma4(rsM, (kb0 + lane) * 8 + 4 * wave, lds_mv + static_cast<uint32_t>((buf * 4 + wave) * AT_MP * 4));
    };

    f32x16_t oacc[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i) oacc[i] = f32x16_t{};
    float m_run = -INFINITY, l_run = 0.f, a0 = 0.f, a1 = 0.f;

    // rows 2 and 3 of the score channels: ones (the softmax denominator) and zeros
    if (threadIdx.x < 2 * AT_MP)
        mv_lds[0][2 * AT_MP + threadIdx.x] = mv_lds[1][2 * AT_MP + threadIdx.x] = threadIdx.x < AT_MP ? 1.f : 0.f;
    // keys that some query of this wave may see
    const int wk_lo = __builtin_amdgcn_readlane(qstart, 0), wk_hi = wq0 + 31;

    const int nkb = static_cast<int>(ceil_div(kend - kstart, AT_BK));
    load_block(0, kstart);
    for (int b = 0; b < nkb; ++b) {
        const int kb0 = kstart + b * AT_BK;
        // this wave's loads of block b have landed; behind the barrier every wave's
        // have, and every wave is done reading the other buffer
        wait_vm_lgkm0<0>();
        dma_barrier();
        if (b + 1 < nkb) load_block((b + 1) & 1, kb0 + AT_BK);
        if (kb0 > wk_hi || kb0 + AT_BK <= wk_lo) continue;  // uniform; the barriers are above
        // LDS addresses are rebuilt inside the loop from an opaque zero: hoisting
        // all of them out of the loop would not fit the register budget
        int lz = 0;
        asm volatile("" : "+v"(lz));
        const uint8_t* kl = kv_lds[b & 1] + l32 * RB + lz;
        const uint8_t* vl = kv_lds[b & 1] + KV_BYTES + v_byte + lz;
        const float* ml = mv_lds[b & 1] + (lane & 3) * AT_MP + lz;
        const int k_x = half ^ k_swz(l32), v_x = v_chunk ^ v_swz(v_key);  // 32-key tiles and 4-key steps keep the swizzle

        // S^T = K Q^T for the two 32-key tiles; K fragments read two slices ahead
        // (the scheduling barriers keep the compiler from hoisting every LDS
        // read of the block, which would not fit the register budget)
        f32x16_t s[2] = {f32x16_t{}, f32x16_t{}};
        auto kfrag = [&](int c, int t) {
            return *reinterpret_cast<const bf16x8_t*>(kl + t * 32 * RB + ((2 * c) ^ k_x) * 16);
        };
        bf16x8_t ka[3][2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            ka[c][0] = kfrag(c, 0);
            ka[c][1] = kfrag(c, 1);
        }
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            if (c + 2 < KC) {
                ka[(c + 2) % 3][0] = kfrag(c + 2, 0);
                ka[(c + 2) % 3][1] = kfrag(c + 2, 1);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
                s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[c % 3][t], __builtin_bit_cast(bf16x8_t, qf[c]), s[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // The block maximum of this query's logits; keys outside the query's
        // sample or past its diagonal are masked, except in blocks that every
        // query of the wave sees whole (the common case, checked per wave).
        const bool full = kb0 >= wq_start_max && kb0 + AT_BK - 1 <= wq0;
        float mx = -INFINITY;
        if (full) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[t][e]);
        } else {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = kb0 + t * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                    const float x = (key >= qstart && key <= qe) ? s[t][e] : -INFINITY;
                    s[t][e] = x;
                    mx = fmaxf(mx, x);
                }
        }
        const float mblk = fmaxf(mx, __shfl_xor(mx, 32, kWave)) * scale_log2;
        // Lazy rescaling: the reference m_run moves only when a block's maximum
        // exceeds it by more than 8 (log2 units), so exp2 stays below 2^8 and
        // the accumulators are rescaled in few blocks. Both halves of a query
        // take the same decision.
        const bool grow = mblk > m_run + 8.f;
        if (__builtin_amdgcn_ballot_w64(grow) != 0) {
            const float m_new = grow ? mblk : m_run;
            const float alpha = grow ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;  // m_run = -inf: 0
            m_run = m_new;
            l_run *= alpha;
            a0 *= alpha;
            a1 *= alpha;
#pragma unroll
            for (int i = 0; i < DT; ++i) oacc[i] *= alpha;
        }
        const float m_use = m_run == -INFINITY ? 0.f : m_run;
        // The score channels and the softmax denominator in float32 on the
        // matrix cores beside the exponentials: v_mfma_f32_4x4x1 treats each
        // group of four lanes by itself, so with lane c of a group holding
        // channel c of a key (vision, text, 1, 0) and every lane the key's
        // probability for its own query, element c of a lane's result is its
        // query's sum of channel c. (Three FMAs per probability on the vector
        // ALUs, which bound the block, became one 8-cycle matrix instruction.)
        f32x4_t sc[2] = {f32x4_t{}, f32x4_t{}};
        // four consecutive keys of this lane, one group ahead
        auto chan = [&](int i) { return *reinterpret_cast<const f32x4_t*>(ml + 8 * i + 4 * half); };
        // V fragments of 16-key slice c: keys 16c + 4 half + 0..3 and 16c + 8 + 4 half + 0..3 of dim 32i + lane % 32
        auto vfrag = [&](int c, at_i32x4 (&va)[DT]) {
#pragma unroll
            for (int i = 0; i < DT; ++i) {
                const uint8_t* va_i = vl + ((4 * i) ^ v_x) * 16;
                const at_v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((at_lds_v4i16*)(va_i + 16 * c * RB));
                const at_v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((at_lds_v4i16*)(va_i + (16 * c + 8) * RB));
                const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                va[i] = at_i32x4{static_cast<int>(l2.x), static_cast<int>(l2.y), static_cast<int>(h2.x), static_cast<int>(h2.y)};
            }
        };
        at_i32x4 va[2][DT];
        f32x4_t mcn = chan(0);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                __builtin_amdgcn_sched_barrier(0);
                const f32x4_t mc = mcn;
                if (4 * t + g < 7) mcn = chan(4 * t + g + 1);
                else vfrag(0, va[0]);  // the value product's first slice comes in under the last group
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[t][4 * g + e], scale_log2, -m_use));
                    s[t][4 * g + e] = p;
                    sc[t] = __builtin_amdgcn_mfma_f32_4x4x1f32(mc[e], p, sc[t], 0, 0, 0);
                }
            }
        a0 += sc[0][0] + sc[1][0];
        a1 += sc[0][1] + sc[1][1];
        l_run += sc[0][2] + sc[1][2];
        // O^T += V^T P^T over four 16-key slices
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c < 3) vfrag(c + 1, va[(c + 1) & 1]);
            const f32x16_t& st = s[c >> 1];
            const int e0 = 8 * (c & 1);
            const at_i32x4 pb{static_cast<int>(pack_bf16x2(st[e0 + 0], st[e0 + 1])),
                              static_cast<int>(pack_bf16x2(st[e0 + 2], st[e0 + 3])),
                              static_cast<int>(pack_bf16x2(st[e0 + 4], st[e0 + 5])),
                              static_cast<int>(pack_bf16x2(st[e0 + 6], st[e0 + 7]))};
#pragma unroll
            for (int i = 0; i < DT; ++i)
                oacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, va[c & 1][i]),
                                                                  __builtin_bit_cast(bf16x8_t, pb), oacc[i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // both halves of the wave hold partial sums of the same query
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    const float a0t = a0 + __shfl_xor(a0, 32, kWave);
    const float a1t = a1 + __shfl_xor(a1, 32, kWave);
    if (!q_ok) return;
    const float inv = 1.f / l_tot;
    uint16_t* orow = o + (static_cast<int64_t>(qi) * H + hq) * DH;
#pragma unroll
    for (int i = 0; i < DT; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int d0 = i * 32 + 8 * g + 4 * half;
            *reinterpret_cast<uint2*>(orow + d0) =
                make_uint2(pack_bf16x2(oacc[i][4 * g] * inv, oacc[i][4 * g + 1] * inv),
                           pack_bf16x2(oacc[i][4 * g + 2] * inv, oacc[i][4 * g + 3] * inv));
        }
    if (half == 0) {
        float* mh = m_heads + (static_cast<int64_t>(qi) * H + hq) * 2;
        mh[0] = a0t / l_tot;
        mh[1] = a1t / l_tot;
    }
}

// Eq. 3 head average and Eq. 4 mix: one wave per token.
template <bool BF16>
__global__ void __launch_bounds__(256) attn_update_kernel(const void* __restrict__ x, const void* __restrict__ x_attn,
                                                          int64_t T, int d, const float* __restrict__ m_heads, int H,
                                                          const float* m_in, float* m_out) {
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 4 + threadIdx.x / kWave;
    if (j >= T) return;
    const int lane = lane_id();
    float sx = 0.f, sa = 0.f;
    for (int c = lane * 8; c < d; c += kWave * 8) {
        float a[8], b[8];
        load8<BF16>(x, j * d + c, a);
        load8<BF16>(x_attn, j * d + c, b);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            sx += a[e] * a[e];
            sa += b[e] * b[e];
        }
    }
    sx = wave_sum_u(sx);
    sa = wave_sum_u(sa);
    if (lane != 0) return;
    const float nx = sqrtf(sx), na = sqrtf(sa);
    float t0 = 0.f, t1 = 0.f;
    for (int h = 0; h < H; ++h) {
        t0 += m_heads[(j * H + h) * 2];
        t1 += m_heads[(j * H + h) * 2 + 1];
    }
    const float invh = 1.f / static_cast<float>(H);
    const float m0 = m_in[j * 2], m1 = m_in[j * 2 + 1];
    const float den = nx + na;
    float r0 = m0, r1 = m1;
    if (den > 0.f) {
        r0 = (na * (t0 * invh) + nx * m0) / den;
        r1 = (na * (t1 * invh) + nx * m1) / den;
    }
    m_out[j * 2] = r0;
    m_out[j * 2 + 1] = r1;
}

__global__ void attn_init_kernel(const uint8_t* __restrict__ modality_id, int64_t T, float* __restrict__ M) {
    for (int64_t j = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; j < T;
         j += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const uint8_t m = modality_id[j];
        M[2 * j] = m == 0 ? 1.f : 0.f;
        M[2 * j + 1] = m == 1 ? 1.f : 0.f;
    }
}

}  // namespace

hipError_t launch_attention(const void* q, const void* k, const void* v, int64_t T, int H, int Hkv, int head_dim,
                            const int32_t* sample_offsets, int n_batch, const float* m_in, float scale, void* o,
                            float* m_heads, hipStream_t stream) {
    if (T == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(ceil_div(T, AT_BQ) * H));
    const float scale_log2 = scale * 1.4426950408889634f;
    const bool dma = (reinterpret_cast<uintptr_t>(k) | reinterpret_cast<uintptr_t>(v)) % 16 == 0;
    const auto kernel = head_dim == 128 ? (dma ? attn_fwd_kernel<128, true> : attn_fwd_kernel<128, false>)
                                        : (dma ? attn_fwd_kernel<64, true> : attn_fwd_kernel<64, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(AT_THREADS), 0, stream, static_cast<const uint16_t*>(q),
                       static_cast<const uint16_t*>(k), static_cast<const uint16_t*>(v), T, H, Hkv, sample_offsets,
                       n_batch, m_in, scale_log2, static_cast<uint16_t*>(o), m_heads);
    return hipGetLastError();
}

hipError_t launch_attn_update(const void* x, const void* x_attn, int act_dtype, int64_t T, int d,
                              const float* m_heads, int H, const float* m_in, float* m_out, hipStream_t stream) {
    if (T == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(ceil_div(T, 4)));
    if (act_dtype == 1)
        hipLaunchKernelGGL(attn_update_kernel<true>, grid, dim3(256), 0, stream, x, x_attn, T, d, m_heads, H, m_in, m_out);
    else
        hipLaunchKernelGGL(attn_update_kernel<false>, grid, dim3(256), 0, stream, x, x_attn, T, d, m_heads, H, m_in, m_out);
    return hipGetLastError();
}

hipError_t launch_attn_init(const uint8_t* modality_id, int64_t T, float* M, hipStream_t stream) {
    if (T == 0) return hipSuccess;
    const int64_t b = ceil_div(T, 256);
    hipLaunchKernelGGL(attn_init_kernel, dim3(static_cast<unsigned>(b < 4096 ? b : 4096)), dim3(256), 0, stream,
                       modality_id, T, M);
    return hipGetLastError();
}

}  // namespace smoes
