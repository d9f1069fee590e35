// Grouped SwiGLU experts, shared experts and the weighted combine.
//
// Groups: g < E is routed expert g over its expert-contiguous rows
// [off[g], off[g+1]) (rows gathered from x through perm_token inside the
// GEMM's loader, so no permuted copy of x is written); g = E is the merged
// shared expert over all T tokens. A work table (prefix over groups of
// m_tiles * n_tiles, written on the device by the permutation) lets one
// launch cover every group without any host synchronisation.
//
// Block -> tile mapping: blocks are dealt round-robin to the 8 XCDs, so block b
// runs on XCD b % 8. Each XCD takes one contiguous eighth of the work list,
// ordered (group, super-row of m-tiles, n-tile, m-tile): the tiles that share
// a weight slice run back to back on one XCD and hit its L2 (8 m-tiles per
// super-row for the row-major path; the packed path picks the count per
// product).
//
// bf16, packed weights (the fast path, gemm_bf16_pk_kernel): 16x16x32 MFMA
// tiles with the weights loaded straight into registers; its layout and
// schedule are described where it is defined.
// bf16, row-major weights: 128 x 128 tiles, 4 waves of 64 x 64 (2 x 2 MFMA
// 32x32x16 bf16 tiles), fp32 accumulation. Operand tiles are copied HBM ->
// LDS by buffer loads with an LDS destination (no register staging) through
// a three-stage ring of K = 32 slices; the MFMA fragments are read back with
// 16-byte LDS reads from XOR-swizzled rows. The results leave through LDS as
// 16-byte row chunks.
//   GEMM1: B rows 0..63 are gate rows, 64..127 the matching up rows, so a
//          wave holds gate and up outputs of the same (row, column) in the
//          same lane: the SwiGLU epilogue is register-local. H is bf16.
//   GEMM2: Y = H W2^T, bf16.
// f32 (exact path for float32 layers): gemm_rm_kernel on the float32 matrix
// instructions, same work table.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace smoes {

namespace {

constexpr int kThreads = 256;
constexpr int kGroupM = 8;  // m-tiles per super-row in the work order

// rows per tile of the row-major matrix tiles (gemm_rm_kernel)
constexpr int FBM = 64;

struct ExpWs {
    void* h_r;   // [R, inter]
    void* h_s;   // [T, shared_inter]
    void* y_r;   // [R, d]
    void* y_s;   // [T, d]
    int32_t* work1;  // [E + 2]
    int32_t* work2;  // [E + 2]
};

size_t esz(int act_dtype) { return act_dtype == 1 ? 2 : 4; }

ExpWs carve(void* ws, int64_t T, int d, int k, int inter, int shared_inter, int act_dtype, int E) {
    ExpWs w;
    const int64_t R = T * k;
    char* p = static_cast<char*>(ws);
    const size_t s = esz(act_dtype);
    w.h_r = p;
    p += align_up(s * R * inter, 256);
    w.h_s = p;
    p += align_up(s * T * shared_inter, 256);
    w.y_r = p;
    p += align_up(s * R * d, 256);
    w.y_s = p;
    p += align_up(s * T * d, 256);
    w.work1 = reinterpret_cast<int32_t*>(p);
    p += align_up(sizeof(int32_t) * (E + 2), 256);
    w.work2 = reinterpret_cast<int32_t*>(p);
    return w;
}

struct Tile {
    int g;          // group (E = shared)
    int64_t row0;   // first row of the tile in the group's row space (global row index)
    int rows;       // valid rows in the tile
    int nt;         // n-tile
};

// Decode this block's tile; returns false when the block has no work.
// Block b runs on XCD b % 8. The routed items and the shared-expert items are
// each cut into 8 contiguous ranges, one per XCD, so every XCD gets the same
// share of both kinds (shared tiles can have a longer K than routed ones).
// Inside a group items run (super-row of group_m m-tiles, n-tile, m-tile).
// part: 0 every item, 1 routed items only, 2 shared items only. The shared
// part never reads the work table (its item count follows from T and the
// tiling), so it can run before the routing has been permuted.
__device__ __forceinline__ bool decode_tile(const int32_t* __restrict__ work, const int32_t* __restrict__ off,
                                            int E, int64_t T, int bm, int nt_routed, int nt_shared,
                                            int part, Tile& t, int group_m = kGroupM) {
    const int xcd = blockIdx.x & 7;
    const int slot = blockIdx.x >> 3;
    int g, local;
    int64_t base, rows_g;
    if (part == 2) {
        const int ns = static_cast<int>(ceil_div(T, bm)) * nt_shared;
        const int s8 = (ns + 7) / 8;
        const int s_lo = min(xcd * s8, ns), s_hi = min(s_lo + s8, ns);
        if (slot >= s_hi - s_lo) return false;
        g = E;
        local = s_lo + slot;
    } else {
        const int routed = work[E];
        const int ns = part == 1 ? 0 : work[E + 1] - routed;
        const int r8 = (routed + 7) / 8, s8 = (ns + 7) / 8;
        const int r_lo = min(xcd * r8, routed), r_hi = min(r_lo + r8, routed);
        const int s_lo = min(xcd * s8, ns), s_hi = min(s_lo + s8, ns);
        // shared items first: their K can be longer (GEMM2), and blocks are
        // dispatched in index order, so the longest tiles start earliest
        int w;
        if (slot < s_hi - s_lo) w = routed + s_lo + slot;
        else if (slot < (s_hi - s_lo) + (r_hi - r_lo)) w = r_lo + (slot - (s_hi - s_lo));
        else return false;
        if (w >= routed) {
            g = E;
            local = w - routed;
        } else {
            // the last g with work[g] <= w: lane l holds entries l, l + 64, ... of the
            // table and the offsets, all loaded at once (a binary search waits for
            // log2(E) dependent loads before the tile's first operand load)
            const int lane = lane_id();
            int wv[4], ov[4], on[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (64 * q >= E) break;  // uniform
                const int e = lane + 64 * q < E ? lane + 64 * q : E - 1;
                wv[q] = work[e];
                ov[q] = off[e];
                on[q] = off[e + 1];
            }
            int n = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (64 * q >= E) break;
                n += __popcll(__ballot(lane + 64 * q < E && wv[q] <= w));
            }
            g = n - 1;  // work[0] = 0
            int wg = 0, o0 = 0, o1 = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (64 * q >= E) break;
                if ((g >> 6) == q) {
                    wg = __builtin_amdgcn_readlane(wv[q], g & 63);
                    o0 = __builtin_amdgcn_readlane(ov[q], g & 63);
                    o1 = __builtin_amdgcn_readlane(on[q], g & 63);
                }
            }
            local = w - wg;
            base = o0;
            rows_g = o1 - o0;
        }
    }
    int ntn;
    if (g < E) {
        ntn = nt_routed;
    } else {
        base = 0;
        rows_g = T;
        ntn = nt_shared;
    }
    const int m_tiles = static_cast<int>(ceil_div(rows_g, bm));
    const int sb = local / (group_m * ntn);
    const int r = local % (group_m * ntn);
    const int gm = m_tiles - sb * group_m < group_m ? m_tiles - sb * group_m : group_m;
    const int mt = sb * group_m + r % gm;
    t.g = g;
    t.nt = r / gm;
    t.row0 = base + static_cast<int64_t>(mt) * bm;
    const int64_t left = rows_g - static_cast<int64_t>(mt) * bm;
    t.rows = static_cast<int>(left < bm ? left : bm);
    return true;
}

typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;

__device__ __forceinline__ float silu(float a) { return a / (1.0f + expf(-a)); }

__device__ __forceinline__ uint4 as_uint4(i32x4_t v) {
    return make_uint4(static_cast<uint32_t>(v.x), static_cast<uint32_t>(v.y), static_cast<uint32_t>(v.z),
                      static_cast<uint32_t>(v.w));
}

struct GemmArgs {
    int64_t T;
    int d, E, k, inter, shared_inter;
    int part;    // work items of this launch: 0 all, 1 routed, 2 shared
    const void* x;
    const void* w13;
    const void* w2;
    const void* ws13;
    const void* ws2;
    const int32_t* off;
    const int32_t* perm_token;
    const int32_t* work;
    void* h_r;
    void* h_s;
    void* y_r;
    void* y_s;
    // backward (modes 3-5 of the packed kernel)
    const void* dout;   // [T][d] upstream gradient
    const void* w2t;    // packed W2^T per expert (N = inter, K = d)
    const void* ws2t;   // packed Ws2^T (N = shared_inter, K = d)
    const void* w13t;   // packed W13^T per expert (N = d, K = 2 inter)
    const void* ws13t;  // packed Ws13^T (N = d, K = 2 shared_inter)
    void* ab_r;         // [R][2 inter] pre-activations (gate | up), routed rows
    void* ab_s;         // [T][2 shared_inter]
    void* dx_r;         // [R][d] input gradient of each routed row
    void* dx_s;         // [T][d] shared experts' input gradient
    const float* wrow;  // [R] combine weight of each routed row
    // mode 4 outputs, k-packed (wgrad.hip): the routed rows' [dA dB] and w H (kp:
    // padded row prefix of the experts), the shared [dA dB]; mode 5 reads [dA dB]
    uint16_t* pt_dab_r;
    uint16_t* pt_wh_r;
    uint16_t* pt_dab_s;
    const int32_t* kp;
    // shared down GEMM with the combine in its epilogue (mode 7)
    const int32_t* inv;    // [T][k] routed row of each (token, slot)
    const float* topk_w;   // [T][k] combine weights
    void* out;             // [T][d] layer output
};

// ============================================================== bf16 MFMA path

// The operand tiles go straight from HBM to LDS (buffer_load ... lds: each wave instruction writes
// 64 x 16 bytes contiguously), through a ring of STAGES buffers, with one
// barrier per K step and no VGPR staging. Rows are unpadded (BK bf16) and the
// 16-byte chunks of a row are XOR-swizzled with (row / SWZ_DIV) % CPR so that
// the MFMA fragment reads of consecutive rows fall in different banks.
template <int WAVES_M_, int WAVES_N_, int TM_, int TN_, int BK_, int STAGES_, int SWZ_DIV_>
struct DmaCfg {
    static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, TM = TM_, TN = TN_, BK = BK_;
    static constexpr int STAGES = STAGES_, SWZ_DIV = SWZ_DIV_;
    static constexpr int THREADS = WAVES_M * WAVES_N * 64;
    static constexpr int BM = WAVES_M * TM * 32;
    static constexpr int BNB = WAVES_N * TN * 32;
    static constexpr int CPR = BK / 8;                 // 16-byte chunks per row
    static constexpr int RPI = 64 / CPR;               // rows per DMA instruction (1 KB)
    static constexpr int IA = BM / RPI / (THREADS / 64);   // A instructions per wave per stage
    static constexpr int IB = BNB / RPI / (THREADS / 64);  // B instructions per wave per stage
    static_assert(IA * RPI * (THREADS / 64) == BM && IB * RPI * (THREADS / 64) == BNB, "tile / wave mismatch");
    static_assert(TN % 2 == 0, "gate/up pairs need an even TN");
};

// 128 rows x 128 B-rows (GEMM1: 64 gate + 64 up rows; GEMM2: 128 output columns),
// 4 waves of 64 x 64, K step 32, three-stage ring (48 KB of LDS: 3 blocks per CU)
using DCfg = DmaCfg<2, 2, 2, 2, 32, 3, 2>;

template <class C>
constexpr int tile_cols(int mode) { return mode == 1 ? C::BNB / 2 : C::BNB; }

template <class C>
__device__ __forceinline__ int dma_slot(int row, int chunk) {
    return chunk ^ ((row / C::SWZ_DIV) % C::CPR);
}


template <int MODE, class C>
__global__ void __launch_bounds__(C::THREADS, 1)
gemm_bf16_dma_kernel(GemmArgs p) {
    constexpr int BM = C::BM, BNB = C::BNB, BK = C::BK, CPR = C::CPR, RPI = C::RPI;
    constexpr int TM = C::TM, TN = C::TN, IA = C::IA, IB = C::IB, ST = C::STAGES;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BNB * BK * 2;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[ST][A_BYTES + B_BYTES];
    constexpr int TC = tile_cols<C>(MODE);
    const int nt_r = static_cast<int>(ceil_div(MODE == 1 ? p.inter : p.d, TC));
    const int nt_s = MODE == 1 ? static_cast<int>(ceil_div(p.shared_inter, TC)) : nt_r;
    Tile t;
    if (!decode_tile(p.work, p.off, p.E, p.T, BM, nt_r, nt_s, p.part, t)) return;
    const bool shared = t.g == p.E;
    const int wave = threadIdx.x / kWave, lane = lane_id();
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;

    int K, n_out;
    const uint16_t* Abase;
    const uint16_t* Bbase;
    int a_ld;
    int64_t a_rows, b_rows;
    if constexpr (MODE == 1) {
        K = p.d;
        n_out = shared ? p.shared_inter : p.inter;
        Abase = static_cast<const uint16_t*>(p.x);
        a_ld = p.d;
        a_rows = p.T;
        b_rows = 2 * static_cast<int64_t>(n_out);
        Bbase = shared ? static_cast<const uint16_t*>(p.ws13)
                       : static_cast<const uint16_t*>(p.w13) + static_cast<int64_t>(t.g) * 2 * p.inter * p.d;
    } else {
        K = shared ? p.shared_inter : p.inter;
        n_out = p.d;
        Abase = shared ? static_cast<const uint16_t*>(p.h_s) : static_cast<const uint16_t*>(p.h_r);
        a_ld = K;
        a_rows = shared ? p.T : p.T * p.k;
        b_rows = p.d;
        Bbase = shared ? static_cast<const uint16_t*>(p.ws2)
                       : static_cast<const uint16_t*>(p.w2) + static_cast<int64_t>(t.g) * p.d * p.inter;
    }
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(Abase), 0, static_cast<int>(a_rows * a_ld * 2), kBufferFlags);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(Bbase), 0, static_cast<int>(b_rows * K * 2), kBufferFlags);

    // Lane `lane` of this wave's q-th instruction fills LDS row R = (wave * I + q) * RPI + lane / CPR,
    // slot lane % CPR, with the row's chunk slot ^ swizzle(R).
    const int lrow = lane / CPR, lslot = lane % CPR;
    int aoff[IA], boff[IB];  // element offset of the row start
    int achk[IA], bchk[IB];  // k offset of the chunk this lane moves (after the swizzle)
#pragma unroll
    for (int q = 0; q < IA; ++q) {
        const int R = (wave * IA + q) * RPI + lrow;
        const int rr = R < t.rows ? R : 0;
        int src;
        if (MODE == 1 && !shared) src = p.perm_token[t.row0 + rr];
        else src = static_cast<int>(t.row0 + rr);
        aoff[q] = src * a_ld;
        achk[q] = (lslot ^ ((R / C::SWZ_DIV) % CPR)) * 8;
    }
#pragma unroll
    for (int q = 0; q < IB; ++q) {
        const int R = (wave * IB + q) * RPI + lrow;
        int bi;
        if constexpr (MODE == 1) {
            int cc = t.nt * TC + (R % (BNB / 2));
            if (cc >= n_out) cc = 0;
            bi = R < BNB / 2 ? cc : n_out + cc;
        } else {
            int cc = t.nt * TC + R;
            if (cc >= n_out) cc = 0;
            bi = cc;
        }
        boff[q] = bi * K;
        bchk[q] = (lslot ^ ((R / C::SWZ_DIV) % CPR)) * 8;
    }
    // a chunk past K (K % 8 == 0) gets an offset beyond the record count: the DMA writes zeros
    auto issue = [&](int stage, int k0) {
        uint8_t* base = lds[stage];
#pragma unroll
        for (int q = 0; q < IA; ++q) {
            const int k = k0 + achk[q];
            const int vo = k < K ? (aoff[q] + k) * 2 : kOutOfRange;
            auto* dst = (__attribute__((address_space(3))) void*)(base + (wave * IA + q) * 1024);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, dst, 16, vo, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < IB; ++q) {
            const int k = k0 + bchk[q];
            const int vo = k < K ? (boff[q] + k) * 2 : kOutOfRange;
            auto* dst = (__attribute__((address_space(3))) void*)(base + A_BYTES + (wave * IB + q) * 1024);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, dst, 16, vo, 0, 0, 0);
        }
    };
    int bsub[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if constexpr (MODE == 1)
            bsub[j] = (j < TN / 2) ? (wn * (TN / 2) + j) * 32 : BNB / 2 + (wn * (TN / 2) + j - TN / 2) * 32;
        else
            bsub[j] = (wn * TN + j) * 32;
    }
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x16_t{};
    const int half = lane >> 5, l32 = lane & 31;
    auto compute = [&](int stage) {
        const uint8_t* base = lds[stage];
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int c = ks * 2 + half;
            bf16x8_t af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int R = (wm * TM + i) * 32 + l32;
                af[i] = *reinterpret_cast<const bf16x8_t*>(base + R * (BK * 2) + dma_slot<C>(R, c) * 16);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int R = bsub[j] + l32;
                bfr[j] = *reinterpret_cast<const bf16x8_t*>(base + A_BYTES + R * (BK * 2) + dma_slot<C>(R, c) * 16);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
    };

    // K loop: ST-stage ring. Before reading stage kt, this wave waits until at
    // most (ST - 2) newer stages of its own loads are in flight and its LDS
    // reads are done, then a barrier makes every wave's loads visible and
    // frees the stage that the next loads overwrite.
    static_assert(ST == 3, "the loop below is written for three stages");
    constexpr int PER_STAGE = IA + IB;
    const int nk = static_cast<int>(ceil_div(K, BK));
    issue(0, 0);
    issue(1, BK);
    int kt = 0;
    for (; kt + 3 <= nk; kt += 3) {
        wait_vm_lgkm0<PER_STAGE>();
        __builtin_amdgcn_s_barrier();
        issue(2, (kt + 2) * BK);
        compute(0);
        wait_vm_lgkm0<PER_STAGE>();
        __builtin_amdgcn_s_barrier();
        issue(0, (kt + 3) * BK);
        compute(1);
        wait_vm_lgkm0<PER_STAGE>();
        __builtin_amdgcn_s_barrier();
        issue(1, (kt + 4) * BK);
        compute(2);
    }
    if (kt < nk) {
        wait_vm_lgkm0<PER_STAGE>();
        __builtin_amdgcn_s_barrier();
        issue(2, (kt + 2) * BK);
        compute(0);
    }
    if (kt + 1 < nk) {
        wait_vm_lgkm0<PER_STAGE>();
        __builtin_amdgcn_s_barrier();
        compute(1);
    }
    wait_vm_lgkm0<0>();  // drain the ring: the epilogue reuses its LDS
    __builtin_amdgcn_s_barrier();

    // Epilogue through LDS: each wave writes its bf16 results (GEMM1: the
    // SwiGLU output) into a [BM][TC + 8] tile, then every thread stores whole
    // 16-byte row chunks. Element v of a 32x32 MFMA tile sits at row
    // 8*(v/4) + 4*half + v%4, column l32.
    constexpr int OP = TC + 8;  // row pitch (bf16) of the output tile
    static_assert(BM * OP * 2 <= ST * (A_BYTES + B_BYTES), "output tile must fit the ring");
    uint16_t* otile = reinterpret_cast<uint16_t*>(&lds[0][0]);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = (wm * TM + i) * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
            if constexpr (MODE == 1) {
#pragma unroll
                for (int j = 0; j < TN / 2; ++j) {
                    const int c = (wn * (TN / 2) + j) * 32 + l32;
                    otile[r * OP + c] = f32_to_bf16(silu(acc[i][j][v]) * acc[i][j + TN / 2][v]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int c = (wn * TN + j) * 32 + l32;
                    otile[r * OP + c] = f32_to_bf16(acc[i][j][v]);
                }
            }
        }
    }
    __syncthreads();
    uint16_t* O;
    if constexpr (MODE == 1) O = shared ? static_cast<uint16_t*>(p.h_s) : static_cast<uint16_t*>(p.h_r);
    else O = shared ? static_cast<uint16_t*>(p.y_s) : static_cast<uint16_t*>(p.y_r);
    constexpr int CH = TC / 8;  // 16-byte chunks per output row
    const int col0 = t.nt * TC;
    for (int q = threadIdx.x; q < BM * CH; q += C::THREADS) {
        const int r = q / CH, ch = q % CH;
        const int c = col0 + ch * 8;
        if (r < t.rows && c < n_out)  // n_out % 8 == 0: a chunk is all in or all out
            *reinterpret_cast<uint4*>(O + (t.row0 + r) * n_out + c) =
                *reinterpret_cast<const uint4*>(otile + r * OP + ch * 8);
    }
}

// ============================================================== bf16 MFMA path, packed weights
//
// Packed weights: a matrix W[N][K] (N output rows, K contraction) is stored as
// 16-byte fragments P[2 ceil(N/32)][ceil(K/32)][64][8] with
//   P[h][c][l][e] = W[16 h + l % 16][32 c + 8 (l / 16) + e]   (zero outside W),
// which is exactly the A operand of v_mfma_f32_16x16x32_bf16 for output
// rows 16 h .. 16 h + 15 and contraction slice 32 c .. 32 c + 31: one wave
// loads it with one fully coalesced 1 KB buffer load, straight into VGPRs.
// (N is padded to a multiple of 32 so that a matrix holds the same number of
// 16-row groups in every packed form.) GEMM1 packs the gate and up rows
// interleaved by 16-row groups in blocks of 32 output columns (groups 4q ..
// 4q + 3 = gate rows 32q.., up rows 32q.., gate rows 32q + 16.., up rows
// 32q + 16..), so one wave holds gate and up outputs of the same (row,
// column) in the same lane.
//
// The 16x16x32 instruction rather than 32x32x16: both run at the same
// nominal rate and the tile below feeds them the same operand bytes, but with
// random bf16 operands and every SIMD busy the chip holds ~12 % more 16x16x32
// flops under its power limit (1.98 vs 1.76 PFLOP/s sustained from registers).
//
// Tiles: 128 rows x 4 waves; each wave owns all 128 rows and 64 B-rows (four
// 16-row groups: 8 x 4 MFMA tiles of 16 x 16). The weights never pass through
// LDS and no two waves read the same weight bytes; only the token rows (x
// gathered through perm_token for GEMM1, H for GEMM2) are staged HBM -> LDS by
// buffer_load ... lds through a three-stage ring of K = 64 slices. The
// weight loads of the next slice and the token-row DMA of the slice after
// are spread between the MFMAs of the current one.
//   GEMM1: 128 H columns per tile (32 per wave), SwiGLU in registers.
//   GEMM2: 256 output columns per tile (64 per wave).
constexpr int PK_BM = 128, PK_BK = 64, PK_WAVES = 4, PK_THREADS = PK_WAVES * 64, PK_ST = 3;
constexpr int PK_IA = PK_BM * PK_BK * 2 / 1024 / PK_WAVES;  // A DMA instructions per wave per stage
// Modes: 1 GEMM1 (+ SwiGLU), 2 GEMM2, and for the backward 3 GEMM1 with the
// raw gate and up outputs, 4 dH = dout W2 (rows gathered, scaled by the combine
// weight) with the SwiGLU backward in the epilogue, 5 dX = [dA dB] W13, and 6
// GEMM1 writing both H and the gate and up outputs (a forward that keeps them
// for the backward); 7 the shared experts' GEMM2 whose epilogue is the
// combine (run after the routed GEMM2 has written every routed row). Modes 1, 3 and 6 pair gate and up groups (32 H columns
// per wave); 2, 4 and 5 give each wave two consecutive 32-column groups.
constexpr int pk_family(int mode) { return (mode == 1 || mode == 3 || mode == 6) ? 1 : 2; }
// Row tiles per super-row of the work order (row tiles that take one weight
// slice back to back), chosen by same-box A/B at 16384 x 4096 with 160 + 2
// experts: 4 for the down products of the forward (modes 2, 7; 8 -> 4 took
// the routed launch from 1.29 to 1.27 ms), 16 for the rest (gate/up: the
// merged launch 2.83 -> 2.79 ms; the backward's dX 1.56 -> 1.53 ms, dH
// unchanged; 4 there made the backward 0.9 % slower).
constexpr int pk_group_m(int mode) { return (mode == 2 || mode == 7) ? 4 : 16; }
constexpr int pk_tile_cols(int mode) { return pk_family(mode) == 1 ? PK_WAVES * 32 : PK_WAVES * 64; }
constexpr int pk_out_cols(int mode) {
    return (mode == 3 || mode == 6) ? 2 * pk_tile_cols(mode) : pk_tile_cols(mode);
}
constexpr int pk_epi_bytes(int mode) {
    return mode == 4 ? 32 * (3 * pk_tile_cols(mode) + 8) * 2 : PK_BM * (pk_out_cols(mode) + 8) * 2;
}
constexpr int pk_lds_bytes(int mode) {
    return PK_ST * PK_BM * PK_BK * 2 > pk_epi_bytes(mode) ? PK_ST * PK_BM * PK_BK * 2 : pk_epi_bytes(mode);
}

// Elements of one packed matrix with n rows (n_groups = ceil(n / 32) pairs of 16-row groups) and
// contraction k.
__host__ __device__ inline int64_t packed_elems(int64_t n_groups, int k) {
    return n_groups * ((k + 31) / 32) * 1024;
}


template <int MODE>
__global__ void __launch_bounds__(PK_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm_bf16_pk_kernel(GemmArgs p) {
    constexpr int BM = PK_BM, BK = PK_BK, IA = PK_IA;
    constexpr int A_BYTES = BM * BK * 2;
    constexpr int TC = pk_tile_cols(MODE);
    __shared__ __attribute__((aligned(1024))) uint8_t lds[pk_lds_bytes(MODE)];
    constexpr int FAM = pk_family(MODE);
    const int nt_r = static_cast<int>(ceil_div((FAM == 1 || MODE == 4) ? p.inter : p.d, TC));
    const int nt_s = (FAM == 1 || MODE == 4) ? static_cast<int>(ceil_div(p.shared_inter, TC)) : nt_r;
    Tile t;
    if (!decode_tile(p.work, p.off, p.E, p.T, BM, nt_r, nt_s, p.part, t, pk_group_m(MODE))) return;
    const bool shared = t.g == p.E;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();

    int K, n_out;
    const uint16_t* Abase;
    int64_t a_rows;
    const uint16_t* Bw;  // this wave's first packed group
    int b_groups;        // packed groups of this wave that hold weights (0..2)
    if constexpr (FAM == 1) {
        K = p.d;
        n_out = shared ? p.shared_inter : p.inter;
        Abase = static_cast<const uint16_t*>(p.x);
        a_rows = p.T;
        const int ng = 2 * static_cast<int>(ceil_div(n_out, 32));  // gate + up groups
        const uint16_t* W = shared ? static_cast<const uint16_t*>(p.ws13)
                                   : static_cast<const uint16_t*>(p.w13) + t.g * packed_elems(ng, K);
        const int q = t.nt * PK_WAVES + wave;  // output group of this wave
        b_groups = 2 * q < ng ? 2 : 0;
        Bw = W + packed_elems(b_groups ? 2 * q : 0, K);
    } else {
        const uint16_t* Wr;
        const uint16_t* Ws;
        if constexpr (MODE == 4) {  // dH = dout W2: rows of dout, contraction over d
            K = p.d;
            n_out = shared ? p.shared_inter : p.inter;
            Abase = static_cast<const uint16_t*>(p.dout);
            a_rows = p.T;
            Wr = static_cast<const uint16_t*>(p.w2t);
            Ws = static_cast<const uint16_t*>(p.ws2t);
        } else if constexpr (MODE == 5) {  // dX = [dA dB] W13: contraction over 2 inter
            K = 2 * (shared ? p.shared_inter : p.inter);
            n_out = p.d;
            // the group's k-packed rows (K columns: a multiple of 32)
            const int64_t kp0 = shared ? 0 : p.kp[t.g];
            a_rows = shared ? ceil_div(p.T, 16) * 16 : p.kp[t.g + 1] - kp0;
            Abase = (shared ? p.pt_dab_s : p.pt_dab_r) + kp0 * K;
            Wr = static_cast<const uint16_t*>(p.w13t);
            Ws = static_cast<const uint16_t*>(p.ws13t);
        } else {
            K = shared ? p.shared_inter : p.inter;
            n_out = p.d;
            Abase = shared ? static_cast<const uint16_t*>(p.h_s) : static_cast<const uint16_t*>(p.h_r);
            a_rows = shared ? p.T : p.T * p.k;
            Wr = static_cast<const uint16_t*>(p.w2);
            Ws = static_cast<const uint16_t*>(p.ws2);
        }
        const int ng = static_cast<int>(ceil_div(n_out, 32));
        const uint16_t* W = shared ? Ws : Wr + t.g * packed_elems(ng, K);
        const int g0 = t.nt * (2 * PK_WAVES) + 2 * wave;
        b_groups = ng - g0 >= 2 ? 2 : (ng - g0 > 0 ? ng - g0 : 0);
        Bw = W + packed_elems(b_groups ? g0 : 0, K);
    }
    K = uniform_int(K);
    const int kc_n = (K + 31) / 32;  // packed 32-wide contraction slices per 16-row group
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(uniform_ptr(Abase)), 0, uniform_int(static_cast<int>(a_rows * K * 2)), kBufferFlags);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(uniform_ptr(Bw)), 0, uniform_int(2 * b_groups * kc_n * 1024), kBufferFlags);

    // A DMA: instruction q of this wave fills LDS rows (wave * IA + q) * 8 .. + 7 of the stage;
    // lane moves the 16-byte chunk (lane % 8) ^ swizzle(row) of its row into slot lane % 8.
    // aoff: element offset of the row start; rows past the tile get 2^30, whose
    // byte offset (>= 2^31) is out of range: zero fill without memory traffic.
    // Mode 5: instruction q of wave w brings the k-packed block of 16-row slice 2 w + q / 2 and
    // 32-column group q % 2 of the stage, 1 KB; the two row halves' 16-byte chunks are XORed with
    // 0 and 4, so that a transposing read (below) spreads over the banks.
    const int a_ks = MODE == 5 ? uniform_int(static_cast<int>(a_rows / 16)) : 0;  // 16-row slices of the group
    const int a_ks0 = MODE == 5 ? uniform_int(static_cast<int>(t.row0 - (shared ? 0 : p.off[t.g])) / 16) : 0;
    int asrc[IA];
#pragma unroll
    for (int q = 0; q < IA; ++q) {
        const int R = (wave * IA + q) * 8 + lane / 8;
        const int rr = R < t.rows ? R : 0;
        if ((FAM == 1 || MODE == 4) && !shared) asrc[q] = p.perm_token[t.row0 + rr];
        else asrc[q] = static_cast<int>(t.row0 + rr);
    }
    // Weight fragments of stage s: b[j][h] is 16-row group h of K slice 32 (2 s + j).
    // Quarter q of a stage loads groups 2 (q % 2) and 2 (q % 2) + 1 of slice q / 2.
    auto issue_bq = [&](i32x4_t (&b)[2][4], int s, int q) {
        const int j = q >> 1;
        const int kc = s * 2 + j;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int h = 2 * (q & 1) + u;
            const int vo = (((h * kc_n + kc) * 64 + lane) * 16) | (kc < kc_n ? 0 : kOutOfRange);
            b[j][h] = __builtin_amdgcn_raw_buffer_load_b128(rsB, vo, 0, 0);
        }
    };
    // the first stage's weights come in while the row indices do (all of this after
    // them: 0.3 % of a layer of 4096 tokens, 0.6 % of one of 16384 x 4096)
    i32x4_t b0[2][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) issue_bq(b0, 0, q);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t aoff[IA];
    int achk[IA];
#pragma unroll
    for (int q = 0; q < IA; ++q) {
        const int R = (wave * IA + q) * 8 + lane / 8;
        aoff[q] = R < t.rows ? static_cast<uint32_t>(asrc[q]) * static_cast<uint32_t>(K) : (1u << 30);
        achk[q] = ((lane % 8) ^ ((R / 2) % 8)) * 8;
    }
    // One A DMA instruction (rows (wave * IA + q) * 8 ..) of stage s into ring slot `slot`.
    // (Mode 5 issues it as inline assembly: before a transposing read the compiler would wait for
    // every load in flight that it knows to write LDS: 966 -> 1542 us for the routed dX.)
    const i32x4_t rs5 = buf_rsrc(Abase, static_cast<int>(a_rows * K * 2));
    const uint32_t lds_base = lds_address(lds);
    auto issue_aq = [&](int slot, int s, int q) {
        if constexpr (MODE == 5) {
            const int cg = 2 * s + (q & 1), ks = a_ks0 + 2 * wave + (q >> 1);
            const int so = cg < kc_n && ks < a_ks ? (cg * a_ks + ks) * 1024 : kOutOfRange;
            const int vo = static_cast<int>(static_cast<uint32_t>(so) +
                                            static_cast<uint32_t>((lane ^ ((lane & 32) >> 3)) * 16));
            dma16(rs5, vo, lds_base + static_cast<uint32_t>(slot * A_BYTES + (wave * IA + q) * 1024));
        } else {
            const int k = s * BK + achk[q];
            const int vo = static_cast<int>(((aoff[q] + static_cast<uint32_t>(k)) * 2u) |
                                            (k < K ? 0u : static_cast<uint32_t>(kOutOfRange)));
            auto* dst = (__attribute__((address_space(3))) void*)(lds + slot * A_BYTES + (wave * IA + q) * 1024);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, dst, 16, vo, 0, 0, 0);
        }
    };
    // acc[i][h]: token rows 16 i .. 16 i + 15 x weight rows 16 h .. 16 h + 15 of this wave
    f32x4_t acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int h = 0; h < 4; ++h) acc[i][h] = f32x4_t{};
    const int quad = lane >> 4, l16 = lane & 15;
    // mode 5's transposing reads: lane j of a 16-lane group supplies the address of column 8 quad +
    // j / 4 (+ 4 in the second read: the chunk's bit 2), rows 4 (j % 4) .. and receives row j
    const int tr0 = ((((l16 & 3) >> 1) * 32 + 8 * quad + (l16 >> 2)) ^ (((l16 & 3) >> 1) * 4)) * 16 + (l16 & 1) * 8;

    // Stage s from ring slot `slot` with weight registers bc, while the loads of
    // the next stages go out between the MFMAs. A stage (K = 64) runs in four
    // quarters q: K slice j = q / 2 against token tiles 2 u + q % 2 (u < MT);
    // quarter q issues the weight loads of stage s + 1 for
    // quarter q (2 loads) and the A DMA q of stage s + 2, reads the token
    // fragments of quarter q + 1 and runs 4 MT MFMAs. A wave issues in order,
    // so spreading the memory instructions over the MFMAs keeps the matrix
    // pipe fed while the address unit drains them.
    static_assert(IA == 4, "one A DMA per quarter stage");
    // MT: 32-row sub-tiles that take part (1-4: a short last tile of an
    // expert skips the MFMAs and fragment reads of its empty sub-tiles).
    auto stage_run = [&](auto mt_c, int slot, int s, const i32x4_t (&bc)[2][4], i32x4_t (&bn)[2][4]) {
        constexpr int MT = decltype(mt_c)::value;
        const uint8_t* base = lds + slot * A_BYTES;
        const int nslot = slot == 0 ? 2 : slot - 1;  // (slot + 2) % 3
        bf16x8_t af[2][4];
        int tr = tr0;
        if constexpr (MODE == 5) asm volatile("" : "+v"(tr));  // rebuilt per stage: its sums would not fit the registers
        // token fragment of tile 2 u + q % 2, K slice q / 2: row 16 i + l % 16, k 32 j + 8 (l / 16) ..
        auto rd = [&](int q, bf16x8_t (&a)[4]) {
            const int c = (q >> 1) * 4 + quad;
#pragma unroll
            for (int u = 0; u < MT; ++u) {
                if constexpr (MODE == 5) {
                    const uint8_t* a0 = base + ((2 * u + (q & 1)) * 2 + (q >> 1)) * 1024;
                    const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(a0 + tr));
                    const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(a0 + (tr ^ 64)));
                    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                    a[u] = __builtin_bit_cast(bf16x8_t, make_uint4(l2.x, l2.y, h2.x, h2.y));
                } else {
                    const int R = (2 * u + (q & 1)) * 16 + l16;
                    a[u] = *reinterpret_cast<const bf16x8_t*>(base + R * (BK * 2) + ((c ^ ((R / 2) % 8)) * 16));
                }
            }
        };
        rd(0, af[0]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __builtin_amdgcn_sched_barrier(0);
            issue_bq(bn, s + 1, q);
            issue_aq(nslot, s + 2, q);
            if (q < 3) rd(q + 1, af[(q + 1) & 1]);
#pragma unroll
            for (int u = 0; u < MT; ++u)
#pragma unroll
                for (int h = 0; h < 4; ++h)  // transposed tile: rows = weight rows, columns = tokens
                    acc[2 * u + (q & 1)][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, bc[q >> 1][h]), af[q & 1][u], acc[2 * u + (q & 1)][h], 0, 0, 0);
            // order: one VMEM after each of the first MFMAs, then one LDS read after each of
            // the following MFMAs, then the rest of the MFMAs
            constexpr int NM = 4 * MT;
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                if (v < NM) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
#pragma unroll
            for (int v = 0; v < MT; ++v) {
                if (3 + v < NM) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, MODE == 5 ? 2 : 1, 0);
            }
            if (NM > 3 + MT) __builtin_amdgcn_sched_group_barrier(0x008, NM - 3 - MT, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Loads retire in order. Issue order: B(0), A(0), A(1), then per quarter q of
    // stage s - 1: B(s)[q] (2), A(s + 1)[q] (1). Before stage s reads LDS slot s % 3,
    // at most the 12 loads issued after A(s)'s last DMA may still fly (B(s)
    // and A(s + 1); A(1) alone before stage 0); the compiler waits for B(s)'s registers by itself. The
    // barrier makes every wave's DMA of A(s) visible and frees the slot that
    // A(s + 2) overwrites. Unrolled by two so the B register sets stay static.
    // Past the end of K the loads go out of range and return zeros, so every
    // stage issues the same count and the waits stay exact.
    const int nk = static_cast<int>(ceil_div(K, BK));
    auto barrier = [] {
        if constexpr (MODE == 5) dma_barrier();  // its loads are inline assembly
        else __builtin_amdgcn_s_barrier();
    };
    auto kloop = [&](auto mt_c) {
        i32x4_t b1[2][4];
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int q = 0; q < IA; ++q) issue_aq(st, st, q);
        wait_vm_lgkm0<IA>();
        int s = 0, slot = 0;
        for (; s + 2 <= nk; s += 2) {
            wait_vm_lgkm0<12>();
            barrier();
            stage_run(mt_c, slot, s, b0, b1);
            slot = slot == 2 ? 0 : slot + 1;
            wait_vm_lgkm0<12>();
            barrier();
            stage_run(mt_c, slot, s + 1, b1, b0);
            slot = slot == 2 ? 0 : slot + 1;
        }
        if (s < nk) {
            wait_vm_lgkm0<12>();
            barrier();
            stage_run(mt_c, slot, s, b0, b1);
        }
    };
    const int trows = uniform_int(t.rows);
    if (trows > 96) kloop(std::integral_constant<int, 4>{});
    else if (trows > 64) kloop(std::integral_constant<int, 3>{});
    else if (trows > 32) kloop(std::integral_constant<int, 2>{});
    else kloop(std::integral_constant<int, 1>{});
    wait_vm_lgkm0<0>();  // drain: the epilogue reuses the ring
    barrier();

    // Epilogue through LDS: [BM][TC + 8] bf16 tile, then 16-byte row chunks.
    // The accumulators hold transposed 16x16 tiles: element e of lane l of
    // acc[i][h] is output column 16 h + 4 (l / 16) + e of the wave's columns,
    // token row 16 i + l % 16, so each lane writes four adjacent columns as
    // one 8-byte store.
    auto pack4 = [](float a, float b, float c, float d) {
        return make_uint2(static_cast<uint32_t>(f32_to_bf16(a)) | (static_cast<uint32_t>(f32_to_bf16(b)) << 16),
                          static_cast<uint32_t>(f32_to_bf16(c)) | (static_cast<uint32_t>(f32_to_bf16(d)) << 16));
    };
    if constexpr (MODE == 4) {
        // dH = w * (dout W2) and the SwiGLU backward with the saved gate (a)
        // and up (b) pre-activations: dA = dH b silu'(a), dB = dH silu(a),
        // plus w H = w silu(a) b for the dW2 product (routed rows). In four
        // passes of 32 rows: the rows' a | b slices come into LDS as whole
        // rows, each lane turns its four adjacent columns into dA | dB | w H
        // in place, and the three go out (w H for routed rows only) k-packed for
        // the weight gradients and the dX GEMM: 16 rows x 32 columns per 1 KB, a
        // lane's eight rows of one column by two transposing LDS reads. (As
        // passes of their own three k-packs read the rows back: at 16384 tokens,
        // d 2048, 64 experts top-6 of 1408 and two shared ones 118 + 198 + 57 us;
        // [dA dB] stored as rows too, for the dX GEMM, 919 + 296 us for the routed
        // and the shared launch, without 812 + 260.)
        const uint16_t* AB = static_cast<const uint16_t*>(shared ? p.ab_s : p.ab_r);
        const int64_t kp0 = shared ? 0 : p.kp[t.g];
        const int64_t Ks = shared ? ceil_div(p.T, 16) : (p.kp[t.g + 1] - kp0) / 16;
        const int64_t ks0 = (t.row0 - (shared ? 0 : p.off[t.g])) / 16;  // the tile's first 16-row slice of its group
        uint16_t* PD = (shared ? p.pt_dab_s : p.pt_dab_r) + kp0 * (2 * n_out);  // 2 n_out is a multiple of 32
        uint16_t* PH = shared ? nullptr : p.pt_wh_r + kp0 * (32 * ceil_div(n_out, 32));
        const int64_t ld = 2 * static_cast<int64_t>(n_out);
        constexpr int EP = 3 * TC + 8;  // LDS row: a | b | w H (pitch = 4 mod 64 dwords)
        uint16_t* el = reinterpret_cast<uint16_t*>(lds);
        const int col0 = t.nt * TC;
        const int ncols = n_out - col0 < TC ? n_out - col0 : TC;  // multiple of 16
        // 16-byte chunks of a pass's a | b rows held by each thread; the next
        // pass's chunks are loaded while the current one is processed
        constexpr int LCH = 32 * (2 * TC / 8) / PK_THREADS;
        auto load_pass = [&](int i, uint4 (&v)[LCH]) {
            const int rows_here = t.rows - i * 32;
            const int64_t rbase = t.row0 + i * 32;
#pragma unroll
            for (int u = 0; u < LCH; ++u) {
                const int q = threadIdx.x + u * PK_THREADS;
                const int r = q / (2 * TC / 8), ch = q % (2 * TC / 8);
                const int part = ch / (TC / 8), c = (ch % (TC / 8)) * 8;
                v[u] = (r < rows_here && c < ncols)
                           ? *reinterpret_cast<const uint4*>(AB + (rbase + r) * ld + part * n_out + col0 + c)
                           : make_uint4(0, 0, 0, 0);
            }
        };
        uint4 cur[LCH], nxt[LCH];
        load_pass(0, cur);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rows_here = t.rows - i * 32;
            if (rows_here <= 0) break;  // uniform
            const int64_t rbase = t.row0 + i * 32;
#pragma unroll
            for (int u = 0; u < LCH; ++u) {
                const int q = threadIdx.x + u * PK_THREADS;
                const int r = q / (2 * TC / 8), ch = q % (2 * TC / 8);
                *reinterpret_cast<uint4*>(el + r * EP + (ch / (TC / 8)) * TC + (ch % (TC / 8)) * 8) = cur[u];
            }
            if (i + 1 < 4) load_pass(i + 1, nxt);
            __syncthreads();
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const int lr = 16 * tt + l16;  // row of the pass
                const bool in = lr < rows_here;
                const float w = shared ? 1.0f : (in ? p.wrow[rbase + lr] : 0.0f);
                uint16_t* er = el + lr * EP;
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int col = wave * 64 + 16 * h + 4 * quad;
                    const uint2 av = *reinterpret_cast<const uint2*>(er + col);
                    const uint2 bv = *reinterpret_cast<const uint2*>(er + TC + col);
                    const float a[4] = {__uint_as_float(av.x << 16), __uint_as_float(av.x & 0xffff0000u),
                                        __uint_as_float(av.y << 16), __uint_as_float(av.y & 0xffff0000u)};
                    const float bb[4] = {__uint_as_float(bv.x << 16), __uint_as_float(bv.x & 0xffff0000u),
                                         __uint_as_float(bv.y << 16), __uint_as_float(bv.y & 0xffff0000u)};
                    float da[4], db[4], wh[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float dh = in ? w * acc[2 * i + tt][h][e] : 0.0f;
                        const float sg = 1.0f / (1.0f + __expf(-a[e]));
                        const float sa = a[e] * sg;  // silu(a)
                        da[e] = dh * bb[e] * (sg + sa * (1.0f - sg));
                        db[e] = dh * sa;
                        wh[e] = w * sa * bb[e];
                    }
                    *reinterpret_cast<uint2*>(er + col) = pack4(da[0], da[1], da[2], da[3]);
                    *reinterpret_cast<uint2*>(er + TC + col) = pack4(db[0], db[1], db[2], db[3]);
                    *reinterpret_cast<uint2*>(er + 2 * TC + col) = pack4(wh[0], wh[1], wh[2], wh[3]);
                }
            }
            __syncthreads();
            // k-packed: lane l takes column 32 f + l % 32 of the wave's 64 and rows 8 (l / 32) .. + 7
            // of slice tt; in each 16-lane group lane j supplies the address of row j / 4, columns
            // 4 (j % 4) .. and receives column j of four rows. Rows past the group are zero here (a
            // and b, and dh by choice: beside an infinite weight their accumulators are NaN), as
            // the padding has to be.
            const int tr0 = (8 * (lane >> 5) + ((lane & 15) >> 2)) * EP + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                if (16 * tt >= rows_here) break;  // uniform
#pragma unroll
                for (int part = 0; part < 3; ++part) {
                    if (part == 2 && shared) break;
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        const int c = wave * 64 + 32 * f;
                        const uint16_t* src = el + tr0 + 16 * tt * EP + part * TC + c;
                        const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)src);
                        const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(src + 4 * EP));
                        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                        const int cl = c + (lane & 31);
                        if (cl < ncols) {
                            const int cc = (part == 1 ? n_out : 0) + col0 + cl;  // column of [dA dB] or of w H
                            uint16_t* P = part < 2 ? PD : PH;
                            *reinterpret_cast<uint4*>(P + ((cc >> 5) * Ks + ks0 + 2 * i + tt) * 512 +
                                                      ((lane >> 5) * 32 + (cc & 31)) * 8) =
                                make_uint4(l2.x, l2.y, h2.x, h2.y);
                        }
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < LCH; ++u) cur[u] = nxt[u];
        }
        return;
    }
    // OK: 1 H = silu(gate) * up, 3 the gate | up pre-activations, 2 / 5 the
    // plain accumulators. Mode 6 writes H, then the pre-activations.
    auto epilogue = [&](auto ok_c) {
        constexpr int OK = decltype(ok_c)::value;
        constexpr int OC = OK == 3 ? 2 * TC : TC;  // tile columns written (3: gate block then up block)
        constexpr int OP = OC + 8;
        uint16_t* otile = reinterpret_cast<uint16_t*>(lds);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int r = i * 16 + l16;
            const int c0 = 4 * quad;
            if constexpr (OK == 1) {  // groups 2 p (gate) and 2 p + 1 (up): H columns 16 p ..
#pragma unroll
                for (int pq = 0; pq < 2; ++pq) {
                    float h[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) h[e] = silu(acc[i][2 * pq][e]) * acc[i][2 * pq + 1][e];
                    *reinterpret_cast<uint2*>(otile + r * OP + wave * 32 + 16 * pq + c0) = pack4(h[0], h[1], h[2], h[3]);
                }
            } else if constexpr (OK == 3) {  // gate block, then up block
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    *reinterpret_cast<uint2*>(otile + r * OP + (h & 1) * TC + wave * 32 + 16 * (h >> 1) + c0) =
                        pack4(acc[i][h][0], acc[i][h][1], acc[i][h][2], acc[i][h][3]);
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    *reinterpret_cast<uint2*>(otile + r * OP + wave * 64 + 16 * h + c0) =
                        pack4(acc[i][h][0], acc[i][h][1], acc[i][h][2], acc[i][h][3]);
            }
        }
        __syncthreads();
        if constexpr (OK == 7) {
            // out_j = sum_s w_js Y_r[inv(j, s)] + Ys_j for the tile's tokens and
            // columns, in the combine kernel's order (float32, slots in order,
            // then the bf16 shared row from the tile): two 8-column items per
            // thread at a time, their row indices, then four row loads each
            const int kk = p.k;
            const int32_t* inv = p.inv;
            const float* tw = p.topk_w;
            const uint16_t* yr = static_cast<const uint16_t*>(p.y_r);
            uint16_t* out = static_cast<uint16_t*>(p.out);
            const int64_t dd = p.d;
            constexpr int CH = OC / 8;
            const int col0 = t.nt * TC;
            for (int q0 = threadIdx.x; q0 < BM * CH; q0 += 2 * PK_THREADS) {
                int64_t j[2];
                int c[2], r[2];
                bool ok[2];
                float v[2][8];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int q = q0 + u * PK_THREADS;
                    r[u] = q / CH;
                    c[u] = col0 + (q % CH) * 8;
                    j[u] = t.row0 + r[u];
                    ok[u] = q < BM * CH && r[u] < t.rows && c[u] < n_out;  // d % 8 == 0
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[u][e] = 0.0f;
                }
                for (int s0 = 0; s0 < kk; s0 += 4) {
                    int row[2][4];
                    float wt[2][4];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int sv = 0; sv < 4; ++sv) {
                            const bool in = ok[u] && s0 + sv < kk;
                            row[u][sv] = in ? inv[j[u] * kk + s0 + sv] : -1;
                            wt[u][sv] = in ? tw[j[u] * kk + s0 + sv] : 0.0f;
                        }
                    uint4 y[2][4];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int sv = 0; sv < 4; ++sv)
                            y[u][sv] = row[u][sv] >= 0
                                           ? *reinterpret_cast<const uint4*>(yr + static_cast<int64_t>(row[u][sv]) * dd + c[u])
                                           : make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int sv = 0; sv < 4; ++sv) {
                            if (s0 + sv >= kk) continue;
                            const uint32_t w4[4] = {y[u][sv].x, y[u][sv].y, y[u][sv].z, y[u][sv].w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                v[u][2 * e] = fmaf(wt[u][sv], __uint_as_float(w4[e] << 16), v[u][2 * e]);
                                v[u][2 * e + 1] = fmaf(wt[u][sv], __uint_as_float(w4[e] & 0xffff0000u), v[u][2 * e + 1]);
                            }
                        }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (!ok[u]) continue;
                    const uint4 ys = *reinterpret_cast<const uint4*>(otile + r[u] * OP + (c[u] - col0));
                    const uint32_t w4[4] = {ys.x, ys.y, ys.z, ys.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[u][2 * e] += __uint_as_float(w4[e] << 16);
                        v[u][2 * e + 1] += __uint_as_float(w4[e] & 0xffff0000u);
                    }
                    *reinterpret_cast<uint4*>(out + j[u] * dd + c[u]) =
                        make_uint4(static_cast<uint32_t>(f32_to_bf16(v[u][0])) | (static_cast<uint32_t>(f32_to_bf16(v[u][1])) << 16),
                                   static_cast<uint32_t>(f32_to_bf16(v[u][2])) | (static_cast<uint32_t>(f32_to_bf16(v[u][3])) << 16),
                                   static_cast<uint32_t>(f32_to_bf16(v[u][4])) | (static_cast<uint32_t>(f32_to_bf16(v[u][5])) << 16),
                                   static_cast<uint32_t>(f32_to_bf16(v[u][6])) | (static_cast<uint32_t>(f32_to_bf16(v[u][7])) << 16));
                }
            }
            return;
        }
        uint16_t* O;
        if constexpr (OK == 1) O = shared ? static_cast<uint16_t*>(p.h_s) : static_cast<uint16_t*>(p.h_r);
        else if constexpr (OK == 3) O = shared ? static_cast<uint16_t*>(p.ab_s) : static_cast<uint16_t*>(p.ab_r);
        else if constexpr (OK == 5) O = shared ? static_cast<uint16_t*>(p.dx_s) : static_cast<uint16_t*>(p.dx_r);
        else O = shared ? static_cast<uint16_t*>(p.y_s) : static_cast<uint16_t*>(p.y_r);
        constexpr int CH = OC / 8;
        const int col0 = t.nt * TC;
        for (int q = threadIdx.x; q < BM * CH; q += PK_THREADS) {
            const int r = q / CH, ch = q % CH;
            if constexpr (OK == 3) {  // gate block to columns [0, n_out), up block to [n_out, 2 n_out)
                const int part = (ch * 8) / TC;
                const int c = col0 + ch * 8 - part * TC;
                if (r < t.rows && c < n_out)
                    *reinterpret_cast<uint4*>(O + (t.row0 + r) * (2 * static_cast<int64_t>(n_out)) + part * n_out +
                                              c) = *reinterpret_cast<const uint4*>(otile + r * OP + ch * 8);
            } else {
                const int c = col0 + ch * 8;
                if (r < t.rows && c < n_out)  // n_out % 8 == 0: a chunk is all in or all out
                    *reinterpret_cast<uint4*>(O + (t.row0 + r) * n_out + c) =
                        *reinterpret_cast<const uint4*>(otile + r * OP + ch * 8);
            }
        }
    };
    if constexpr (MODE == 6) {
        epilogue(std::integral_constant<int, 1>{});
        __syncthreads();  // every H row chunk has left the tile
        epilogue(std::integral_constant<int, 3>{});
    } else {
        epilogue(std::integral_constant<int, MODE>{});
    }
}

// Pack `batch` row-major matrices into the fragment order above; k % 8 == 0.
// interleave: the source has 2 * n rows (gate rows then up rows) and 16-row
// group 4q + 2v + h takes rows 32q + 16v.. of half h; otherwise the source has
// n rows. One block per 16-row group and kPackCols columns: whole row pieces of 1
// KB come in, and the fragments go out of LDS, 1 KB each. (One thread per
// fragment, 64 bytes of each of 16 rows per wave load: 278 us for 64 gate / up
// matrices of 2816 x 2048, now 246, 6 TB/s.)
constexpr int kPackCols = 512;
typedef uint32_t pack_src4_t __attribute__((ext_vector_type(4), aligned(2)));  // the source may start at any element
constexpr int64_t kPackBlocks = 1 << 22;  // a launch holds fewer than 2^32 threads
__global__ void __launch_bounds__(256)
pack_rows_kernel(const uint16_t* __restrict__ src, unsigned items, int n, int k, int interleave,
                 uint16_t* __restrict__ dst) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[16][kPackCols + 8];  // row pitch = 4 mod 64 dwords
    const int ng = (interleave ? 4 : 2) * ((n + 31) / 32);  // 16-row groups
    const int kc_n = (k + 31) / 32;
    const int nc = (k + kPackCols - 1) / kPackCols;
    for (unsigned item = blockIdx.x; item < items; item += gridDim.x) {  // one each below kPackBlocks
        const unsigned bg = item / nc;  // (matrix, group)
        const int c0 = static_cast<int>(item % nc) * kPackCols;
        const int64_t b = bg / ng;
        const int g = static_cast<int>(bg % ng);
        const int wave = threadIdx.x / kWave, lane = lane_id();
        const int64_t src_rows = interleave ? 2 * static_cast<int64_t>(n) : n;
        const int r0 = interleave ? (g / 4) * 32 + ((g / 2) % 2) * 16 : g * 16;  // of the half
        const int base = interleave ? (g % 2) * n : 0;
        const int col = c0 + lane * 8;
        pack_src4_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = r0 + wave * 4 + i;
            v[i] = r < n && col < k
                       ? *reinterpret_cast<const pack_src4_t*>(src + (b * src_rows + base + r) * k + col)
                       : pack_src4_t{};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<uint4*>(&tile[wave * 4 + i][lane * 8]) = make_uint4(v[i].x, v[i].y, v[i].z, v[i].w);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPackCols / 32 / 4; ++i) {
            const int c = wave * (kPackCols / 32 / 4) + i;  // 32-column slice of the block
            if (c0 / 32 + c >= kc_n) break;
            *reinterpret_cast<uint4*>(dst + ((static_cast<int64_t>(bg) * kc_n + c0 / 32 + c) * 64 + lane) * 8) =
                *reinterpret_cast<const uint4*>(&tile[lane % 16][32 * c + 8 * (lane / 16)]);
        }
        __syncthreads();  // the tile is read before the next item is written
    }
}

// The same for matrices stored [k][n] (the packed matrix is the transpose), not
// interleaved; n % 8 == 0. One block per 32-row slice and kPackCols source
// columns: 1 KB row pieces come in, a fragment is two transposing LDS reads of
// four rows of 16 columns per 16 lanes. (One thread per fragment, eight 2-byte
// loads down a column: 502 us for the 64 matrices of 2816 x 2048 above, now
// 246.)
__global__ void __launch_bounds__(256)
pack_cols_kernel(const uint16_t* __restrict__ src, unsigned items, int n, int k, uint16_t* __restrict__ dst) {
    constexpr int P = kPackCols + 16;  // row pitch = 8 mod 64 dwords
    __shared__ __attribute__((aligned(16))) uint16_t tile[32 * P];
    const int ng = 2 * ((n + 31) / 32);  // 16-column groups
    const int kc_n = (k + 31) / 32;
    const int nc = (n + kPackCols - 1) / kPackCols;
    const int wave = threadIdx.x / kWave, lane = lane_id();
    for (unsigned item = blockIdx.x; item < items; item += gridDim.x) {  // one each below kPackBlocks
        const int c = static_cast<int>(item % kc_n);  // slice
        const int64_t b = item / kc_n / nc;
        const int n0 = static_cast<int>(item / kc_n % nc) * kPackCols;
        const int col = n0 + lane * 8;
        pack_src4_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int kk = c * 32 + wave * 8 + i;
            v[i] = kk < k && col < n ? *reinterpret_cast<const pack_src4_t*>(src + (b * k + kk) * n + col) : pack_src4_t{};
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *reinterpret_cast<uint4*>(tile + (wave * 8 + i) * P + lane * 8) = make_uint4(v[i].x, v[i].y, v[i].z, v[i].w);
        __syncthreads();
        // lane j of a 16-lane group supplies the address of row j / 4, columns 4 (j % 4) .. and
        // receives column j of four rows: rows 8 (lane / 16) .. + 3, then + 4 .. + 7
        const uint16_t* t0 = tile + (8 * (lane >> 4) + ((lane & 15) >> 2)) * P + 4 * (lane & 3);
#pragma unroll
        for (int i = 0; i < kPackCols / 16 / 4; ++i) {
            const int f = wave * (kPackCols / 16 / 4) + i, g = n0 / 16 + f;
            if (g >= ng) break;  // uniform
            const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(t0 + 16 * f));
            const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(t0 + 16 * f + 4 * P));
            const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
            *reinterpret_cast<uint4*>(dst + (((b * ng + g) * kc_n + c) * 64 + lane) * 8) =
                make_uint4(l2.x, l2.y, h2.x, h2.y);
        }
        __syncthreads();  // the tile is read before the next item is written
    }
}

// ============================================================== row-major matrix tiles
//
// Float32 layers (forward and backward) and the backward of bf16 layers whose
// weights are row-major. Products and sums are float32: float32 operands run
// on v_mfma_f32_32x32x2_f32. A bf16 layer runs on v_mfma_f32_32x32x16_bf16: its
// own tensors (x, dout, the weights) are exact bf16 operands, and a float32
// intermediate (dA dB, w H) enters as three bf16 terms cut off its mantissa (8
// bits each: their sum is the float32 value), so every product is exact and
// only the float32 accumulation rounds, as on the vector ALUs. (The matrix cores
// take bf16 operands below 2^-126 for zero: a value loses its third term below
// about 2^-110, an absolute error under 2^-125.) Steps:
//   RM_FW1  H = silu(X W1^T) * (X W3^T)          rows: routed rows (x gathered) / tokens
//   RM_FW2  Y = H W2^T
//   GB_AB   [A | B] = X W13^T
//   GB_DH   dH = w dout W2, then the SwiGLU backward: dA, dB and w H
//   GB_DX   dX = [dA dB] W13
//   GB_DW2  dW2[n][c]  = sum over the group's rows of dout[tok][n] (w H)[c]
//   GB_DW13 dW13[m][n] = sum over the group's rows of [dA dB][m] x[tok][n]
// Row steps take their tiles from the work table (decode_tile); weight steps
// run one block per (output tile, group), group E the shared experts. An
// expert without rows gets a zero gradient.
//
// Tiles: 64 indices of the F operand (the one that may be float32 in a bf16
// layer) x 64 or 128 of the H operand, 4 waves of 32 x 32 NH. A K step is eight
// 16-byte chunks per index (64 bf16 or 32 float32): each thread loads its
// chunks of both operands into registers one step ahead, turns an operand
// whose memory runs along the index into chunks along K, and writes them to
// LDS: in a float32 layer to the other of two buffers, one barrier per step; in
// a bf16 layer to the only one, two barriers, because its tiles are short (an
// expert's 250 rows are four steps of the weight gradients) and four blocks per
// CU hide their start and end where two cannot. In a float32 layer the matrix cores bound a tile (64
// cycles per 4096 flops), and 64 x 64 gives small layers enough tiles; in a
// bf16 layer the LDS reads do (four fragments per three products at 64 x 64,
// five per six at 64 x 128, hence NH = 2).
// Against float32 vector-ALU tiles (64 x 64, K steps of 16): at 1000 tokens x
// 1024, 16 experts of 512, top-4, one shared, row-major bf16, GB_AB / DH / DX /
// DW2 / DW13 343 / 177 / 264 / 151 / 228 -> 26 / 34 / 50 / 53 / 77 us; the
// forward of the 512 x 256 float32 layer with 8 experts of 512, top-2, 44 + 58
// -> 17 + 15 us.
enum { GB_AB = 0, GB_DH = 1, GB_DX = 2, GB_DW2 = 3, GB_DW13 = 4, RM_FW1 = 5, RM_FW2 = 6 };

struct RmArgs {
    int64_t T;
    int d, E, inter, shared_inter, part;
    const int32_t* off;
    const int32_t* perm_token;
    const int32_t* work;
    const void* x;     // [T][d] layer dtype
    const void* dout;  // [T][d]
    const void* w13;   // [E][2 inter][d]
    const void* w2;    // [E][d][inter]
    const void* ws13;  // [2 shared_inter][d]
    const void* ws2;   // [d][shared_inter]
    float* h_r;        // [R][inter] (RM_FW1 writes, RM_FW2 reads)
    float* h_s;        // [T][shared_inter]
    float* y_r;        // [R][d]
    float* y_s;        // [T][d]
    float* ab_r;       // [R][2 inter]
    float* ab_s;       // [T][2 shared_inter]
    float* dab_r;
    float* dab_s;
    float* wh_r;       // [R][inter]
    float* wh_s;       // [T][shared_inter]
    float* dx_r;       // [R][d]
    float* dx_s;       // [T][d]
    const float* wrow; // [R]
    void* dw13;        // layer dtype, shapes of w13 ...
    void* dw2;
    void* dws13;
    void* dws2;
};

// H indices per tile: 128 for bf16 operands, 64 for float32
__host__ __device__ constexpr int rm_nh(bool bf16) { return bf16 ? 2 : 1; }

// output column tiles of a row step for a group with n_out inner columns
__host__ __device__ __forceinline__ int rm_row_tiles(int mode, int n_out, int d, bool bf16) {
    if (mode == RM_FW1) return static_cast<int>(ceil_div(n_out, 32));  // 32 gate + 32 up rows
    return static_cast<int>(ceil_div(mode == GB_AB ? 2 * n_out : mode == GB_DH ? n_out : d, 64 * rm_nh(bf16)));
}

// vector loads at the alignment of one element (rows start at multiples of 8
// elements, the tensors themselves wherever the caller put them)
template <bool B16>
struct RmVec {
    typedef uint32_t v1 __attribute__((aligned(4)));
    typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(4)));
    typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct RmVec<true> {
    typedef uint32_t v1 __attribute__((aligned(2)));
    typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(2)));
    typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(2)));
};
template <bool B16, int N>
__device__ __forceinline__ void rm_load_words(const void* p, uint32_t (&w)[N]) {
    if constexpr (N == 1) {
        w[0] = *static_cast<const typename RmVec<B16>::v1*>(p);
    } else if constexpr (N == 2) {
        const auto v = *static_cast<const typename RmVec<B16>::v2*>(p);
        w[0] = v.x;
        w[1] = v.y;
    } else {
        static_assert(N % 4 == 0, "whole 16-byte loads");
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            const auto v = static_cast<const typename RmVec<B16>::v4*>(p)[i];
            w[4 * i] = v.x;
            w[4 * i + 1] = v.y;
            w[4 * i + 2] = v.z;
            w[4 * i + 3] = v.w;
        }
    }
}

// One operand's share of a thread: NC chunks of CK elements along K.
//   SRC16: bf16 in memory (else float32). KC: memory runs along K (row pointers
//   fixed, K moves), else along the index (CK rows of NC adjacent indices).
//   P: bf16 terms a float32 element is cut into (0: it stays float32).
template <bool SRC16, bool KC, int NC, int CK, int P>
struct RmOperand {
    static constexpr int OUTER = KC ? NC : CK;                       // separately addressed pieces
    static constexpr int WORDS = (KC ? CK : NC) * (SRC16 ? 2 : 4) / 4;  // 32-bit words of a piece
    static constexpr int PLANES = SRC16 || P == 0 ? 1 : P;
    uint32_t raw[OUTER][WORDS];

    static __device__ __forceinline__ int lds_row(int u) {
        return KC ? static_cast<int>(threadIdx.x >> 3) + 32 * u : NC * static_cast<int>(threadIdx.x & 31) + u;
    }
    static __device__ __forceinline__ int lds_chunk() { return KC ? threadIdx.x & 7 : threadIdx.x >> 5; }

    // zero the elements whose K index (this thread's chunk starts at kk) is past K
    __device__ __forceinline__ void cut(int kk, int K) {
#pragma unroll
        for (int o = 0; o < OUTER; ++o)
#pragma unroll
            for (int w = 0; w < WORDS; ++w)
                if ((KC ? kk : kk + o) >= K) raw[o][w] = 0;  // K % 8 == 0 where memory runs along it
    }
    // chunks of plane q of plane_bytes each, row pitch 128 bytes, swizzled
    __device__ __forceinline__ void put(uint8_t* base, int plane_bytes) const {
        const int c = lds_chunk();
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int R = lds_row(u);
            uint8_t* dst = base + R * 128 + ((c ^ (((R >> 1) ^ (R >> 4)) & 7)) * 16);
            if constexpr (SRC16) {
                uint32_t o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (KC) o[i] = raw[u][i];
                    else o[i] = __builtin_amdgcn_perm(raw[2 * i + 1][u / 2], raw[2 * i][u / 2], u & 1 ? 0x07060302 : 0x05040100);
                }
                *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
            } else if constexpr (P == 0) {
                uint32_t o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = KC ? raw[u][i] : raw[i][u];
                *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
            } else {
                // hi = the upper 16 bits, then the same of the exact remainders; an
                // infinity keeps its first term alone
                uint32_t o[3][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t t0[2], t1[2], t2[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int e = 2 * i + h;
                        const uint32_t v = KC ? raw[u][e] : raw[e][u];
                        t0[h] = v;
                        float r = __uint_as_float(v) - __uint_as_float(v & 0xffff0000u);
                        r = (v & 0x7fffffffu) == 0x7f800000u ? 0.0f : r;
                        t1[h] = __float_as_uint(r);
                        t2[h] = __float_as_uint(r - __uint_as_float(t1[h] & 0xffff0000u));
                    }
                    o[0][i] = __builtin_amdgcn_perm(t0[1], t0[0], 0x07060302);
                    o[1][i] = __builtin_amdgcn_perm(t1[1], t1[0], 0x07060302);
                    o[2][i] = __builtin_amdgcn_perm(t2[1], t2[0], 0x07060302);
                }
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uint4*>(dst + q * plane_bytes) = make_uint4(o[q][0], o[q][1], o[q][2], o[q][3]);
            }
        }
    }
};

// eight bf16 with the infinities and NaN replaced by zero
__device__ __forceinline__ uint4 rm_finite(uint4 h) {
    auto keep = [](uint32_t w) {
        const uint32_t hi = (w & 0x7f800000u) == 0x7f800000u ? 0u : 0xffff0000u;
        const uint32_t lo = (w & 0x7f80u) == 0x7f80u ? 0u : 0xffffu;
        return w & (hi | lo);
    };
    return make_uint4(keep(h.x), keep(h.y), keep(h.z), keep(h.w));
}

template <int MODE, bool BF16>
__global__ void __launch_bounds__(kThreads, BF16 ? 4 : 2)
gemm_rm_kernel(RmArgs p) {
    constexpr bool kRows = MODE != GB_DW2 && MODE != GB_DW13;
    constexpr bool kFwd = MODE == RM_FW1 || MODE == RM_FW2;
    constexpr int NH = rm_nh(BF16), BH = 64 * NH;
    constexpr int CK = BF16 ? 8 : 4, KS = 8 * CK, ES = BF16 ? 2 : 4;
    // F: rows of x / dout / H (along K), [dA dB] (rows: along K; weight steps: along the index), w H
    constexpr bool kF16 = BF16 && (MODE == GB_AB || MODE == GB_DH);
    constexpr bool kHkc = MODE == GB_AB || kFwd;  // H: W13 / W2 rows along K, else along the index
    using OpF = RmOperand<kF16, kRows, 2, CK, BF16 ? 3 : 0>;
    using OpH = RmOperand<BF16, kHkc, 2 * NH, CK, 0>;
    constexpr int F_BYTES = 64 * 128, H_BYTES = BH * 128;
    constexpr int BUF = OpF::PLANES * F_BYTES + H_BYTES;
    constexpr int NB = BF16 ? 1 : 2;  // LDS buffers
    __shared__ __attribute__((aligned(1024))) uint8_t lds[NB][BUF];

    const int tid = threadIdx.x;
    int g, f0, h0, NF, N, K;
    int64_t row0;
    if constexpr (kRows) {
        Tile t;
        if (!decode_tile(p.work, p.off, p.E, p.T, 64, rm_row_tiles(MODE, p.inter, p.d, BF16),
                         rm_row_tiles(MODE, p.shared_inter, p.d, BF16), p.part, t))
            return;
        g = t.g;
        row0 = t.row0;
        const int n = g == p.E ? p.shared_inter : p.inter;
        f0 = 0;
        NF = t.rows;
        h0 = t.nt * (MODE == RM_FW1 ? 32 : BH);
        N = MODE == GB_AB ? 2 * n : (MODE == GB_DH || MODE == RM_FW1) ? n : p.d;
        K = MODE == GB_DX ? 2 * n : MODE == RM_FW2 ? n : p.d;
    } else {
        g = blockIdx.y;
        const int n = g == p.E ? p.shared_inter : p.inter;
        NF = MODE == GB_DW2 ? n : 2 * n;
        N = p.d;
        const int th = static_cast<int>(ceil_div(N, BH));
        if (static_cast<int>(blockIdx.x) >= static_cast<int>(ceil_div(NF, 64)) * th) return;
        f0 = static_cast<int>(blockIdx.x) / th * 64;
        h0 = static_cast<int>(blockIdx.x) % th * BH;
        row0 = g == p.E ? 0 : p.off[g];
        K = g == p.E ? static_cast<int>(p.T) : p.off[g + 1] - p.off[g];
    }
    const bool shared = g == p.E;
    const int n_out = shared ? p.shared_inter : p.inter;
    const int ldab = 2 * n_out;
    const char* W13 = shared ? static_cast<const char*>(p.ws13)
                             : static_cast<const char*>(p.w13) + ES * static_cast<int64_t>(g) * 2 * p.inter * p.d;
    const char* W2 = shared ? static_cast<const char*>(p.ws2)
                            : static_cast<const char*>(p.w2) + ES * static_cast<int64_t>(g) * p.d * p.inter;
    float* ab = shared ? p.ab_s : p.ab_r;
    float* dab = shared ? p.dab_s : p.dab_r;
    float* wh = shared ? p.wh_s : p.wh_r;

    // Indices past the tile read index 0 (their outputs are not written), K
    // past its end reads K index 0 and is zeroed, so every load is in bounds.
    constexpr int EF = kF16 ? 2 : 4;
    const char* fp[OpF::OUTER];  // kRows: the row of each chunk; else fp[0]: this thread's columns of row row0
    if constexpr (kRows) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = OpF::lds_row(u) < NF ? OpF::lds_row(u) : 0;
            if constexpr (MODE == GB_DX) fp[u] = reinterpret_cast<const char*>(dab + (row0 + r) * ldab);
            else if constexpr (MODE == RM_FW2)
                fp[u] = reinterpret_cast<const char*>((shared ? p.h_s : p.h_r) + (row0 + r) * n_out);
            else {
                const int64_t tok = shared ? row0 + r : p.perm_token[row0 + r];
                fp[u] = static_cast<const char*>(MODE == GB_DH ? p.dout : p.x) + EF * tok * p.d;
            }
        }
    } else {
        const int i = f0 + 2 * (tid & 31) < NF ? f0 + 2 * (tid & 31) : f0;
        fp[0] = reinterpret_cast<const char*>(MODE == GB_DW2 ? wh + row0 * n_out + i : dab + row0 * ldab + i);
    }
    const char* hp[OpH::OUTER];  // kHkc: the weight row of each chunk; else hp[0]: this thread's columns of row 0
    if constexpr (kHkc) {
#pragma unroll
        for (int u = 0; u < 2 * NH; ++u) {
            const int R = OpH::lds_row(u);
            int64_t wr;
            if constexpr (MODE == RM_FW1) {  // 32 gate rows, then the matching up rows
                const int c = h0 + (R & 31) < N ? h0 + (R & 31) : 0;
                wr = R < 32 ? c : n_out + c;
            } else {
                wr = h0 + R < N ? h0 + R : 0;
            }
            hp[u] = MODE == RM_FW2 ? W2 + ES * wr * n_out : W13 + ES * wr * p.d;
        }
    } else {
        const int i = h0 + 2 * NH * (tid & 31) < N ? h0 + 2 * NH * (tid & 31) : h0;
        const char* b = MODE == GB_DH ? W2 : MODE == GB_DX ? W13 : static_cast<const char*>(MODE == GB_DW2 ? p.dout : p.x);
        hp[0] = b + ES * static_cast<int64_t>(i);
    }
    const int64_t f_ld = 4 * static_cast<int64_t>(MODE == GB_DW2 ? n_out : ldab);
    const int64_t h_ld = ES * static_cast<int64_t>(MODE == GB_DH ? n_out : p.d);

    const int nk = static_cast<int>(ceil_div(K, KS));
    // tokens of this thread's K rows of one step (weight steps: dout / x rows), loaded a step ahead
    int tok[CK];
    auto load_tok = [&](int s) {
        if constexpr (!kRows) {
#pragma unroll
            for (int e = 0; e < CK; ++e) {
                int kk = s * KS + OpH::lds_chunk() * CK + e;
                kk = kk < K ? kk : 0;
                tok[e] = shared ? kk : p.perm_token[row0 + kk];
            }
        }
    };
    auto load = [&](OpF& opf, OpH& oph, int s) {
        const int kf = s * KS + OpF::lds_chunk() * CK, kh = s * KS + OpH::lds_chunk() * CK;
        if constexpr (kRows) {
#pragma unroll
            for (int u = 0; u < 2; ++u) rm_load_words<kF16>(fp[u] + EF * (kf < K ? kf : 0), opf.raw[u]);
        } else {
#pragma unroll
            for (int e = 0; e < CK; ++e) rm_load_words<kF16>(fp[0] + f_ld * (kf + e < K ? kf + e : 0), opf.raw[e]);
        }
        if constexpr (kHkc) {
#pragma unroll
            for (int u = 0; u < 2 * NH; ++u) rm_load_words<BF16>(hp[u] + ES * (kh < K ? kh : 0), oph.raw[u]);
        } else {
#pragma unroll
            for (int e = 0; e < CK; ++e) {
                const int64_t r = kRows ? (kh + e < K ? kh + e : 0) : tok[e];
                rm_load_words<BF16>(hp[0] + h_ld * r, oph.raw[e]);
            }
        }
    };
    auto store = [&](OpF& opf, OpH& oph, int s) {
        if ((s + 1) * KS > K) {
            opf.cut(s * KS + OpF::lds_chunk() * CK, K);
            oph.cut(s * KS + OpH::lds_chunk() * CK, K);
        }
        uint8_t* b = lds[s % NB];
        opf.put(b, F_BYTES);
        oph.put(b + OpF::PLANES * F_BYTES, H_BYTES);
    };

    const int wave = tid / kWave, lane = lane_id();
    const int wf = wave >> 1, wh_ = wave & 1, half = lane >> 5, l32 = lane & 31;
    // acc[j]: 32 F indices (rows; GB_DW2: columns) x 32 H indices
    f32x16_t acc[NH];
#pragma unroll
    for (int j = 0; j < NH; ++j) acc[j] = f32x16_t{};
    // again_c: H's infinities (and NaN) meet only the first of F's three terms
    auto compute = [&](int s, auto again_c) {
        const uint8_t* b = lds[s % NB];
        auto frag = [&](const uint8_t* base, int R, int c) {
            return *reinterpret_cast<const uint4*>(base + R * 128 + ((c ^ (((R >> 1) ^ (R >> 4)) & 7)) * 16));
        };
        if constexpr (decltype(again_c)::value) {
#pragma unroll 1
            for (int e = 0; e < 4 * 3; ++e) {
                const int q = 2 - e % 3, c = 2 * (e / 3) + half;
                const bf16x8_t fv = __builtin_bit_cast(bf16x8_t, frag(b + q * F_BYTES, 32 * wf + l32, c));
#pragma unroll
                for (int j = 0; j < NH; ++j) {
                    const uint4 h = frag(b + 3 * F_BYTES, 32 * (NH * wh_ + j) + l32, c);
                    const bf16x8_t hv = __builtin_bit_cast(bf16x8_t, q > 0 ? rm_finite(h) : h);
                    acc[j] = MODE == GB_DW2 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(hv, fv, acc[j], 0, 0, 0)
                                            : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv, hv, acc[j], 0, 0, 0);
                }
            }
            return;
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c = 2 * ks + half;
            uint4 f[OpF::PLANES], h[NH];
#pragma unroll
            for (int q = 0; q < OpF::PLANES; ++q) f[q] = frag(b + q * F_BYTES, 32 * wf + l32, c);
#pragma unroll
            for (int j = 0; j < NH; ++j) h[j] = frag(b + OpF::PLANES * F_BYTES, 32 * (NH * wh_ + j) + l32, c);
            if constexpr (BF16) {
#pragma unroll
                for (int q = OpF::PLANES - 1; q >= 0; --q)  // smallest terms first
#pragma unroll
                    for (int j = 0; j < NH; ++j) {
                        const bf16x8_t fv = __builtin_bit_cast(bf16x8_t, f[q]), hv = __builtin_bit_cast(bf16x8_t, h[j]);
                        acc[j] = MODE == GB_DW2 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(hv, fv, acc[j], 0, 0, 0)
                                                : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv, hv, acc[j], 0, 0, 0);
                    }
            } else {
                const f32x4_t fv = __builtin_bit_cast(f32x4_t, f[0]), hv = __builtin_bit_cast(f32x4_t, h[0]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[0] = MODE == GB_DW2 ? __builtin_amdgcn_mfma_f32_32x32x2f32(hv[e], fv[e], acc[0], 0, 0, 0)
                                            : __builtin_amdgcn_mfma_f32_32x32x2f32(fv[e], hv[e], acc[0], 0, 0, 0);
            }
        }
    };
    auto kloop = [&](auto again_c) {
        // PD steps of operands are in registers or in flight: a float32 step is
        // 1024 cycles of matrix work, less than the latency of its loads, so there
        // the loads run two steps ahead of the step that is written to LDS (17.3 ->
        // 16.5 and 15.7 -> 15.0 us for the forward above); in a bf16 layer the
        // registers for that cost the fourth block per CU (GB_DW2 / DW13 53 / 77
        // -> 58 / 85 us)
        constexpr int PD = BF16 ? 1 : 2;
        OpF opf[PD];
        OpH oph[PD];
        load_tok(0);
        load(opf[0], oph[0], 0);
        load_tok(1);
        if constexpr (PD == 2) {
            if (nk > 1) load(opf[1], oph[1], 1);
            load_tok(2);
        }
        store(opf[0], oph[0], 0);
        if (nk > PD) load(opf[0], oph[0], PD);
        load_tok(PD + 1);
        __syncthreads();
        // step s; r: the registers that hold step s + 1
        auto step = [&](int s, OpF& rf, OpH& rh) {
            if constexpr (NB == 2) {
                // the buffer written here was last read before the barrier that ended step s - 1
                if (s + 1 < nk) store(rf, rh, s + 1);
                if (s + 1 + PD < nk) {
                    load(rf, rh, s + 1 + PD);
                    load_tok(s + 2 + PD);
                }
                compute(s, again_c);
            } else {
                compute(s, again_c);
                if (s + 1 < nk) {
                    __syncthreads();  // every wave is done reading step s
                    store(rf, rh, s + 1);
                    if (s + 1 + PD < nk) {
                        load(rf, rh, s + 1 + PD);
                        load_tok(s + 2 + PD);
                    }
                }
            }
            __syncthreads();
        };
        for (int s = 0; s < nk; s += PD) {
            step(s, opf[PD - 1], oph[PD - 1]);
            if constexpr (PD == 2) {
                if (s + 1 < nk) step(s + 1, opf[0], oph[0]);
            }
        }
    };
    if (nk > 0) kloop(std::false_type{});
    if constexpr (OpF::PLANES == 3) {
        // A term of F that is exactly zero (the lower ones of any value that is itself a bf16,
        // and of one in fifty others) times an infinity of H is NaN, where the float32 product is
        // that infinity. Such a tile is multiplied once more; every other one only looks at its sums.
        bool nan = false;
#pragma unroll
        for (int j = 0; j < NH; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) nan |= acc[j][v] != acc[j][v];
        uint32_t* vote = reinterpret_cast<uint32_t*>(lds);  // every wave is done with the last step
        if (lane == 0) vote[wave] = 0;
        if (nan) vote[wave] = 1;
        __syncthreads();
        nan = (vote[0] | vote[1] | vote[2] | vote[3]) != 0;
        __syncthreads();
        if (nan) {
#pragma unroll
            for (int j = 0; j < NH; ++j) acc[j] = f32x16_t{};
            kloop(std::true_type{});
        }
    }

    // element v of a 32 x 32 tile: row 8 (v / 4) + 4 half + v % 4, column l32
    if constexpr (MODE == RM_FW1) {
        // gate and up sit in different waves: through LDS, then whole rows of 32 columns
        float* C = reinterpret_cast<float*>(lds);
        static_assert(64 * 65 * 4 <= NB * BUF, "the output tile fits the operand buffers");
#pragma unroll
        for (int v = 0; v < 16; ++v)
            C[(32 * wf + 8 * (v >> 2) + 4 * half + (v & 3)) * 65 + 32 * wh_ + l32] = acc[0][v];
        __syncthreads();
        float* H = shared ? p.h_s : p.h_r;
        for (int q = tid; q < 64 * 32; q += kThreads) {
            const int r = q / 32, c = q % 32, col = h0 + c;
            if (r < NF && col < N) H[(row0 + r) * n_out + col] = silu(C[r * 65 + c]) * C[r * 65 + 32 + c];
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NH; ++j) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int tr = 8 * (v >> 2) + 4 * half + (v & 3);
            const float a = acc[j][v];
            if constexpr (MODE == GB_DW2) {
                const int n = h0 + 32 * (NH * wh_ + j) + tr, c = f0 + 32 * wf + l32;
                if (n >= N || c >= NF) continue;
                const int64_t e = (shared ? 0 : static_cast<int64_t>(g) * p.d * p.inter) + static_cast<int64_t>(n) * NF + c;
                void* out = shared ? p.dws2 : p.dw2;
                if constexpr (BF16) static_cast<uint16_t*>(out)[e] = f32_to_bf16(a);
                else static_cast<float*>(out)[e] = a;
            } else {
                const int rr = f0 + 32 * wf + tr, col = h0 + 32 * (NH * wh_ + j) + l32;
                if (rr >= NF || col >= N) continue;
                if constexpr (MODE == GB_AB) {
                    ab[(row0 + rr) * ldab + col] = a;
                } else if constexpr (MODE == GB_DH) {
                    // SwiGLU backward of h = silu(a) b with dh = w (dout W2)
                    const int64_t r = row0 + rr;
                    const float w = shared ? 1.0f : p.wrow[r];
                    const float dh = w * a;
                    const float av = ab[r * ldab + col], bv = ab[r * ldab + n_out + col];
                    const float sg = 1.0f / (1.0f + expf(-av));
                    const float sa = av * sg;
                    dab[r * ldab + col] = dh * bv * sg * (1.0f + av * (1.0f - sg));
                    dab[r * ldab + n_out + col] = dh * sa;
                    wh[r * n_out + col] = w * sa * bv;
                } else if constexpr (MODE == GB_DX || MODE == RM_FW2) {
                    float* o = MODE == GB_DX ? (shared ? p.dx_s : p.dx_r) : (shared ? p.y_s : p.y_r);
                    o[(row0 + rr) * p.d + col] = a;
                } else {
                    const int64_t e = (shared ? 0 : static_cast<int64_t>(g) * 2 * p.inter * p.d) + static_cast<int64_t>(rr) * N + col;
                    void* out = shared ? p.dws13 : p.dw13;
                    if constexpr (BF16) static_cast<uint16_t*>(out)[e] = f32_to_bf16(a);
                    else static_cast<float*>(out)[e] = a;
                }
            }
        }
    }
}

// ============================================================== combine

template <bool BF16>
__global__ void combine_kernel(int64_t T, int d, int k, const int32_t* __restrict__ inv,
                               const float* __restrict__ topk_w, const void* __restrict__ y_r,
                               const void* __restrict__ y_s, void* __restrict__ out) {
    const int per_row = d / 8;
    const int64_t n = T * per_row;
    for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int64_t j = i / per_row;
        const int c = static_cast<int>(i % per_row) * 8;
        float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int s = 0; s < k; ++s) {
            const float w = topk_w[j * k + s];
            float v[8];
            load8<BF16>(y_r, static_cast<int64_t>(inv[j * k + s]) * d + c, v);
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = fmaf(w, v[q], acc[q]);
        }
        if (y_s != nullptr) {
            float v[8];
            load8<BF16>(y_s, j * d + c, v);
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] += v[q];
        }
        if constexpr (BF16) {
            uint4 o;
            o.x = static_cast<uint32_t>(f32_to_bf16(acc[0])) | (static_cast<uint32_t>(f32_to_bf16(acc[1])) << 16);
            o.y = static_cast<uint32_t>(f32_to_bf16(acc[2])) | (static_cast<uint32_t>(f32_to_bf16(acc[3])) << 16);
            o.z = static_cast<uint32_t>(f32_to_bf16(acc[4])) | (static_cast<uint32_t>(f32_to_bf16(acc[5])) << 16);
            o.w = static_cast<uint32_t>(f32_to_bf16(acc[6])) | (static_cast<uint32_t>(f32_to_bf16(acc[7])) << 16);
            *reinterpret_cast<uint4*>(static_cast<uint16_t*>(out) + j * d + c) = o;
        } else {
            float4* o = reinterpret_cast<float4*>(static_cast<float*>(out) + j * d + c);
            o[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
            o[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
        }
    }
}

GemmArgs make_args(const ExpertArgs& a, const ExpWs& w, const int32_t* work, int part) {
    GemmArgs g;
    g.part = part;
    g.T = a.T;
    g.d = a.d;
    g.E = a.E;
    g.k = a.k;
    g.inter = a.inter;
    g.shared_inter = a.shared_inter;
    g.x = a.x;
    g.w13 = a.w13;
    g.w2 = a.w2;
    g.ws13 = a.ws13;
    g.ws2 = a.ws2;
    g.off = a.expert_offsets;
    g.perm_token = a.perm_token;
    g.work = work;
    g.h_r = w.h_r;
    g.h_s = w.h_s;
    g.y_r = w.y_r;
    g.y_s = w.y_s;
    g.dout = nullptr;
    g.w2t = g.ws2t = g.w13t = g.ws13t = nullptr;
    g.ab_r = a.ab_r;
    g.ab_s = a.ab_s;
    g.dx_r = g.dx_s = nullptr;
    g.wrow = nullptr;
    g.pt_dab_r = g.pt_dab_s = g.pt_wh_r = nullptr;
    g.kp = nullptr;
    g.inv = a.perm_inv;
    g.topk_w = a.topk_w;
    g.out = a.out;
    return g;
}

// the forward of a float32 layer
RmArgs rm_fwd_args(const GemmArgs& a) {
    RmArgs r{};
    r.T = a.T;
    r.d = a.d;
    r.E = a.E;
    r.inter = a.inter;
    r.shared_inter = a.shared_inter;
    r.part = a.part;
    r.off = a.off;
    r.perm_token = a.perm_token;
    r.work = a.work;
    r.x = a.x;
    r.w13 = a.w13;
    r.w2 = a.w2;
    r.ws13 = a.ws13;
    r.ws2 = a.ws2;
    r.h_r = static_cast<float*>(a.h_r);
    r.h_s = static_cast<float*>(a.h_s);
    r.y_r = static_cast<float*>(a.y_r);
    r.y_s = static_cast<float*>(a.y_s);
    return r;
}

// Grid size: 8 XCD ranges, each at most a bound on the routed items over 8
// plus the shared items over 8 (host side; the exact split is made on the device).
int64_t work_bound(int64_t T, int k, int E, int bm, int nt_r, int nt_s, bool has_shared, int part) {
    const int64_t R = T * k;
    const int64_t routed = part == 2 ? 0 : (ceil_div(R, bm) + E) * nt_r;
    const int64_t shared = (has_shared && part != 1) ? ceil_div(T, bm) * nt_s : 0;
    return 8 * (ceil_div(routed, 8) + ceil_div(shared, 8));
}

struct Plan {
    int bm, bm2, nt1_r, nt1_s, nt2;
    bool has_shared;
};

Plan plan_of(const ExpertArgs& a) {
    Plan p;
    const bool bf16 = a.act_dtype == 1;
    const bool pk = bf16 && a.packed;
    p.bm = pk ? PK_BM : bf16 ? DCfg::BM : FBM;
    p.bm2 = p.bm;
    const int tn1 = pk ? pk_tile_cols(1) : bf16 ? tile_cols<DCfg>(1) : 32;  // H columns per GEMM1 tile
    const int tn2 = pk ? pk_tile_cols(2) : bf16 ? tile_cols<DCfg>(2) : 64;  // output columns per GEMM2 tile
    p.nt1_r = static_cast<int>(ceil_div(a.inter, tn1));
    p.nt1_s = static_cast<int>(ceil_div(a.shared_inter, tn1));
    p.nt2 = static_cast<int>(ceil_div(a.d, tn2));
    p.has_shared = a.shared_inter > 0;
    return p;
}

}  // namespace

size_t experts_workspace_bytes(int64_t T, int d, int E, int k, int inter, int shared_inter,
                               int act_dtype) {
    const int64_t R = T * k;
    const size_t s = esz(act_dtype);
    return align_up(s * R * inter, 256) + align_up(s * T * shared_inter, 256) +
           align_up(s * R * d, 256) + align_up(s * T * d, 256) +
           2 * align_up(sizeof(int32_t) * (E + 2), 256);
}

WorkTables experts_work_tables(const ExpertArgs& a, void* ws) {
    ExpWs w = carve(ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    const Plan p = plan_of(a);
    WorkTables t;
    t.work1 = w.work1;
    t.work2 = w.work2;
    t.bm = p.bm;  // both GEMMs use the same tile height
    t.nt1_r = p.nt1_r;
    t.nt1_s = p.nt1_s;
    t.nt2 = p.nt2;
    t.has_shared = p.has_shared ? 1 : 0;
    return t;
}

hipError_t launch_experts_gemm1(const ExpertArgs& a, void* ws, int part, hipStream_t stream) {
    ExpWs w = carve(ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    const Plan p = plan_of(a);
    const GemmArgs g = make_args(a, w, w.work1, part);
    const dim3 grid(static_cast<unsigned>(work_bound(a.T, a.k, a.E, p.bm, p.nt1_r, p.nt1_s, p.has_shared, part)));
    if (grid.x == 0) return hipSuccess;
    if (a.act_dtype == 1 && a.packed && a.ab_r != nullptr)
        hipLaunchKernelGGL(gemm_bf16_pk_kernel<6>, grid, dim3(PK_THREADS), 0, stream, g);
    else if (a.act_dtype == 1 && a.packed)
        hipLaunchKernelGGL(gemm_bf16_pk_kernel<1>, grid, dim3(PK_THREADS), 0, stream, g);
    else if (a.act_dtype == 1)
        hipLaunchKernelGGL((gemm_bf16_dma_kernel<1, DCfg>), grid, dim3(DCfg::THREADS), 0, stream, g);
    else
        hipLaunchKernelGGL((gemm_rm_kernel<RM_FW1, false>), grid, dim3(kThreads), 0, stream, rm_fwd_args(g));
    return hipGetLastError();
}

int64_t experts_shared_down_tiles(int64_t T, int d) { return ceil_div(T, PK_BM) * ceil_div(d, pk_tile_cols(7)); }

hipError_t launch_experts_gemm2_combine(const ExpertArgs& a, void* ws, hipStream_t stream) {
    if (!(a.act_dtype == 1 && a.packed && a.shared_inter > 0)) return hipErrorInvalidValue;
    ExpWs w = carve(ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    const Plan p = plan_of(a);
    const GemmArgs g = make_args(a, w, w.work2, 2);
    const dim3 grid(static_cast<unsigned>(work_bound(a.T, a.k, a.E, p.bm2, p.nt2, p.nt2, p.has_shared, 2)));
    if (grid.x == 0) return hipSuccess;
    hipLaunchKernelGGL(gemm_bf16_pk_kernel<7>, grid, dim3(PK_THREADS), 0, stream, g);
    return hipGetLastError();
}

hipError_t launch_experts_gemm2(const ExpertArgs& a, void* ws, int part, hipStream_t stream) {
    ExpWs w = carve(ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    const Plan p = plan_of(a);
    const GemmArgs g = make_args(a, w, w.work2, part);
    const dim3 grid(static_cast<unsigned>(work_bound(a.T, a.k, a.E, p.bm2, p.nt2, p.nt2, p.has_shared, part)));
    if (grid.x == 0) return hipSuccess;
    if (a.act_dtype == 1 && a.packed)
        hipLaunchKernelGGL(gemm_bf16_pk_kernel<2>, grid, dim3(PK_THREADS), 0, stream, g);
    else if (a.act_dtype == 1)
        hipLaunchKernelGGL((gemm_bf16_dma_kernel<2, DCfg>), grid, dim3(DCfg::THREADS), 0, stream, g);
    else
        hipLaunchKernelGGL((gemm_rm_kernel<RM_FW2, false>), grid, dim3(kThreads), 0, stream, rm_fwd_args(g));
    return hipGetLastError();
}

// ---------------------------------------------------------------- backward (modes 3-5)

// Work table of one tiling (bm rows x nt column tiles per routed expert, then
// the shared items): one block of 256 threads, thread g counts expert g's items
// and an LDS scan forms the prefix sums (E <= 256).
__global__ void __launch_bounds__(256)
bwd_work_kernel(const int32_t* __restrict__ off, int E, int64_t T, int bm, int nt_r, int nt_s, int has_shared,
                int32_t* __restrict__ work) {
    __shared__ int32_t sc[256];
    const int g = threadIdx.x;
    sc[g] = g < E ? static_cast<int32_t>(ceil_div(off[g + 1] - off[g], bm)) * nt_r : 0;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {  // inclusive scan
        const int32_t v = g >= o ? sc[g - o] : 0;
        __syncthreads();
        sc[g] += v;
        __syncthreads();
    }
    if (g == 0) work[0] = 0;
    if (g < E) work[g + 1] = sc[g];
    if (g == 0) work[E + 1] = sc[E - 1] + (has_shared ? static_cast<int32_t>(ceil_div(T, bm)) * nt_s : 0);
}

// The three row steps' tables of the row-major backward (same tiles of FBM
// rows, nt column tiles of the step): table i at work + i (E + 2).
struct RmTables {
    int nt_r[3], nt_s[3];
};
__global__ void __launch_bounds__(256)
rm_work_kernel(const int32_t* __restrict__ off, int E, int64_t T, int has_shared, RmTables t, int32_t* __restrict__ work) {
    __shared__ int32_t sc[4];
    const int g = threadIdx.x, lane = lane_id(), wave = g / kWave;
    int v = g < E ? static_cast<int>(ceil_div(off[g + 1] - off[g], FBM)) : 0;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {  // inclusive scan: the wave, then the waves before
        const int u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    if (lane == kWave - 1) sc[wave] = v;
    __syncthreads();
    for (int w = 0; w < wave; ++w) v += sc[w];
    const int shared = has_shared ? static_cast<int>(ceil_div(T, FBM)) : 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        int32_t* w = work + i * (E + 2);
        if (g == 0) w[0] = 0;
        if (g < E) w[g + 1] = v * t.nt_r[i];
        if (g == E - 1) w[E + 1] = v * t.nt_r[i] + shared * t.nt_s[i];
    }
}

hipError_t launch_generic_bwd_tables(const ExpertArgs& a, int32_t* work, hipStream_t stream) {
    RmTables t;
    const bool bf16 = a.act_dtype == 1;
    for (int i = 0; i < 3; ++i) {
        t.nt_r[i] = rm_row_tiles(GB_AB + i, a.inter, a.d, bf16);
        t.nt_s[i] = rm_row_tiles(GB_AB + i, a.shared_inter, a.d, bf16);
    }
    hipLaunchKernelGGL(rm_work_kernel, dim3(1), dim3(256), 0, stream, a.expert_offsets, a.E, a.T,
                       a.shared_inter > 0 ? 1 : 0, t, work);
    return hipGetLastError();
}

ExpertFwdBuffers experts_fwd_buffers(const ExpertArgs& a, void* ws) {
    const ExpWs w = carve(ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    ExpertFwdBuffers b;
    b.h_r = w.h_r;
    b.h_s = w.h_s;
    b.y_r = w.y_r;
    b.y_s = w.y_s;
    b.work1 = w.work1;
    b.work2 = w.work2;
    return b;
}

hipError_t launch_bwd_gemm(int mode, const ExpertArgs& a, void* fwd_ws, const BwdGemmPtrs& bp, int part,
                           hipStream_t stream) {
    const ExpWs w = carve(fwd_ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    const bool has_shared = a.shared_inter > 0;
    int nt_r, nt_s;
    const int32_t* work;
    if (mode == 3) {
        nt_r = static_cast<int>(ceil_div(a.inter, pk_tile_cols(3)));
        nt_s = static_cast<int>(ceil_div(a.shared_inter, pk_tile_cols(3)));
        work = w.work1;  // the forward GEMM1's table: same tiling
    } else if (mode == 4) {
        nt_r = static_cast<int>(ceil_div(a.inter, pk_tile_cols(4)));
        nt_s = static_cast<int>(ceil_div(a.shared_inter, pk_tile_cols(4)));
        work = bp.work4;
        if (part != 2) {
            hipLaunchKernelGGL(bwd_work_kernel, dim3(1), dim3(256), 0, stream, a.expert_offsets, a.E, a.T, PK_BM, nt_r,
                               nt_s, has_shared ? 1 : 0, bp.work4);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    } else {
        nt_r = nt_s = static_cast<int>(ceil_div(a.d, pk_tile_cols(5)));
        work = w.work2;  // the forward GEMM2's table: same tiling
    }
    GemmArgs g = make_args(a, w, work, part);
    g.dout = bp.dout;
    g.w2t = bp.w2t;
    g.ws2t = bp.ws2t;
    g.w13t = bp.w13t;
    g.ws13t = bp.ws13t;
    g.ab_r = bp.ab_r;
    g.ab_s = bp.ab_s;
    g.dx_r = bp.dx_r;
    g.dx_s = bp.dx_s;
    g.wrow = bp.wrow;
    g.pt_dab_r = static_cast<uint16_t*>(bp.pt_dab_r);
    g.pt_dab_s = static_cast<uint16_t*>(bp.pt_dab_s);
    g.pt_wh_r = static_cast<uint16_t*>(bp.pt_wh_r);
    g.kp = bp.kp;
    const dim3 grid(static_cast<unsigned>(work_bound(a.T, a.k, a.E, PK_BM, nt_r, nt_s, has_shared, part)));
    if (grid.x == 0) return hipSuccess;
    if (mode == 3) hipLaunchKernelGGL(gemm_bf16_pk_kernel<3>, grid, dim3(PK_THREADS), 0, stream, g);
    else if (mode == 4) hipLaunchKernelGGL(gemm_bf16_pk_kernel<4>, grid, dim3(PK_THREADS), 0, stream, g);
    else hipLaunchKernelGGL(gemm_bf16_pk_kernel<5>, grid, dim3(PK_THREADS), 0, stream, g);
    return hipGetLastError();
}

hipError_t launch_generic_bwd(int step, const ExpertArgs& a, const GenericBwdPtrs& bp, hipStream_t stream) {
    RmArgs g{};
    g.T = a.T;
    g.d = a.d;
    g.E = a.E;
    g.inter = a.inter;
    g.shared_inter = a.shared_inter;
    g.off = a.expert_offsets;
    g.perm_token = a.perm_token;
    g.work = bp.work;
    g.x = a.x;
    g.dout = bp.dout;
    g.w13 = a.w13;
    g.w2 = a.w2;
    g.ws13 = a.ws13;
    g.ws2 = a.ws2;
    g.ab_r = bp.ab_r;
    g.ab_s = bp.ab_s;
    g.dab_r = bp.dab_r;
    g.dab_s = bp.dab_s;
    g.wh_r = bp.wh_r;
    g.wh_s = bp.wh_s;
    g.dx_r = bp.dx_r;
    g.dx_s = bp.dx_s;
    g.wrow = bp.wrow;
    g.dw13 = bp.dw13;
    g.dw2 = bp.dw2;
    g.dws13 = bp.dws13;
    g.dws2 = bp.dws2;
    const bool bf16 = a.act_dtype == 1;
    const bool has_shared = a.shared_inter > 0;
    dim3 grid;
    if (step <= GB_DX) {
        const int nt_r = rm_row_tiles(step, a.inter, a.d, bf16), nt_s = rm_row_tiles(step, a.shared_inter, a.d, bf16);
        g.work = bp.work + step * (a.E + 2);
        grid = dim3(static_cast<unsigned>(work_bound(a.T, a.k, a.E, FBM, nt_r, nt_s, has_shared, 0)));
    } else {
        auto tiles = [&](int n_out) {
            return ceil_div(step == GB_DW2 ? n_out : 2 * n_out, 64) * ceil_div(a.d, 64 * rm_nh(bf16));
        };
        const int64_t t_r = tiles(a.inter), t_s = has_shared ? tiles(a.shared_inter) : 0;
        grid = dim3(static_cast<unsigned>(t_r > t_s ? t_r : t_s), static_cast<unsigned>(a.E + (has_shared ? 1 : 0)));
    }
    if (grid.x == 0) return hipSuccess;
#define SMOES_GB(M)                                                                                    \
    do {                                                                                               \
        if (bf16) hipLaunchKernelGGL((gemm_rm_kernel<M, true>), grid, dim3(kThreads), 0, stream, g);  \
        else hipLaunchKernelGGL((gemm_rm_kernel<M, false>), grid, dim3(kThreads), 0, stream, g);      \
    } while (0)
    switch (step) {
        case GB_AB: SMOES_GB(GB_AB); break;
        case GB_DH: SMOES_GB(GB_DH); break;
        case GB_DX: SMOES_GB(GB_DX); break;
        case GB_DW2: SMOES_GB(GB_DW2); break;
        case GB_DW13: SMOES_GB(GB_DW13); break;
        default: return hipErrorInvalidValue;
    }
#undef SMOES_GB
    return hipGetLastError();
}

int64_t packed_weight_elems(int batch, int n, int k, int interleave) {
    const int64_t ng = interleave ? 2 * ceil_div(n, 32) : ceil_div(n, 32);
    return batch * packed_elems(ng, k);
}

hipError_t launch_pack_weights(const void* src, int batch, int n, int k, int interleave, int transpose, void* dst,
                               hipStream_t stream) {
    const int64_t frags = packed_weight_elems(batch, n, k, interleave) / 8;
    if (frags == 0) return hipSuccess;
    const int64_t items = transpose ? static_cast<int64_t>(batch) * ((k + 31) / 32) * ceil_div(n, kPackCols)
                                    : batch * (interleave ? 4 : 2) * ceil_div(n, 32) * ceil_div(k, kPackCols);
    const unsigned blocks = static_cast<unsigned>(items < kPackBlocks ? items : kPackBlocks);
    if (transpose)
        hipLaunchKernelGGL(pack_cols_kernel, dim3(blocks), dim3(256), 0, stream, static_cast<const uint16_t*>(src),
                           static_cast<unsigned>(items), n, k, static_cast<uint16_t*>(dst));
    else
        hipLaunchKernelGGL(pack_rows_kernel, dim3(blocks), dim3(256), 0, stream, static_cast<const uint16_t*>(src),
                           static_cast<unsigned>(items), n, k, interleave, static_cast<uint16_t*>(dst));
    return hipGetLastError();
}

hipError_t launch_experts_combine(const ExpertArgs& a, void* ws, hipStream_t stream) {
    ExpWs w = carve(ws, a.T, a.d, a.k, a.inter, a.shared_inter, a.act_dtype, a.E);
    const int64_t n = a.T * (a.d / 8);
    const unsigned blocks = static_cast<unsigned>(ceil_div(n, 256) < 16384 ? ceil_div(n, 256) : 16384);
    const void* ys = a.shared_inter > 0 ? w.y_s : nullptr;
    if (a.act_dtype == 1)
        hipLaunchKernelGGL(combine_kernel<true>, dim3(blocks), dim3(256), 0, stream, a.T, a.d, a.k,
                           a.perm_inv, a.topk_w, w.y_r, ys, a.out);
    else
        hipLaunchKernelGGL(combine_kernel<false>, dim3(blocks), dim3(256), 0, stream, a.T, a.d, a.k,
                           a.perm_inv, a.topk_w, w.y_r, ys, a.out);
    return hipGetLastError();
}

}  // namespace smoes
