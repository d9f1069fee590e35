// Expert weight gradients of the layer backward: for each group g (a routed
// expert over its expert-contiguous rows, or the merged shared expert over
// all tokens)
//   dW_g[m][n] = sum_r A[ra(r)][m] * B[r][n]
// where the rows of A go through a row map (the permutation's token of a
// routed row) or are the tokens: dW2 = dout^T (w H) with A = dout, dW13 =
// [dA dB]^T X with A = x (and the output transposed). B is k-packed: in the
// matrix cores' fragment order with the contraction (the group's rows)
// contiguous, as the dH GEMM writes w H and [dA dB]; the shared experts' H is
// packed here.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace smoes {

namespace {

// ============================================================ k-packed weight gradients
//
// k-packed, for a row-major S with C columns and a group of rows [r0, r1):
//   P[cg][ks][l][e] = S[r0 + 16 ks + 8 (l / 32) + e][32 cg + l % 32],
// zero past the group's rows; the groups follow each other, each
// padded to a multiple of 16 rows (kp: the padded row prefix). A fragment is
// one 1 KB block: lane l's 16 bytes are an MFMA operand as they are.
// wgrad_pk_kernel runs the forward's packed tiling: 128 (m) x 256 (n)
// tiles, the row-major m operand brought to LDS by buffer-to-LDS loads through
// a three-stage ring of K = 64 slices and read with transposing LDS reads, the
// n operand loaded straight into registers one slice ahead.

constexpr int KP_COLS = 256;  // source columns per k-pack block (8 column groups)

// Padded row prefix of the routed groups: kp[g + 1] = kp[g] + 16 ceil(rows_g / 16).
// a weight-gradient tile's fixed cost in 16-row slices: its start and its output
constexpr int kWpTileCost = 8;

__global__ void __launch_bounds__(256)
kpad_offsets_kernel(const int32_t* __restrict__ off, int E, int32_t* __restrict__ kp, int per0, int per1,
                    int32_t* __restrict__ ranges) {
    __shared__ int32_t sc[256];
    const int g = threadIdx.x;
    const int32_t rows = g < E ? ((off[g + 1] - off[g] + 15) / 16) * 16 : 0;
    sc[g] = rows;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {  // inclusive scan
        const int32_t v = g >= o ? sc[g - o] : 0;
        __syncthreads();
        sc[g] += v;
        __syncthreads();
    }
    if (g == 0) kp[0] = 0;
    if (g < E) kp[g + 1] = sc[g];
    if (ranges == nullptr || g >= E) return;
    // Tile ranges of the 8 XCDs with equal work for the two weight-gradient
    // launches (per0 and per1 tiles per group): a tile of group g costs its
    // 16-row slices plus kWpTileCost for its start and its output, and range
    // x starts at the first tile whose work ends after x / 8 of the total.
    // The group holding a boundary writes it.
    const int64_t w = rows / 16 + kWpTileCost;
    const int64_t pre = (sc[g] - rows) / 16 + static_cast<int64_t>(kWpTileCost) * g;  // work before g, per tile
    const int64_t all = sc[E - 1] / 16 + static_cast<int64_t>(kWpTileCost) * E;
    for (int h = 0; h < 2; ++h) {
        const int64_t per = h == 0 ? per0 : per1;
        int32_t* rg = ranges + 9 * h;
        if (g == 0) {
            rg[0] = 0;
            rg[8] = static_cast<int32_t>(per * E);
        }
        for (int x = 1; x < 8; ++x) {
            const int64_t target = per * all * x / 8;
            if (per * pre <= target && target < per * (pre + w)) {
                const int64_t o = (target - per * pre + w - 1) / w;
                rg[x] = static_cast<int32_t>(per * g + (o < per ? o : per));
            }
        }
    }
}

// One block per (16-row slice, 256 source columns) of one group of T rows: the
// slice's rows come into LDS as rows, and each lane writes one fragment lane (8
// consecutive rows of one column) as 16 bytes.
__global__ void __launch_bounds__(256)
kpack_kernel(const uint16_t* __restrict__ S, int C, int64_t T, uint16_t* __restrict__ P) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[16][KP_COLS + 8];
    const int64_t ks = blockIdx.x, Ks = ceil_div(T, 16);
    const int CG = static_cast<int>(ceil_div(C, 32));
    const int c0 = blockIdx.y * KP_COLS;
    for (int q = threadIdx.x; q < 16 * (KP_COLS / 8); q += blockDim.x) {
        const int rr = q / (KP_COLS / 8), ch = q % (KP_COLS / 8);
        const int64_t r = 16 * ks + rr;
        const int c = c0 + ch * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r < T && c < C)  // C % 8 == 0: a chunk is all in or all out
            v = *reinterpret_cast<const uint4*>(S + r * C + c);
        *reinterpret_cast<uint4*>(&tile[rr][ch * 8]) = v;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < (KP_COLS / 32) * 64; q += blockDim.x) {
        const int f = q / 64, l = q % 64;
        const int cg = c0 / 32 + f;
        if (cg >= CG) continue;
        const int col = f * 32 + (l & 31), rb = 8 * (l >> 5);
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            w[e] = static_cast<uint32_t>(tile[rb + 2 * e][col]) | (static_cast<uint32_t>(tile[rb + 2 * e + 1][col]) << 16);
        *reinterpret_cast<uint4*>(P + (static_cast<int64_t>(cg) * Ks + ks) * 512 + l * 8) =
            make_uint4(w[0], w[1], w[2], w[3]);
    }
}

typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;

// f(0) .. f(3) with the index as a compile-time constant
template <class F>
__device__ __forceinline__ void unroll4(F f) {
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
}

constexpr int WP_BM = 128, WP_TN = 256, WP_BK = 64, WP_ST = 3, WP_THREADS = 256;
// m tiles per super-row of the tile order (16: 1504 -> 1473 us per routed launch at 16384 x 4096,
// 160 experts, against 8; 4: 1492 us)
constexpr int kWpGroupM = 16;
constexpr int WP_A_BYTES = WP_BM * WP_BK * 2;  // 64 rows x 128 columns per stage
constexpr int WP_EPI = 2 * WP_A_BYTES;         // epilogue staging: past ring slots 0 and 1
// half an output tile: 64 m rows of 256 n, or 128 n rows of 128 m (pitches of + 8 elements)
constexpr int wp_epi_bytes(bool nrows) {
    return nrows ? (WP_TN / 2) * (WP_BM + 8) * 2 : (WP_BM / 2) * (WP_TN + 8) * 2;
}
constexpr int WP_LDS = WP_EPI + wp_epi_bytes(true);
static_assert(wp_epi_bytes(true) >= wp_epi_bytes(false), "either half tile fits");
static_assert(WP_LDS >= WP_ST * WP_A_BYTES, "the ring fits");

struct WpArgs {
    int n_groups, M, N;
    const int32_t* kp;   // [n_groups + 1] padded row prefix, or NULL: one group of T rows
    const int32_t* ranges;  // [9] first tile of each XCD's range (work-balanced), or NULL: equal counts
    int64_t T;
    const uint16_t* A;   // m operand, row-major: [T][M]
    const int32_t* map;  // row of A for each row of the groups, or NULL: the row itself
    const int32_t* off;  // [n_groups + 1] first row of each group (with kp)
    int64_t n_rows;      // rows of all groups (entries of map)
    const uint16_t* PB;  // k-packed n operand (N source columns)
    uint16_t* out;       // bf16 [n_groups][M][N], or [n_groups][N][M] (NROWS)
};

// Persistent: block (x = blockIdx % 8, seat) runs on XCD x and takes the
// tiles seat, seat + S, ... of XCD x's range (S blocks per XCD), so the
// resident blocks of an XCD work on consecutive tiles. The first two stages
// of a block's next tile are requested before the output of the current one
// is written (staged through LDS past ring slots 0 and 1, half a tile at a
// time, with buffer stores that every lane issues whatever the bounds), so
// the next tile's first data arrives while the stores drain.
//
// The m operand is dout or x as it is: a stage's 64 rows (MAP: gathered, their
// indices loaded a stage ahead of the DMA that needs them) of the tile's 128
// columns go to LDS row by row, and a fragment is two transposing reads of four
// rows of 16 columns per 16 lanes. DMA q of wave w brings rows 16 w + 4 a + q
// (a = 0..3) as 256-byte LDS rows 16 w + 4 q + a, their 16-byte chunks XORed
// with 4 q, so that the four rows of a transposing read lie in distinct banks.
// k-packed like the n operand, each of the gathered matrices took a pass of its
// own: 2 x 132 + 2 x 29 us for 16384 tokens x 2048, 64 experts top-6.
// NROWS: the output's rows are the n operand's columns (dW13, whose gathered
// operand is its columns): the matrix products swap their operands.
template <bool MAP, bool NROWS>
__global__ void __launch_bounds__(WP_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
wgrad_pk_kernel(WpArgs p) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[WP_LDS];
    const int tiles_m = static_cast<int>(ceil_div(p.M, WP_BM)), tiles_n = static_cast<int>(ceil_div(p.N, WP_TN));
    const int per = tiles_m * tiles_n;
    const int nblk = p.n_groups * per;
    const int xcd = blockIdx.x & 7, seat = blockIdx.x >> 3, seats = gridDim.x >> 3;
    int lo, hi;
    if (p.ranges != nullptr) {
        lo = p.ranges[xcd];
        hi = p.ranges[xcd + 1];
    } else {
        const int nb8 = static_cast<int>(ceil_div(nblk, 8));
        lo = xcd * nb8 < nblk ? xcd * nb8 : nblk;
        hi = lo + nb8 < nblk ? lo + nb8 : nblk;
    }
    lo = uniform_int(lo);
    hi = uniform_int(hi);
    int b = lo + seat;
    if (b >= hi) return;
    const int NG = static_cast<int>(ceil_div(p.N, 32));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int half = lane >> 5;

    const int lrow = 16 * wave + 4 * (lane >> 4) + (lane & 3);  // row of a stage whose index this lane holds
    const i32x4_t rsA = buf_rsrc(p.A, static_cast<int>(p.T * p.M * 2));
    const __amdgpu_buffer_rsrc_t rsI = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(p.map), 0, MAP ? static_cast<int>(p.n_rows * 4) : 0, kBufferFlags);

    // the tile whose operands are being requested: its group, corner, first
    // row, row and 16-row slice counts, and the n operand's descriptor
    struct Tile {
        int g, m0, n0, r0, rows, Ks;
        __amdgpu_buffer_rsrc_t rsB;
    };
    auto decode = [&](int bb) {
        Tile t;
        t.g = bb / per;
        const int tt = bb % per;
        // inside a group: super-rows of kWpGroupM m tiles; each n tile's operand slice serves the
        // m tiles of a super-row back to back
        const int sr = tt / (kWpGroupM * tiles_n), r8 = tt % (kWpGroupM * tiles_n);
        const int gm = tiles_m - sr * kWpGroupM < kWpGroupM ? tiles_m - sr * kWpGroupM : kWpGroupM;
        t.m0 = (sr * kWpGroupM + r8 % gm) * WP_BM;
        t.n0 = (r8 / gm) * WP_TN;
        const int64_t kp0 = p.kp != nullptr ? p.kp[t.g] : 0;
        const int64_t kp1 = p.kp != nullptr ? p.kp[t.g + 1] : ceil_div(p.T, 16) * 16;
        t.Ks = uniform_int(static_cast<int>((kp1 - kp0) / 16));  // 16-row slices of the group
        t.r0 = p.kp != nullptr ? uniform_int(p.off[t.g]) : 0;
        t.rows = p.kp != nullptr ? uniform_int(p.off[t.g + 1]) - t.r0 : static_cast<int>(p.T);
        const uint16_t* PBg = p.PB + 32 * static_cast<int64_t>(NG) * kp0;
        t.rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(uniform_ptr(PBg)), 0,
                                                  uniform_int(NG * t.Ks * 1024), kBufferFlags);
        return t;
    };
    const uint32_t lds_base = lds_address(lds);
    // index of this lane's row of stage s (any value past the group's rows: the DMA masks them)
    auto load_idx = [&](const Tile& t, int s) {
        return MAP ? __builtin_amdgcn_raw_buffer_load_b32(rsI, (t.r0 + 64 * s + lrow) * 4, 0, 0) : 0;
    };
    // byte offset in A of this lane's row of stage s, out of range past the group's rows
    auto row_off = [&](const Tile& t, int s, int idx) {
        const int R = 64 * s + lrow;
        return R < t.rows ? (MAP ? idx : t.r0 + R) * (p.M * 2) : kOutOfRange;
    };
    // A DMA q of a stage with row offsets ro into its ring slot: every lane of a row takes the
    // offset of row 4 (lane / 16) + q of the wave's 16 (a quad broadcast)
    auto issue_aq = [&](const Tile& t, int slot, int ro, auto q_c) {
        constexpr int q = decltype(q_c)::value;
        const int col = t.m0 * 2 + (((lane & 15) * 16) ^ (q * 64));  // M % 8 == 0: a chunk is all in or all out
        const int vo = static_cast<int>(static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(ro, q * 0x55, 0xf, 0xf, true)) +
                                        static_cast<uint32_t>(col)) |
                       (col < p.M * 2 ? 0 : kOutOfRange);
        dma16(rsA, vo, lds_base + slot * WP_A_BYTES + (wave * 4 + q) * 1024);
    };
    // the two n fragments (n groups n0 / 32 + 2 wave + gg) of slice 4 s + j
    auto issue_bj = [&](const Tile& t, i32x4_t (&bq)[4][2], int s, int j) {
        const int ks = 4 * s + j, ng = t.n0 / 32 + 2 * wave;
#pragma unroll
        for (int gg = 0; gg < 2; ++gg) {  // out of range past the group's rows and the matrix edge
            const int so = ks < t.Ks && ng + gg < NG ? ((ng + gg) * t.Ks + ks) * 1024 : kOutOfRange;
            bq[j][gg] = __builtin_amdgcn_raw_buffer_load_b128(
                t.rsB, static_cast<int>(static_cast<uint32_t>(so) + static_cast<uint32_t>(lane * 16)), 0, 0);
        }
    };
    i32x4_t b0[4][2], b1[4][2];
    // stages 0 and 1 of the decoded tile (row indices in i0 and i1): 16 loads per wave, the 4
    // DMAs of stage 0 first
    auto prologue = [&](const Tile& t, int i0, int i1) {
        const int ro0 = row_off(t, 0, i0), ro1 = row_off(t, 1, i1);
        unroll4([&](auto q) { issue_aq(t, 0, ro0, q); });
        unroll4([&](auto j) {
            issue_bj(t, b0, 0, j);
            issue_aq(t, 1, ro1, j);
        });
    };
    f32x16_t acc[4][2];
    // this lane's address for the transposing reads of m group 0, slice 0: row 4 q + 2 half (q =
    // lane % 16 / 4, logical row 8 half + q) and the one after it, columns 16 (lane / 16 % 2) +
    // 4 (lane % 4) ..; m group i is 64 i bytes away under the swizzle
    const int tq = (lane & 15) >> 2;
    const int tr0 = (4 * tq + 2 * half) * 256 + tq * 64 + ((lane >> 4) & 1) * 32 + ((lane & 3) >> 1) * 16 + (lane & 1) * 8;
    // stage s from ring slot `slot`: substep j issues the n fragments of stage
    // s + 1 (2 loads) and the DMA q = j of stage s + 2, reads the m fragments
    // of substep j + 1 and runs 8 MFMAs. ic: row indices of stage s + 2; in: those of
    // stage s + 3, loaded first.
    auto stage_run = [&](const Tile& t, int slot, int s, const i32x4_t (&bc)[4][2], i32x4_t (&bn)[4][2], int ic, int& in) {
        const uint8_t* base = lds + slot * WP_A_BYTES;
        const int nslot = slot == 0 ? 2 : slot - 1;  // (slot + 2) % 3
        bf16x8_t af[2][4];
        auto rd = [&](int j, bf16x8_t (&a)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint8_t* a0 = base + (tr0 ^ (i * 64)) + j * 4096;
                const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)a0);
                const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(a0 + 256));
                const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                a[i] = __builtin_bit_cast(bf16x8_t, make_uint4(l2.x, l2.y, h2.x, h2.y));
            }
        };
        rd(0, af[0]);
        const int ro = row_off(t, s + 2, ic);
        in = load_idx(t, s + 3);
        unroll4([&](auto j_c) {
            constexpr int j = decltype(j_c)::value;
            __builtin_amdgcn_sched_barrier(0);
            issue_bj(t, bn, s + 1, j);
            issue_aq(t, nslot, ro, j_c);
            if constexpr (j < 3) rd(j + 1, af[(j + 1) & 1]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int gg = 0; gg < 2; ++gg) {
                    const bf16x8_t n = __builtin_bit_cast(bf16x8_t, bc[j][gg]);
                    if constexpr (NROWS)  // rows of the MFMA tile: m, columns: n
                        acc[i][gg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[j & 1][i], n, acc[i][gg], 0, 0, 0);
                    else  // rows of the MFMA tile: n, columns: m
                        acc[i][gg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(n, af[j & 1][i], acc[i][gg], 0, 0, 0);
                }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    // Vector memory operations retire in order. Before stage s reads its
    // slot, at most the loads issued after the last DMA of stage s may still
    // fly: for s >= 2 the 12 of stage s - 1's run (n fragments of stage s,
    // DMA of stage s + 1); for s = 0 and 1 of every tile but a block's first
    // also the 16 output stores of the previous tile, issued after this
    // tile's first two stages were requested. Row index loads are not counted:
    // they are the oldest of their run and due in the next one. The barrier makes every
    // wave's DMA visible and frees the slot the DMA of stage s + 2
    // overwrites. Past the group's rows every load is out of range and
    // returns zeros, so every stage issues the same count and the waits stay
    // exact.
    constexpr int kStoresPerTile = (WP_BM * WP_TN / 8) / WP_THREADS;  // 16-byte stores per lane
    Tile cur = decode(b);
    int ie = load_idx(cur, 2), io = 0;  // row indices of the even and odd stage that the DMAs reach next
    {
        const int i0 = load_idx(cur, 0), i1 = load_idx(cur, 1);
        prologue(cur, i0, i1);
    }
    bool after_stores = false;
    for (;;) {
        // the next tile and the row indices of its first two stages, loaded under this one's products
        const int nb = b + seats;
        Tile nxt = cur;
        if (nb < hi) nxt = decode(nb);
        const int n0i = load_idx(nxt, 0), n1i = load_idx(nxt, 1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int gg = 0; gg < 2; ++gg) acc[i][gg] = f32x16_t{};
        const int nk = static_cast<int>(ceil_div(cur.Ks, 4));
        {
            int s = 0, slot = 0;
            if (nk > 0) {
                if (after_stores) wait_vm_lgkm0<12 + kStoresPerTile>();
                else wait_vm_lgkm0<12>();
                dma_barrier();
                stage_run(cur, 0, 0, b0, b1, ie, io);
            }
            if (nk > 1) {
                if (after_stores) wait_vm_lgkm0<12 + kStoresPerTile>();
                else wait_vm_lgkm0<12>();
                dma_barrier();
                stage_run(cur, 1, 1, b1, b0, io, ie);
            }
            s = 2;
            slot = 2;
            for (; s + 2 <= nk; s += 2) {
                wait_vm_lgkm0<12>();
                dma_barrier();
                stage_run(cur, slot, s, b0, b1, ie, io);
                slot = slot == 2 ? 0 : slot + 1;
                wait_vm_lgkm0<12>();
                dma_barrier();
                stage_run(cur, slot, s + 1, b1, b0, io, ie);
                slot = slot == 2 ? 0 : slot + 1;
            }
            if (s < nk) {
                wait_vm_lgkm0<12>();
                dma_barrier();
                stage_run(cur, slot, s, b0, b1, ie, io);
            }
        }
        wait_vm_lgkm0<0>();  // drain: the next tile's DMA reuses the ring
        dma_barrier();
        // output of this tile, then the next tile's first two stages
        const int og = cur.g, om0 = cur.m0, on0 = cur.n0;
        if (nb < hi) {
            cur = nxt;
            ie = load_idx(cur, 2);
            prologue(cur, n0i, n1i);
        }
        const __amdgpu_buffer_rsrc_t rsO = __builtin_amdgcn_make_buffer_rsrc(
            uniform_ptr(p.out + static_cast<int64_t>(og) * p.M * p.N), 0, uniform_int(p.M * p.N * 2), kBufferFlags);
        uint16_t* ot = reinterpret_cast<uint16_t*>(lds + WP_EPI);
        // opaque: the addresses below are rebuilt per tile instead of held in registers across the K loop
        int tid = static_cast<int>(threadIdx.x);
        asm volatile("" : "+v"(tid));
        const int e_half = (tid >> 5) & 1, e_l32 = tid & 31;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // Element v of lane l of acc[i][gg] is n = 8 (v / 4) + 4 half + v % 4 of n group 2 wave
            // + gg of the tile and m = l32 of m group i (NROWS: m and n the other way round). Four
            // adjacent columns of an output row go to LDS as 8 bytes, then whole rows of the half
            // tile (m groups 2 h, 2 h + 1; NROWS: n group h of each wave) to memory.
            constexpr int OC = NROWS ? WP_BM : WP_TN, OP = OC + 8;  // columns and row pitch
            auto put = [&](const f32x16_t& a, int vq, int row, int col) {
                *reinterpret_cast<uint2*>(ot + row * OP + col + 8 * vq + 4 * e_half) =
                    make_uint2(static_cast<uint32_t>(f32_to_bf16(a[4 * vq])) |
                                   (static_cast<uint32_t>(f32_to_bf16(a[4 * vq + 1])) << 16),
                               static_cast<uint32_t>(f32_to_bf16(a[4 * vq + 2])) |
                                   (static_cast<uint32_t>(f32_to_bf16(a[4 * vq + 3])) << 16));
            };
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                if constexpr (NROWS) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) put(acc[i][h], vq, wave * 32 + e_l32, i * 32);
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int gg = 0; gg < 2; ++gg) put(acc[2 * h + i][gg], vq, i * 32 + e_l32, wave * 64 + gg * 32);
                }
            }
            __syncthreads();
            constexpr int CH = OC / 8;
            const int n_r = NROWS ? p.N : p.M, n_c = NROWS ? p.M : p.N;
#pragma unroll
            for (int u = 0; u < kStoresPerTile / 2; ++u) {
                const int q = u * WP_THREADS + tid;
                const int r = q / CH, c = (q % CH) * 8;
                const int row = NROWS ? on0 + (r / 32) * 64 + 32 * h + r % 32 : om0 + 64 * h + r;
                const int col = (NROWS ? om0 : on0) + c;
                // n_c % 8 == 0: a chunk is all in or all out; out of range the store is dropped
                const int vo = (row < n_r && col < n_c) ? (row * n_c + col) * 2 : kOutOfRange;
                __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const i32x4_t*>(ot + r * OP + c), rsO, vo, 0,
                                                       kBufferNonTemporal);
            }
            __syncthreads();  // the half tile's LDS reads are done before the next writes
        }
        if (nb >= hi) break;
        b = nb;
        after_stores = true;
    }
}

}  // namespace

int64_t kpack_elems(int C, int64_t padded_rows) { return 32 * ceil_div(C, 32) * padded_rows; }

int wgrad_tiles_per_group(int M, int N) { return static_cast<int>(ceil_div(M, WP_BM) * ceil_div(N, WP_TN)); }

hipError_t launch_kpad_offsets(const int32_t* off, int E, int32_t* kp, int per0, int per1, int32_t* ranges,
                               hipStream_t stream) {
    if (E < 1 || E > 256) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kpad_offsets_kernel, dim3(1), dim3(256), 0, stream, off, E, kp, per0, per1, ranges);
    return hipGetLastError();
}

hipError_t launch_kpack(const void* S, int C, int64_t T, void* P, hipStream_t stream) {
    if (T == 0 || C == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(ceil_div(T, 16)), static_cast<unsigned>(ceil_div(C, KP_COLS)));
    hipLaunchKernelGGL(kpack_kernel, grid, dim3(256), 0, stream, static_cast<const uint16_t*>(S), C, T,
                       static_cast<uint16_t*>(P));
    return hipGetLastError();
}

hipError_t launch_wgrad_pk(int n_groups, int M, int N, bool n_rows_out, const void* A, const int32_t* map,
                           const int32_t* off, const int32_t* kp, const int32_t* ranges, int64_t T, int64_t n_rows,
                           const void* PB, void* out, hipStream_t stream) {
    if (n_groups == 0 || M == 0 || N == 0) return hipSuccess;
    WpArgs p;
    p.n_groups = n_groups;
    p.M = M;
    p.N = N;
    p.kp = kp;
    p.ranges = ranges;
    p.T = T;
    p.A = static_cast<const uint16_t*>(A);
    p.map = map;
    p.off = off;
    p.n_rows = n_rows;
    p.PB = static_cast<const uint16_t*>(PB);
    p.out = static_cast<uint16_t*>(out);
    // two resident workgroups per CU, 32 CUs per XCD; fewer when there are fewer tiles
    const int64_t nblk = static_cast<int64_t>(n_groups) * ceil_div(M, WP_BM) * ceil_div(N, WP_TN);
    const int64_t per_xcd = ceil_div(nblk, 8) < 64 ? ceil_div(nblk, 8) : 64;
    const auto kernel = map != nullptr ? (n_rows_out ? wgrad_pk_kernel<true, true> : wgrad_pk_kernel<true, false>)
                                       : (n_rows_out ? wgrad_pk_kernel<false, true> : wgrad_pk_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(8 * per_xcd)), dim3(WP_THREADS), 0, stream, p);
    return hipGetLastError();
}

}  // namespace smoes
