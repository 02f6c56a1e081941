// Grouped expert GEMMs over the permuted routes (gated-MLP experts, Appendix E.2;
// weighted sum of Eq. pr2_output).
//
//   GEMM1  H[rows_e, m] = silu(X_e W_gate_e^T) * (X_e W_up_e^T)   X_e gathered from x
//   GEMM2  O[rows_e, d] = g * (H_e W_down_e^T)                     g = replay weight
//
// bf16 path (d % 256 == 0, m % 128 == 0): one workgroup computes a 256-row tile
// of one expert against a 256-row panel of weights (GEMM1: 128 gate rows + the
// matching 128 up rows; GEMM2: 256 rows of W_down).  K advances in slices of 64
// (one 128-byte line per row) copied straight from global memory into LDS with
// 16-byte DMA loads (no register staging), two LDS stages deep (the next slice
// in flight while one is consumed), 16-byte chunks XOR-swizzled per row so the
// MFMA operand reads are free of bank conflicts.
// Eight wavefronts (two per SIMD) in a 4 x 2 arrangement each own 64 rows x 128
// panel rows as 4 x 8 tiles of v_mfma_f32_16x16x32_bf16 (fp32 accumulation;
// it issues about 9 % faster than the 32x32x16 form on gfx950 and gives the
// same sums);
// operand fragments are double-buffered in registers and the LDS reads of each
// K=32 sub-step run among the MFMAs of the one before, across slices too: the
// slice's only barrier sits between its two sub-steps, after which its stage is
// refilled and the next slice's first fragments are read.  (With the barrier at
// the slice's start, all eight wavefronts waited for 96 KiB of LDS reads with
// the matrix units idle.  GEMM1, traced on one box: 334 -> 306 us at 4099 tokens,
// d 2048, 64 experts, k 8, m 1024; with the 384-row panel 826 -> 768 us at 16384
// tokens, 128 experts, m 768.  GEMM2, K = 768: unchanged, its tiles' prologue
// and epilogue outweigh 12 slices.)  A wavefront whose rows are all past the end
// of a partial tile only copies.
// GEMM1's epilogue applies SwiGLU in registers (gate and up tiles of the same
// columns live in the same lanes) and rounds H to bf16; GEMM2's epilogue scales
// by the route weight and rounds O to bf16.  The MFMA operands are given as
// (weights, tokens), so each lane's accumulators hold runs of four consecutive
// output columns of one token row.  GEMM1 stores them 8 bytes at a time
// straight from registers; GEMM2 (and the pre-activation epilogue below)
// stages its outputs through the freed LDS stages so that every store covers
// whole row segments.  Workgroups are mapped so that each XCD takes a
// contiguous range of the tile list (same experts, shared L2).
//
// A third epilogue serves the backward pass: it stores the pre-activations
// a = X_e W_gate_e^T and u = X_e W_up_e^T (bf16) instead of H; a fourth stores
// both (a forward that saves them for the backward).
//
// When m is a multiple of 192, the forward GEMM1 runs a second kernel with a
// 384-row panel (192 gate + 192 up rows; 80 KiB per LDS stage, all 160 KiB of
// LDS in two stages), 17 % fewer copied bytes per flop: each of the eight
// wavefronts owns 64 token rows x 192 panel rows (192 accumulators per lane),
// reads its A fragments once per K=32 step and its B fragments two tiles at a
// time, double-buffered, with the same barrier placement.  Per output the sums
// run in the same K order as the 256-row panel, so H is bitwise the same.
//
// Other shapes and the fp32 path take the fp32-FMA tile kernels of tile.hip.
#include <type_traits>

#include "common.h"

namespace pr2 {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = kTileM;      // 256 rows per tile
constexpr int BP = 256;         // weight panel rows per tile
constexpr int BK = 64;          // K slice: 128 bytes per row
constexpr int ROWB = BK * 2;    // bytes per LDS row (unpadded; chunks are swizzled)
constexpr int CHUNKS = ROWB / 16;   // 16-byte chunks per row
constexpr int NSTAGE = 2;       // LDS stages: slices kt+1 .. kt+NSTAGE-1 in flight during slice kt
constexpr int WM = 64;          // token rows per wavefront
constexpr int WN = 128;         // panel rows per wavefront
constexpr int MT = 16;          // MFMA tile edge (16x16x32)
constexpr int MK = 32;          // K per MFMA
constexpr int NKS = BK / MK;    // MFMA K sub-steps per slice
constexpr int MI = WM / MT;     // MFMA tiles per wavefront, token direction
constexpr int NJ = WN / MT;     // MFMA tiles per wavefront, panel direction
typedef f32x4 accv;             // a lane's accumulators of one tile

__device__ __forceinline__ accv mfma_bf16(bf16x8 a, bf16x8 b, accv c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
constexpr int NWAVE = (BM / WM) * (BP / WN);
constexpr int kGemmThreads = 64 * NWAVE;
constexpr int kNumXcd = 8;
constexpr int kRowsPerDma = 1024 / ROWB;                                   // 8 rows / DMA
constexpr int kGroups = (BM + BP) / kRowsPerDma / NWAVE;                    // DMAs / wavefront
constexpr int STAGEB = (BM + BP) * ROWB;                                    // 64 KiB
constexpr int LDSB = NSTAGE * STAGEB;

struct MfmaArgs {
    const bf16_t* A;        // GEMM1: x [T, d]; GEMM2: H [T*k, m]
    const int* perm_src;    // permuted row -> t*k + s
    int k;
    int Tk;                 // routes (perm_src entries)
    const bf16_t* W0;       // GEMM1: W_gate; GEMM2: W_down
    const bf16_t* W1;       // GEMM1: W_up
    int K;                  // reduction length (d or m)
    int n_out;              // output row length (m or d)
    int ntn;                // panels per expert
    int64_t w_stride;       // elements per expert weight matrix
    const int* tiles;
    const int* tile_count;
    const float* gate;      // GEMM2
    bf16_t* out;
    bf16_t* out2;           // GEMM1 that also saves a | u (MODE 3): [T*k, 2m]
};

// silu(a) = a / (1 + e^-a) with the hardware reciprocal (about 1 ulp; H is rounded to bf16)
__device__ __forceinline__ float silu_f(float a) {
    return a * __builtin_amdgcn_rcpf(1.0f + __expf(-a));
}

// 16-byte chunk c of LDS row r is stored at position c ^ swz(r): any 16 (or
// 8) consecutive rows read at the same chunk hit disjoint banks.  swz depends
// on r % 16 only.
__device__ __forceinline__ int swz(int r) {
    return (r & 7) ^ ((r >> 3) & 1);
}

// wait until at most n of this wavefront's global loads are outstanding
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(n >= 0 && n < 16, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0f70 | n);   // expcnt and lgkmcnt left at their maxima
}

template <int MODE>
__global__ void __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
grouped_gemm_mfma(MfmaArgs g) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[LDSB];

    // XCD-aware mapping: physical block b runs on XCD b % 8; give each XCD a
    // contiguous range of the (tile, panel) work list, every panel of a tile in
    // turn (groups of 2, 4 or 8 tiles, panel by panel inside a group: within 1 %)
    const int64_t L = (int64_t)(*g.tile_count) * g.ntn;
    const int64_t per_xcd = (L + kNumXcd - 1) / kNumXcd;
    const int64_t local = blockIdx.x / kNumXcd;
    if (local >= per_xcd) return;
    const int64_t logical = (int64_t)(blockIdx.x % kNumXcd) * per_xcd + local;
    if (logical >= L) return;
    const int tile = (int)(logical / g.ntn);
    const int pn = (int)(logical % g.ntn);
    const int expert = g.tiles[3 * tile + 0];
    const int row0 = g.tiles[3 * tile + 1];
    const int rows = g.tiles[3 * tile + 2];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // uniform across the wavefront; saying so lets the compiler branch on it
    // with scalar branches instead of per-lane masks
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / (BP / WN);     // token-row block of WM rows
    const int wc = wave % (BP / WN);     // panel block of WN rows
    // a wavefront whose rows are all past the tile's end only helps copy
    const bool active = wr * WM < rows;
    // DMA assignments: wavefront w copies row groups w*kGroups .. of the
    // [A rows | panel rows] tile; lane l moves row grp*kRowsPerDma + l/CHUNKS,
    // position l%CHUNKS.  A wavefront's groups all come from one tensor (the
    // token rows, the gate or up panel, or the down panel), so it keeps one
    // base pointer and a 32-bit element offset per group.
    const int wrow0 = wave * kGroups * kRowsPerDma;
    const bf16_t* sbase;
    if (wrow0 < BM) sbase = g.A;
    else if (MODE != 1) sbase = (wrow0 - BM < 128 ? g.W0 : g.W1) + (int64_t)expert * g.w_stride;
    else sbase = g.W0 + (int64_t)expert * g.w_stride;
    // (wrow0 < BM holds for a whole wavefront: a scalar branch, and the
    // gathered route entries are loaded together before any is used)
    uint32_t soff[kGroups];
    if (wrow0 < BM) {
        // rows past the tile's end read a valid row; their results are never stored
        int rsrc[kGroups];
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            const int r = wrow0 + i * kRowsPerDma + lane / CHUNKS;
            const int rr = r < rows ? r : 0;
            rsrc[i] = MODE != 1 ? g.perm_src[row0 + rr] : row0 + rr;
        }
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            const int r = wrow0 + i * kRowsPerDma + lane / CHUNKS;
            const int64_t row = MODE != 1 ? (int64_t)(min(max(rsrc[i], 0), g.Tk - 1) / g.k) : rsrc[i];
            soff[i] = 2 * (uint32_t)(row * g.K + ((lane % CHUNKS) ^ swz(r)) * 8);
        }
    } else {
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            const int r = wrow0 + i * kRowsPerDma + lane / CHUNKS;  // row in [BM, BM + BP)
            const int pr = r - BM;
            const int64_t off = MODE != 1 ? (int64_t)(pn * 128 + (pr & 127)) * g.K
                                          : (int64_t)(pn * BP + pr) * g.K;
            soff[i] = 2 * (uint32_t)(off + ((lane % CHUNKS) ^ swz(r)) * 8);
        }
    }
    accv acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            acc[i][j] = accv{0.0f, 0.0f, 0.0f, 0.0f};

    // LDS reads for the MFMA operands: lane l reads row (block base + l%MT)
    // and the 16 bytes of one 8-wide K chunk, at position chunk ^ swz(row);
    // block bases are multiples of 16 rows, so the swizzle is the same for
    // every fragment.  Which chunk of the sub-step a lane group g = l/MT
    // takes is free (A and B fragments use the same assignment, so each MFMA
    // still sums over the same K values): a ds_read_b128 serves lanes
    // 8q..8q+7 together with lanes 32+8q..32+8q+7, so groups g and g+2 take chunks differing in the lowest bit (0,2,1,3), which keeps
    // the two halves of every LDS cycle in disjoint banks.
    const int lrow = lane % MT;
    const int sw = swz(lrow);
    const int grp = lane / MT;
    const int cperm = ((grp & 1) << 1) | (grp >> 1);
    int kpos[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
        kpos[ks] = lrow * ROWB + ((((MK / 8) * ks + cperm) ^ sw) << 4);
    int a_base[MI], b_base[NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i) a_base[i] = (wr * WM + i * MT) * ROWB;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        int prow;
        if (MODE != 1) prow = (j < NJ / 2 ? 0 : 128) + wc * (WN / 2) + (j % (NJ / 2)) * MT;
        else prow = wc * WN + j * MT;
        b_base[j] = (BM + prow) * ROWB;
    }

    // copies of this wavefront per slice: 8, fewer (in twos: 16 rows) where its
    // token rows run past a partial tile's end.  No stored output depends on
    // those LDS rows.
    const int ncopy = wrow0 >= BM ? kGroups
                                  : min(kGroups, max(0, (rows - wrow0 + 2 * kRowsPerDma - 1) / (2 * kRowsPerDma)) * 2);
    auto issue = [&](int stage, int k0, int q) __attribute__((always_inline)) {
        if (ncopy <= 2 * q) return;
#pragma unroll
        for (int i = 2 * q; i < 2 * q + 2; ++i)
            dma16_at(sbase + k0, soff[i], &lds[stage * STAGEB + (wave * kGroups + i) * 1024]);
    };
    auto issue_all = [&](int stage, int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kGroups / 2; ++q) issue(stage, k0, q);
    };
    // K loop, one barrier per slice.  A slice is two K=32 sub-steps; the
    // fragments of sub-step s + 1 are read from LDS among the MFMAs of sub-step
    // s, across slices too, so no MFMA waits for a read issued after a barrier.
    // The barrier sits between a slice's two sub-steps: every wavefront holds the
    // slice's last fragments by then, so the slice's stage takes the copies of
    // slice kt + 2, and slice kt + 1 (copied for a whole slice's time) has landed.
    static_assert(NSTAGE == 2 && NKS == 2 && MI == 4 && NJ == 8 && kGroups == 8,
                  "K loop layout");
    const int nk = g.K / BK;             // at least 2 (K is a multiple of 128)
    bf16x8 fa[2][MI], fb[2][NJ];
    auto sync = [&]() __attribute__((always_inline)) {
        wait_vmcnt<0>();
        __syncthreads();
    };
    // MFMAs of one sub-step on fragment set S; among them the copies of one
    // slice (ISSUE) and the reads of the next sub-step's fragments (READ)
    auto phase = [&](auto S_, auto READ, auto ISSUE, int rstage, int ks, int istage,
                     int k0) __attribute__((always_inline)) {
        constexpr int S = decltype(S_)::value;
        const unsigned char* base = lds + rstage * STAGEB + kpos[ks];
        auto read_a = [&](int i) __attribute__((always_inline)) {
            fa[S ^ 1][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(base + a_base[i]));
        };
        auto read_b = [&](int j) __attribute__((always_inline)) {
            fb[S ^ 1][j] = __builtin_bit_cast(bf16x8, *(const u32x4*)(base + b_base[j]));
        };
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (decltype(ISSUE)::value) issue(istage, k0, q);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 2 * q; j < 2 * q + 2; ++j)
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i][j] = mfma_bf16(fb[S][j], fa[S][i], acc[i][j]);
            __builtin_amdgcn_sched_barrier(0);
            if (decltype(READ)::value && q < 3) {
                if (q < 2) {
                    read_a(2 * q);
                    read_b(2 * q);
                    read_a(2 * q + 1);
                    read_b(2 * q + 1);
                } else {
                    read_b(4);
                    read_b(5);
                    read_b(6);
                    read_b(7);
                }
            }
        }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    // the first two slices go out together; slice 0 is waited for alone (a plain
    // barrier: __syncthreads() would wait for slice 1 as well)
    issue_all(0, 0);
    issue_all(1, BK);
    if (ncopy == kGroups) wait_vmcnt<kGroups>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    int kt = 0;
    if (active) {
        const unsigned char* base = lds + kpos[0];
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[0][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(base + a_base[i]));
#pragma unroll
        for (int j = 0; j < NJ; ++j) fb[0][j] = __builtin_bit_cast(bf16x8, *(const u32x4*)(base + b_base[j]));
        __builtin_amdgcn_s_waitcnt(0xc07f);
        for (; kt + 2 < nk; ++kt) {
            phase(C0{}, C1{}, C0{}, kt & 1, 1, 0, 0);
            sync();
            phase(C1{}, C1{}, C1{}, (kt + 1) & 1, 0, kt & 1, (kt + 2) * BK);
        }
        phase(C0{}, C1{}, C0{}, kt & 1, 1, 0, 0);
        sync();
        phase(C1{}, C1{}, C0{}, (kt + 1) & 1, 0, 0, 0);
        ++kt;
        phase(C0{}, C1{}, C0{}, kt & 1, 1, 0, 0);
        phase(C1{}, C0{}, C0{}, 0, 0, 0, 0);
    } else {
        // only copies, with the same barriers
        for (; kt + 2 < nk; ++kt) {
            sync();
            issue_all(kt & 1, (kt + 2) * BK);
        }
        sync();
    }
    // Epilogue.  The MFMA computed the transposed tile (weights x tokens), so
    // accumulator element v of lane l is column 4*(l/16) + v of token row l%16 of
    // its block: runs of four consecutive outputs per lane.
    if ((MODE == 0 || MODE == 3) && active) {
        // GEMM1: H = silu(gate) * up, stored straight from registers, one
        // 8-byte write per run (gate and up tiles of the same columns sit in
        // the same lanes)
        const int ncol0 = 4 * (lane / MT);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int r = wr * WM + i * MT + (lane % MT);
            if (r >= rows) continue;
            bf16_t* orow = g.out + ((int64_t)row0 + r) * g.n_out;
#pragma unroll
            for (int j = 0; j < NJ / 2; ++j) {
                const int col = pn * 128 + wc * (WN / 2) + j * MT + ncol0;
                uint32_t w[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float h0 = silu_f(acc[i][j][2 * h]) * acc[i][j + NJ / 2][2 * h];
                    const float h1 = silu_f(acc[i][j][2 * h + 1]) * acc[i][j + NJ / 2][2 * h + 1];
                    w[h] = (uint32_t)f32_to_bf16(h0) | ((uint32_t)f32_to_bf16(h1) << 16);
                }
                *(uint2*)(orow + col) = make_uint2(w[0], w[1]);
            }
        }
    }
    // MODE 3 goes on to save the pre-activations a | u as MODE 2 stores them
    if (MODE == 0) return;

    // GEMM2 (route weight times the output) and the pre-activations (a and u)
    // are staged: the rounded outputs go into this wavefront's LDS region (64
    // rows of CW columns per output block, 16-byte chunks XOR-swizzled by
    // row, the two 8-byte halves of a chunk swapped in rows with bit 3 set so
    // that the 16 rows of one 8-byte write cycle hit 16 distinct bank pairs)
    // and are read back 16 bytes per lane, so that each global store
    // covers whole row segments (256 or 128 contiguous bytes) instead of
    // 8-byte pieces of 16 rows: measured 10 % faster for GEMM2 (and slower
    // for GEMM1, whose outputs are half as wide).
    // Every wavefront must be done with the operand stages first.
    // GEMM2: the route weights of this lane's MI token rows (rows clamped into
    // the tile, so that the loads all go out together; padding rows are not stored)
    float gw[MI];
    if (MODE == 1 && active) {
        int src[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) src[i] = g.perm_src[row0 + min(wr * WM + i * MT + (lane % MT), rows - 1)];
#pragma unroll
        for (int i = 0; i < MI; ++i) gw[i] = g.gate[min(max(src[i], 0), g.Tk - 1)];
    }
    __syncthreads();
    if (!active) return;
    constexpr int CW = MODE == 1 ? WN : WN / 2;          // columns per output block
    constexpr bool kPreact = MODE == 2 || MODE == 3;     // stores a | u
    constexpr int NB = kPreact ? 2 : 1;                   // output blocks per wavefront
    constexpr int RB = CW * 2;                            // bytes per staged row
    constexpr int NCH = RB / 16;                          // 16-byte chunks per row
    unsigned char* stage_w = lds + wave * (NB * WM * RB);
    auto spos = [&](int blk, int row, int col) {          // byte offset of (row, col), col % 4 == 0
        const int ch = (col >> 3) ^ (row & (NCH - 1));
        return blk * WM * RB + row * RB + (ch << 4) + (((col & 4) << 1) ^ (row & 8));
    };
    const int ncol0 = 4 * (lane / MT);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row = i * MT + (lane % MT);
#pragma unroll
        for (int j = 0; j < (MODE == 1 ? NJ : NJ / 2); ++j) {
            const int col = j * MT + ncol0;
            if (kPreact) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int jj = j + half * (NJ / 2);
                    const uint32_t w0 = (uint32_t)f32_to_bf16(acc[i][jj][0]) |
                                        ((uint32_t)f32_to_bf16(acc[i][jj][1]) << 16);
                    const uint32_t w1 = (uint32_t)f32_to_bf16(acc[i][jj][2]) |
                                        ((uint32_t)f32_to_bf16(acc[i][jj][3]) << 16);
                    *(uint2*)(stage_w + spos(half, row, col)) = make_uint2(w0, w1);
                }
            } else {
                const uint32_t w0 = (uint32_t)f32_to_bf16(gw[i] * acc[i][j][0]) |
                                    ((uint32_t)f32_to_bf16(gw[i] * acc[i][j][1]) << 16);
                const uint32_t w1 = (uint32_t)f32_to_bf16(gw[i] * acc[i][j][2]) |
                                    ((uint32_t)f32_to_bf16(gw[i] * acc[i][j][3]) << 16);
                *(uint2*)(stage_w + spos(0, row, col)) = make_uint2(w0, w1);
            }
        }
    }
    // the wavefront's own region: LDS operations of one wavefront complete in order
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    constexpr int RPI = 64 / NCH;                         // rows per 64-lane pass
    const int rsub = lane / NCH, ch = lane % NCH;
    bf16_t* const dst = MODE == 3 ? g.out2 : g.out;
    const int ldo = MODE == 3 ? 2 * g.n_out : g.n_out;   // MODE 3: H rows are m, a | u rows 2m
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
        int colbase;
        if (MODE == 1) colbase = pn * BP + wc * WN;
        else colbase = blk * (ldo / 2) + pn * 128 + wc * (WN / 2);
#pragma unroll
        for (int p = 0; p < WM / RPI; ++p) {
            const int row = p * RPI + rsub;
            const int r = wr * WM + row;
            u32x4 v = *(const u32x4*)(stage_w + blk * WM * RB + row * RB + ((ch ^ (row & (NCH - 1))) << 4));
            if (row & 8) v = u32x4{v[2], v[3], v[0], v[1]};
            if (r < rows) *(u32x4*)(dst + ((int64_t)row0 + r) * ldo + colbase + ch * 8) = v;
        }
    }
}

// ------------------------------------------- GEMM1 with a 384-row panel --
constexpr int BPW = 384;                          // panel rows
constexpr int WNW = 192;                          // panel rows per wavefront (96 gate + 96 up)
constexpr int NJW = WNW / MT;                     // 12
constexpr int STAGEBW = (BM + BPW) * ROWB;        // 80 KiB
constexpr int LDSBW = NSTAGE * STAGEBW;           // 160 KiB
constexpr int kAGroupsW = BM / kRowsPerDma / NWAVE;          // 4 token-row groups per wavefront
constexpr int kWGroupsW = (BPW / 2) / kRowsPerDma / NWAVE;   // 3 gate (and 3 up) groups per wavefront
static_assert(kAGroupsW * kRowsPerDma * NWAVE == BM && kWGroupsW * kRowsPerDma * NWAVE * 2 == BPW,
              "row groups divide evenly");

__global__ void __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
gemm1_wide(MfmaArgs g) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[LDSBW];
    const int64_t L = (int64_t)(*g.tile_count) * g.ntn;
    const int64_t per_xcd = (L + kNumXcd - 1) / kNumXcd;
    const int64_t local = blockIdx.x / kNumXcd;
    if (local >= per_xcd) return;
    const int64_t logical = (int64_t)(blockIdx.x % kNumXcd) * per_xcd + local;
    if (logical >= L) return;
    const int tile = (int)(logical / g.ntn);
    const int pn = (int)(logical % g.ntn);
    const int expert = g.tiles[3 * tile + 0];
    const int row0 = g.tiles[3 * tile + 1];
    const int rows = g.tiles[3 * tile + 2];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / (BPW / WNW);
    const int wc = wave % (BPW / WNW);
    const bool active = wr * WM < rows;

    // copies: wavefront w moves token-row groups 4w..4w+3, gate groups
    // 3w..3w+2 and up groups 3w..3w+2 (8 rows of 128 bytes each)
    const bf16_t* wg = g.W0 + (int64_t)expert * g.w_stride;
    const bf16_t* wu = g.W1 + (int64_t)expert * g.w_stride;
    uint32_t soa[kAGroupsW], sog[kWGroupsW], sou[kWGroupsW];
    {
        int rsrc[kAGroupsW];
#pragma unroll
        for (int i = 0; i < kAGroupsW; ++i) {
            const int r = (wave * kAGroupsW + i) * kRowsPerDma + lane / CHUNKS;
            rsrc[i] = g.perm_src[row0 + (r < rows ? r : 0)];
        }
#pragma unroll
        for (int i = 0; i < kAGroupsW; ++i) {
            const int r = (wave * kAGroupsW + i) * kRowsPerDma + lane / CHUNKS;
            const int64_t row = (int64_t)(min(max(rsrc[i], 0), g.Tk - 1) / g.k);
            soa[i] = 2 * (uint32_t)(row * g.K + ((lane % CHUNKS) ^ swz(r)) * 8);
        }
#pragma unroll
        for (int i = 0; i < kWGroupsW; ++i) {
            const int pr = (wave * kWGroupsW + i) * kRowsPerDma + lane / CHUNKS;   // 0..191
            const uint32_t off = (uint32_t)((int64_t)(pn * (BPW / 2) + pr) * g.K);
            sog[i] = 2 * (off + ((lane % CHUNKS) ^ swz(BM + pr)) * 8);
            sou[i] = 2 * (off + ((lane % CHUNKS) ^ swz(BM + BPW / 2 + pr)) * 8);
        }
    }
    // copies n0 .. n1-1 of a slice: token-row groups, then gate, then up groups;
    // a wavefront whose 32 token rows are all past a partial tile's end copies none
    const bool acopies = wave * kAGroupsW * kRowsPerDma < rows;
    auto issue = [&](int stage, int k0, int n0, int n1) __attribute__((always_inline)) {
        unsigned char* sb = lds + stage * STAGEBW;
#pragma unroll
        for (int n = n0; n < n1; ++n) {
            if (n < kAGroupsW) {
                if (acopies) dma16_at(g.A + k0, soa[n], sb + (wave * kAGroupsW + n) * 1024);
            } else if (n < kAGroupsW + kWGroupsW)
                dma16_at(wg + k0, sog[n - kAGroupsW],
                         sb + (BM / kRowsPerDma + wave * kWGroupsW + n - kAGroupsW) * 1024);
            else
                dma16_at(wu + k0, sou[n - kAGroupsW - kWGroupsW],
                         sb + ((BM + BPW / 2) / kRowsPerDma + wave * kWGroupsW + n - kAGroupsW -
                               kWGroupsW) * 1024);
        }
    };

    accv acc[MI][NJW];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJW; ++j)
            acc[i][j] = accv{0.0f, 0.0f, 0.0f, 0.0f};

    const int lrow = lane % MT;
    const int sw = swz(lrow);
    const int grp = lane / MT;
    const int cperm = ((grp & 1) << 1) | (grp >> 1);
    int kpos[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
        kpos[ks] = lrow * ROWB + ((((MK / 8) * ks + cperm) ^ sw) << 4);
    const int a0 = (wr * WM) * ROWB;
    // panel row of fragment j: gate rows for j < NJW/2, the matching up rows after
    const int b0 = (BM + wc * (WNW / 2)) * ROWB;

    // K loop: a slice is 12 steps (two K=32 sub-steps of six panel-fragment
    // pairs), each of 8 MFMAs.  The pair of step p + 1 is read before the MFMAs of
    // step p, the token fragments of the next sub-step as the last pair's MFMAs
    // release theirs, across slices too, so no MFMA waits for a read issued after
    // a barrier.  The slice's one barrier sits before its last step: every
    // wavefront then holds all of the slice's fragments, so the slice's stage
    // takes the copies of slice kt + 2, and slice kt + 1 has landed.
    static_assert(NSTAGE == 2 && NKS == 2 && NJW == 12 && MI == 4, "K loop layout");
    constexpr int kNP = NJW / 2;                          // pairs per sub-step
    constexpr int kCopies = kAGroupsW + 2 * kWGroupsW;    // copies per wavefront and slice
    const int nk = g.K / BK;             // at least 2 (K is a multiple of 256)
    bf16x8 fa[MI], fb[2][2];
    auto read_pair = [&](int stage, int ks, int jp) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 2 * jp + h;
            const int prow = (j < NJW / 2 ? 0 : BPW / 2) + (j % (NJW / 2)) * MT;
            fb[jp & 1][h] = __builtin_bit_cast(
                bf16x8, *(const u32x4*)(lds + stage * STAGEBW + kpos[ks] + b0 + prow * ROWB));
        }
    };
    auto read_a = [&](int stage, int ks, int i) __attribute__((always_inline)) {
        fa[i] = __builtin_bit_cast(
            bf16x8, *(const u32x4*)(lds + stage * STAGEBW + kpos[ks] + a0 + i * MT * ROWB));
    };
    auto sync = [&]() __attribute__((always_inline)) {
        wait_vmcnt<0>();
        __syncthreads();
    };
    // one slice; NEXT: a slice follows (its first fragments are read here);
    // ISSUE: the slice after that one is copied here
    auto slice = [&](auto NEXT, auto ISSUE, int kt) __attribute__((always_inline)) {
        constexpr bool next = decltype(NEXT)::value, copy = decltype(ISSUE)::value;
        const int st = kt & 1;
#pragma unroll
        for (int p = 0; p < 2 * kNP; ++p) {
            const int ks = p / kNP, jp = p % kNP;
            const bool last = p == 2 * kNP - 1;
            if (last && next) sync();
            if (!last) read_pair(st, (p + 1) / kNP, (p + 1) % kNP);
            else if (next) read_pair(st ^ 1, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    acc[i][2 * jp + h] = mfma_bf16(fb[jp & 1][h], fa[i], acc[i][2 * jp + h]);
                if (jp == kNP - 1 && (!last || next)) {
                    __builtin_amdgcn_sched_barrier(0);
                    read_a(last ? st ^ 1 : st, last ? 0 : 1, i);
                    if (last && copy) issue(st, (kt + 2) * BK, i * kCopies / MI, (i + 1) * kCopies / MI);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    issue(0, 0, 0, kCopies);
    sync();
    issue(1, BK, 0, kCopies);
    if (active) {
#pragma unroll
        for (int i = 0; i < MI; ++i) read_a(0, 0, i);
        read_pair(0, 0, 0);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        int kt = 0;
        for (; kt + 2 < nk; ++kt) slice(C1{}, C1{}, kt);
        slice(C1{}, C0{}, kt);
        slice(C0{}, C0{}, kt + 1);
    } else {
        // only copies, with the same barriers
        for (int kt = 0; kt + 1 < nk; ++kt) {
            sync();
            if (kt + 2 < nk) issue(kt & 1, (kt + 2) * BK, 0, kCopies);
        }
    }
    if (!active) return;
    // H = silu(gate) * up straight from registers (8-byte runs)
    const int ncol0 = 4 * (lane / MT);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int r = wr * WM + i * MT + (lane % MT);
        if (r >= rows) continue;
        bf16_t* orow = g.out + ((int64_t)row0 + r) * g.n_out;
#pragma unroll
        for (int j = 0; j < NJW / 2; ++j) {
            const int col = pn * (BPW / 2) + wc * (WNW / 2) + j * MT + ncol0;
            uint32_t w[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float h0 = silu_f(acc[i][j][2 * h]) * acc[i][j + NJW / 2][2 * h];
                const float h1 = silu_f(acc[i][j][2 * h + 1]) * acc[i][j + NJW / 2][2 * h + 1];
                w[h] = (uint32_t)f32_to_bf16(h0) | ((uint32_t)f32_to_bf16(h1) << 16);
            }
            *(uint2*)(orow + col) = make_uint2(w[0], w[1]);
        }
    }
}

// --------------------------------------------- few rows per expert (decode) --
// With a few routes per expert both GEMMs stream the experts' weights, and what
// matters is bytes in flight.  The tiles above wait for all of a slice's copies at
// its barrier; here a workgroup of four wavefronts takes 64 token rows x 128 panel
// rows (GEMM1: 64 gate rows and the matching 64 up rows) through a ring of three
// 64-K stages, two slices in flight, and two workgroups share a CU (72 KiB of LDS
// each), so copies never stop.  Token rows past 64 are the next blockIdx.y (the
// weights are read again then).  Sums run in the K order of the tiles above, so the
// results are bitwise theirs.
//
// Work order: XCD b % 8 takes a contiguous range of the (tile, panel) list.  With
// the panels dealt round-robin over the XCDs, all resident workgroups (they walk K
// nearly in step) read one contiguous stretch of weights, and where a row is a
// multiple of 8 KiB their copies fell on few memory channels: a layer of 64 tokens,
// d 4096, 64 experts, m 2048 took 664 us against 597 with the tiles, now 567; 128
// experts, d 4096, m 1536 865 (859), now 813; m 4096, d 2048 649 (589), now 567.
// Rows of other lengths: within 3 % (d 3840 538 -> 536).  The parts after the first,
// which only busy experts have, are dealt round-robin, or an XCD whose range holds
// several busy experts would finish last (512 tokens under a sorted Zipf load: 325 us
// round-robin, 434 in ranges).
constexpr int kFewM = 64;           // token rows per workgroup
constexpr int kFewP = 128;          // panel rows
constexpr int kFewStageB = (kFewM + kFewP) * ROWB;      // 24 KiB
constexpr int kFewStages = 3;

template <int MODE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
few_rows_gemm(MfmaArgs g) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kFewStages * kFewStageB];
    const int part = blockIdx.y;             // 64-row part of the tile
    const int L = *g.tile_count * g.ntn;
    int item = blockIdx.x;
    if (part == 0) {                         // the XCD's range
        const int per_xcd = (L + kNumXcd - 1) / kNumXcd;
        const int local = blockIdx.x / kNumXcd;
        if (local >= per_xcd) return;
        item = (blockIdx.x % kNumXcd) * per_xcd + local;
    }
    if (item >= L) return;
    const int tile = item / g.ntn, pn = item % g.ntn;
    const int expert = __builtin_amdgcn_readfirstlane(g.tiles[3 * tile + 0]);
    const int row0 = __builtin_amdgcn_readfirstlane(g.tiles[3 * tile + 1]) + part * kFewM;
    const int rows = min(kFewM, __builtin_amdgcn_readfirstlane(g.tiles[3 * tile + 2]) - part * kFewM);
    if (rows <= 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // copies: panel rows 32 wave .. + 31 (four of 8 rows), token rows 16 wave .. + 15
    // (two, fewer past the tile's end).  Panel row p < 64: gate row 64 pn + p, else up
    // row 64 pn + p - 64 (GEMM2: output row 128 pn + p).
    const bf16_t* wb = (MODE == 0 && wave >= 2 ? g.W1 : g.W0) + (int64_t)expert * g.w_stride;
    const int prow0 = MODE == 0 ? 64 * pn + 32 * (wave & 1) : 128 * pn + 32 * wave;
    uint32_t woff[4], xoff[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 8 * i + lane / 8;
        woff[i] = 2u * (uint32_t)((prow0 + r) * g.K + ((lane % 8) ^ swz(r)) * 8);
    }
    const int nx = max(0, min(2, (rows - 16 * wave + 7) / 8));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = 16 * wave + 8 * i + lane / 8;
        const int q = row0 + min(r, rows - 1);
        const int64_t row = MODE == 0 ? (int64_t)(min(max(g.perm_src[q], 0), g.Tk - 1) / g.k) : q;
        xoff[i] = 2u * (uint32_t)(row * g.K + ((lane % 8) ^ swz(r)) * 8);
    }
    auto issue = [&](int s) __attribute__((always_inline)) {
        unsigned char* st = lds + (s % kFewStages) * kFewStageB;
#pragma unroll
        for (int i = 0; i < 4; ++i) dma16_at(wb + s * BK, woff[i], st + (kFewM + 32 * wave + 8 * i) * ROWB);
        if (nx > 0) dma16_at(g.A + s * BK, xoff[0], st + 16 * wave * ROWB);
        if (nx > 1) dma16_at(g.A + s * BK, xoff[1], st + (16 * wave + 8) * ROWB);
    };
    // slice s has landed, the one after it may still be in flight
    auto wait_one = [&]() __attribute__((always_inline)) {
        if (nx == 2) wait_vmcnt<6>();
        else if (nx == 1) wait_vmcnt<5>();
        else wait_vmcnt<4>();
    };
    const int lrow = lane % 16, grp = lane / 16;
    const int cperm = ((grp & 1) << 1) | (grp >> 1);
    int kpos[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) kpos[ks] = lrow * ROWB + (((4 * ks + cperm) ^ swz(lrow)) << 4);
    // this wavefront's two 16-row panel tiles: gate and up rows 16 wave (GEMM2:
    // output rows 32 wave, + 16)
    const int b0 = (kFewM + (MODE == 0 ? 16 : 32) * wave) * ROWB;
    const int b1 = b0 + (MODE == 0 ? 64 : 16) * ROWB;
    accv acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = accv{0.0f, 0.0f, 0.0f, 0.0f};
    const int mi = (rows + 15) / 16;
    const int nk = g.K / BK;             // at least 2
    issue(0);
    issue(1);
    for (int s = 0; s < nk; ++s) {
        if (s + 1 < nk) wait_one();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        if (s + 2 < nk) issue(s + 2);
        const unsigned char* st = lds + (s % kFewStages) * kFewStageB;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 w0 = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + b0 + kpos[ks]));
            const bf16x8 w1 = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + b1 + kpos[ks]));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i >= mi) continue;
                const bf16x8 x = __builtin_bit_cast(bf16x8, *(const u32x4*)(st + 16 * i * ROWB + kpos[ks]));
                acc[i][0] = mfma_bf16(w0, x, acc[i][0]);
                acc[i][1] = mfma_bf16(w1, x, acc[i][1]);
            }
        }
    }
    // lane l holds outputs 4 (l / 16) .. + 3 of token row l % 16
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 16 * i + lrow;
        if (r >= rows) continue;
        bf16_t* orow = g.out + ((int64_t)row0 + r) * g.n_out;
        uint32_t o[2];
        if (MODE == 0) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float h0 = silu_f(acc[i][0][2 * h]) * acc[i][1][2 * h];
                const float h1 = silu_f(acc[i][0][2 * h + 1]) * acc[i][1][2 * h + 1];
                o[h] = (uint32_t)f32_to_bf16(h0) | ((uint32_t)f32_to_bf16(h1) << 16);
            }
            *(uint2*)(orow + 64 * pn + 16 * wave + 4 * grp) = make_uint2(o[0], o[1]);
        } else {
            const float gw = g.gate[min(max(g.perm_src[row0 + r], 0), g.Tk - 1)];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    o[h] = (uint32_t)f32_to_bf16(gw * acc[i][j][2 * h]) |
                           ((uint32_t)f32_to_bf16(gw * acc[i][j][2 * h + 1]) << 16);
                *(uint2*)(orow + 128 * pn + 32 * wave + 16 * j + 4 * grp) = make_uint2(o[0], o[1]);
            }
        }
    }
}

}  // namespace

bool mfma_shape_ok(const pr2_moe_desc& d) {
    // copy offsets are 32-bit element offsets from the tensor (or expert) base
    const int64_t lim = (int64_t)1 << 31;
    const int64_t Tk = d.T * (int64_t)d.k;
    return d.act_dtype == PR2_BF16 && d.d % BP == 0 && d.m % 128 == 0 && d.d % BK == 0 &&
           d.m % BK == 0 && d.T * (int64_t)d.d < lim && Tk * d.m < lim &&
           (int64_t)d.m * d.d < lim;
}

// The few-rows kernels are taken up to this many routes per expert on average (GEMM1:
// 8 where it would otherwise run the 384-row panel, else 16; GEMM2: 32), from replay
// calls of one layer, both forms in turn on the same buffers, mean of six sets of
// buffers (the tiles' time moves up to 15 % with where the weights lie).  Gain of the
// few-rows form in us of the call under an even load | 8 experts e^3 times as busy
// | a Zipf(1.1) load:
//   d/N/m             routes     tiles             GEMM1               GEMM2
//   2048/128/768          2   244  217  209     9   19   32         17   12   13
//    (384-row panel)      8   265  259  256    11   -2    6         12    8   11
//                        32   297  348  357                         11   10   10
//   4096/128/1536         2   842  658  618    38    4   40         57   36   26
//    (384-row panel)      8   901  899  838    19  -14   -5         39   28   37
//                        32   913 1027 1071                         37   13    7
//   2048/64/1024          8   198  191  194    11   11   11          6    6    6
//                        16   192  207  208     8    0    0          6    1   -1
//                        32   192  217  211                          6   -2   -1
//   2048/64/1408         16   239  248  254    12   -1    9          8   -3   -2
//                        32   255  280  286                          7   -2   10
//   4096/64/2048          8   595  612  601    15   30   28         11   16   17
//                        16   606  623  610    22  -20  -13          9  -13   -5
//                        32   623  659  655                          8  -10   -7
// The limits are where an uneven load begins to lose; an even one gains beyond them.
static bool few_rows_ok(const pr2_moe_desc& d, int routes_per_expert) {
    return d.T * (int64_t)d.k <= (int64_t)routes_per_expert * d.N;
}

static dim3 few_rows_grid(int64_t items) {
    return dim3((unsigned)((items + kNumXcd - 1) / kNumXcd * kNumXcd), kTileM / kFewM);
}

hipError_t launch_expert_gemms(const pr2_moe_desc& d, const void* x, const void* W_gate,
                               const void* W_up, const void* W_down, const float* gate,
                               const ReplayWs& ws, hipStream_t s, void* au_out) {
    if (mfma_shape_ok(d)) {
        MfmaArgs g1{};
        g1.A = (const bf16_t*)x;
        g1.perm_src = ws.perm_src;
        g1.k = d.k;
        g1.Tk = (int)(d.T * d.k);
        g1.W0 = (const bf16_t*)W_gate;
        g1.W1 = (const bf16_t*)W_up;
        g1.K = d.d;
        g1.n_out = d.m;
        g1.ntn = d.m / 128;
        g1.w_stride = (int64_t)d.m * d.d;
        g1.tiles = ws.tiles;
        g1.tile_count = ws.tile_count;
        g1.gate = gate;
        g1.out = (bf16_t*)ws.H;
        int64_t work = ws.max_tiles * g1.ntn;
        int64_t grid = ((work + kNumXcd - 1) / kNumXcd) * kNumXcd;
        if (!au_out && few_rows_ok(d, d.m % (BPW / 2) == 0 ? 8 : 16)) {
            LaunchScope scope("gemm1_few_rows", s);
            g1.ntn = d.m / (kFewP / 2);
            hipLaunchKernelGGL(few_rows_gemm<0>, few_rows_grid(ws.max_tiles * g1.ntn), dim3(256), 0, s, g1);
        } else if (!au_out && d.m % (BPW / 2) == 0) {
            // the 384-row panel: m / 192 panels per tile
            g1.ntn = d.m / (BPW / 2);
            const int64_t wide = ws.max_tiles * g1.ntn;
            const int64_t wgrid = ((wide + kNumXcd - 1) / kNumXcd) * kNumXcd;
            LaunchScope scope("gemm1_gate_up_swiglu", s);
            hipLaunchKernelGGL(gemm1_wide, dim3((unsigned)wgrid), dim3(kGemmThreads), 0, s, g1);
            g1.ntn = d.m / 128;
        } else if (au_out) {
            g1.out2 = (bf16_t*)au_out;
            LaunchScope scope("gemm1_gate_up_swiglu_save", s);
            hipLaunchKernelGGL(grouped_gemm_mfma<3>, dim3((unsigned)grid), dim3(kGemmThreads), 0,
                               s, g1);
        } else {
            LaunchScope scope("gemm1_gate_up_swiglu", s);
            hipLaunchKernelGGL(grouped_gemm_mfma<0>, dim3((unsigned)grid), dim3(kGemmThreads), 0,
                               s, g1);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        MfmaArgs g2 = g1;
        g2.A = (const bf16_t*)ws.H;
        g2.W0 = (const bf16_t*)W_down;
        g2.W1 = nullptr;
        g2.K = d.m;
        g2.n_out = d.d;
        g2.ntn = d.d / BP;
        g2.out = (bf16_t*)ws.O;
        work = ws.max_tiles * g2.ntn;
        grid = ((work + kNumXcd - 1) / kNumXcd) * kNumXcd;
        if (few_rows_ok(d, 32)) {
            LaunchScope scope("gemm2_few_rows", s);
            g2.ntn = d.d / kFewP;
            hipLaunchKernelGGL(few_rows_gemm<1>, few_rows_grid(ws.max_tiles * g2.ntn), dim3(256), 0, s, g2);
        } else {
            LaunchScope scope("gemm2_down_scale", s);
            hipLaunchKernelGGL(grouped_gemm_mfma<1>, dim3((unsigned)grid), dim3(kGemmThreads), 0,
                               s, g2);
        }
        return hipGetLastError();
    }
    hipError_t e = launch_tile_gate_up(d, x, W_gate, W_up, ws, au_out, ws.H, s);
    if (e != hipSuccess) return e;
    return launch_tile_down(d, W_down, gate, ws, s);
}

hipError_t launch_preact(const pr2_moe_desc& d, const void* x, const void* W_gate,
                         const void* W_up, const ReplayWs& ws, void* AU, hipStream_t s) {
    if (mfma_shape_ok(d)) {
        MfmaArgs g{};
        g.A = (const bf16_t*)x;
        g.perm_src = ws.perm_src;
        g.k = d.k;
        g.Tk = (int)(d.T * d.k);
        g.W0 = (const bf16_t*)W_gate;
        g.W1 = (const bf16_t*)W_up;
        g.K = d.d;
        g.n_out = 2 * d.m;
        g.ntn = d.m / 128;
        g.w_stride = (int64_t)d.m * d.d;
        g.tiles = ws.tiles;
        g.tile_count = ws.tile_count;
        g.out = (bf16_t*)AU;
        const int64_t work = ws.max_tiles * g.ntn;
        const int64_t grid = ((work + kNumXcd - 1) / kNumXcd) * kNumXcd;
        LaunchScope scope("bwd_preact_gate_up", s);
        hipLaunchKernelGGL(grouped_gemm_mfma<2>, dim3((unsigned)grid), dim3(kGemmThreads), 0, s, g);
        return hipGetLastError();
    }
    return launch_tile_gate_up(d, x, W_gate, W_up, ws, AU, nullptr, s);
}

}  // namespace pr2
