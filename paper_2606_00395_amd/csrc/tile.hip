// Grouped expert products for the shapes without an MFMA kernel: fp32 layers, and
// bf16 layers whose d is not a multiple of 256 or m not of 128 (gated-MLP
// experts, Appendix E.2, forward and replay backward).
//
// One workgroup of 256 threads forms a 64 x 64 output tile; K advances 32 at a
// time, both operands staged through LDS as fp32, the loads of two steps in
// flight; each thread keeps 4 x 4 outputs and adds in K
// order with one FMA per term, so an output's sum is that of a serial loop.
// These layers are small (the fp32 correctness layer: 512 routes, d 64, m 128), so
// a launch's latency and its serial chain of loads are what they cost; one thread
// per output, each walking its own weight row, took 10 to 40 us per product there,
// these tiles 8 to 17 (the input gradient 38 -> 17), and grew with the size (the
// products of 2800 routes, d = m = 260, 32 experts: 6.8 ms in all, now 0.29).  Loads are 4 elements wide where the rows allow it.
#include <type_traits>

#include "common.h"

namespace pr2 {
namespace {

enum TileMode { T_PRE = 0, T_DOWN = 1, T_DH = 2, T_DX = 3, T_WD = 4, T_WGU = 5 };

constexpr int kT = 64;          // output tile edge
constexpr int kTK = 32;         // K step
constexpr int kLd = kT + 4;     // LDS row (floats)
constexpr int kSub = kTileM / kT;   // sub-tiles per tile-list entry

typedef float f4 __attribute__((ext_vector_type(4)));

struct TileArgs {
    const int* perm_src;
    const int* tiles;
    const int* tile_count;
    const int* offsets;
    int k, d, m, np;
    int vec;                // rows of every operand start 4-element aligned
    const void* x;
    const void* dy;
    const void* Wg;
    const void* Wu;
    const void* Wd;
    const float* gate;
    const void* AUin;       // T_DH
    void* AU;               // T_PRE: a | u out (or null); T_DH: da | du out; T_DX, T_WGU: in
    void* H;                // T_PRE: out (or null); T_DOWN: in; T_DH: g H out; T_WD: in
    void* O;                // T_DOWN, T_DX: out
    float* dgp;
    float* dWg;
    float* dWu;
    float* dWd;
};

// elements i .. i+3 of p where they are below n, else zero
template <typename T>
__device__ __forceinline__ f4 load4(const T* p, int i, int n, bool vec) {
    typedef T v4 __attribute__((ext_vector_type(4)));
    f4 r = {0.0f, 0.0f, 0.0f, 0.0f};
    if (vec) {
        if (i < n) {
            const v4 v = *(const v4*)(p + i);
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = Act<T>::to_f32(v[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + e < n) r[e] = Act<T>::to_f32(p[i + e]);
    }
    return r;
}

template <int MODE, typename T>
__global__ void __launch_bounds__(256) tile_gemm(TileArgs g) {
    constexpr bool kWeight = MODE == T_WD || MODE == T_WGU;     // contracted over routes
    constexpr int NB = MODE == T_PRE ? 2 : 1;                   // B operands (gate and up)
    // B's K runs along its rows in memory (T_PRE, T_DOWN) or across them
    constexpr bool kBCont = MODE == T_PRE || MODE == T_DOWN;
    __shared__ __attribute__((aligned(16))) float As[kTK][kLd];
    __shared__ __attribute__((aligned(16))) float Bs[NB][kTK][kLd];

    int expert, row0, rows, c0, K, ncols, q0 = 0;
    if (kWeight) {
        expert = blockIdx.x;
        q0 = g.offsets[expert];
        K = g.offsets[expert + 1] - q0;
        const int nrow = MODE == T_WD ? g.d : 2 * g.m;
        ncols = MODE == T_WD ? g.m : g.d;
        row0 = blockIdx.y * kT;
        rows = min(kT, nrow - row0);
        c0 = blockIdx.z * kT;
    } else {
        const int tile = blockIdx.x, sub = blockIdx.z;
        if (tile >= *g.tile_count) return;
        rows = min(kT, g.tiles[3 * tile + 2] - sub * kT);
        if (rows <= 0) return;
        expert = g.tiles[3 * tile];
        row0 = g.tiles[3 * tile + 1] + sub * kT;
        c0 = blockIdx.y * kT;
        K = MODE == T_PRE || MODE == T_DH ? g.d : MODE == T_DOWN ? g.m : 2 * g.m;
        ncols = MODE == T_PRE || MODE == T_DH ? g.m : g.d;
    }
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const bool vec = g.vec;
    const int64_t ew = (int64_t)expert * g.m * g.d;
    const int d = g.d, m = g.m;

    // loads: K-contiguous operands by (row r, 8 K values), others by (K row, 8 columns)
    const int lr = tid >> 2, lk = (tid & 3) * 8;
    const int sk = tid >> 3, sc = (tid & 7) * 8;
    // K-contiguous row operand: this thread's row (rows past the end read row 0)
    const T* arow = nullptr;
    if (!kWeight) {
        const int64_t q = row0 + (lr < rows ? lr : 0);
        if (MODE == T_PRE) arow = (const T*)g.x + (int64_t)(g.perm_src[q] / g.k) * d;
        if (MODE == T_DH) arow = (const T*)g.dy + (int64_t)(g.perm_src[q] / g.k) * d;
        if (MODE == T_DOWN) arow = (const T*)g.H + q * m;
        if (MODE == T_DX) arow = (const T*)g.AU + q * 2 * m;
    }
    const T* brow[NB];
    if (kBCont) {
        const int64_t c = min(c0 + lr, ncols - 1);
        if (MODE == T_PRE) {
            brow[0] = (const T*)g.Wg + ew + c * d;
            brow[NB - 1] = (const T*)g.Wu + ew + c * d;
        } else {
            brow[0] = (const T*)g.Wd + ew + c * m;
        }
    }
    // two steps of loads in flight
    f4 rab[2][2], rbb[2][NB][2];
    auto fetch = [&](auto P, int k0) __attribute__((always_inline)) {
        auto& ra = rab[decltype(P)::value];
        auto& rb = rbb[decltype(P)::value];
        int64_t tok = 0;                    // token of this thread's K row (T_WD, T_WGU)
        const bool kin = k0 + sk < K;
        if (kWeight && kin) tok = g.perm_src[q0 + k0 + sk] / g.k;
        const int64_t qk = q0 + k0 + sk;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!kWeight) ra[h] = load4(arow, k0 + lk + 4 * h, K, vec);
            else if (MODE == T_WD)
                ra[h] = load4((const T*)g.dy + tok * d, row0 + sc + 4 * h, kin ? d : 0, vec);
            else
                ra[h] = load4((const T*)g.AU + qk * 2 * m, row0 + sc + 4 * h, kin ? 2 * m : 0, vec);
            if (kBCont) {
#pragma unroll
                for (int b = 0; b < NB; ++b) rb[b][h] = load4(brow[b], k0 + lk + 4 * h, K, vec);
            } else {
                const T* p;
                if (MODE == T_DH) p = (const T*)g.Wd + ew + (int64_t)(k0 + sk) * m;
                if (MODE == T_DX)
                    p = k0 + sk < m ? (const T*)g.Wg + ew + (int64_t)(k0 + sk) * d
                                    : (const T*)g.Wu + ew + (int64_t)(k0 + sk - m) * d;
                if (MODE == T_WD) p = (const T*)g.H + qk * m;
                if (MODE == T_WGU) p = (const T*)g.x + tok * d;
                rb[0][h] = load4(p, c0 + sc + 4 * h, kin ? ncols : 0, vec);
            }
        }
    };
    float acc[NB][4][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[b][u][v] = 0.0f;
    auto step = [&](auto P, int k0) __attribute__((always_inline)) {
        const auto& ra = rab[decltype(P)::value];
        const auto& rb = rbb[decltype(P)::value];
        if (k0) __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!kWeight) {
#pragma unroll
                for (int e = 0; e < 4; ++e) As[lk + 4 * h + e][lr] = ra[h][e];
            } else {
                *(f4*)&As[sk][sc + 4 * h] = ra[h];
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (kBCont) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) Bs[b][lk + 4 * h + e][lr] = rb[b][h][e];
                } else {
                    *(f4*)&Bs[b][sk][sc + 4 * h] = rb[b][h];
                }
            }
        }
        __syncthreads();
        if (k0 + 2 * kTK < K) fetch(P, k0 + 2 * kTK);
        // (K rows past the end are zeros)
#pragma unroll
        for (int kk = 0; kk < kTK; ++kk) {
            const f4 a = *(const f4*)&As[kk][ty * 4];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const f4 w = *(const f4*)&Bs[b][kk][tx * 4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[b][u][v] = fmaf(a[u], w[v], acc[b][u][v]);
            }
        }
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    if (K > 0) fetch(P0{}, 0);
    if (K > kTK) fetch(P1{}, kTK);
    for (int k0 = 0; k0 < K; k0 += 2 * kTK) {
        step(P0{}, k0);
        if (k0 + kTK < K) step(P1{}, k0 + kTK);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = ty * 4 + u;
        const bool rin = r < rows;
        const int64_t q = row0 + r;
        float gq = 0.0f;
        if ((MODE == T_DOWN || MODE == T_DH) && rin) gq = g.gate[g.perm_src[q]];
        float part = 0.0f;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = c0 + tx * 4 + v;
            if (!rin || c >= ncols) continue;
            const float s = acc[0][u][v];
            if (MODE == T_PRE) {
                const float up = acc[NB - 1][u][v];
                if (g.AU) {
                    T* o = (T*)g.AU + q * 2 * m;
                    o[c] = Act<T>::from_f32(s);
                    o[m + c] = Act<T>::from_f32(up);
                }
                if (g.H) ((T*)g.H)[q * m + c] = Act<T>::from_f32(s / (1.0f + expf(-s)) * up);
            } else if (MODE == T_DOWN) {
                ((T*)g.O)[q * d + c] = Act<T>::from_f32(gq * s);
            } else if (MODE == T_DH) {
                const T* ain = (const T*)g.AUin + q * 2 * m;
                T* au = (T*)g.AU + q * 2 * m;
                float da, du, hg, hG;
                swiglu_bwd<sizeof(T) == 2>(Act<T>::to_f32(ain[c]), Act<T>::to_f32(ain[m + c]), s, gq, da,
                                           du, hg, hG);
                au[c] = Act<T>::from_f32(da);
                au[m + c] = Act<T>::from_f32(du);
                ((T*)g.H)[q * m + c] = Act<T>::from_f32(hg);
                part += hG;
            } else if (MODE == T_DX) {
                ((T*)g.O)[q * d + c] = Act<T>::from_f32(s);
            } else if (MODE == T_WD) {
                g.dWd[ew + (int64_t)q * m + c] = s;
            } else {
                if (q < m) g.dWg[ew + q * d + c] = s;
                else g.dWu[ew + (q - m) * d + c] = s;
            }
        }
        if (MODE == T_DH) {
            // the row's sum over this tile's 64 columns (16 lanes, 4 each)
            for (int off = 8; off >= 1; off >>= 1) part += __shfl_xor(part, off, 16);
            if (tx == 0 && rin) g.dgp[q * g.np + blockIdx.y] = part;
        }
    }
}

TileArgs tile_args(const pr2_moe_desc& d, const ReplayWs& ws) {
    TileArgs g{};
    g.perm_src = ws.perm_src;
    g.tiles = ws.tiles;
    g.tile_count = ws.tile_count;
    g.offsets = ws.offsets;
    g.k = d.k;
    g.d = d.d;
    g.m = d.m;
    g.vec = d.d % 4 == 0 && d.m % 4 == 0;
    return g;
}

template <int MODE>
hipError_t launch_tile(const pr2_moe_desc& d, const ReplayWs& ws, const TileArgs& g,
                       const char* name, hipStream_t s) {
    auto tiles = [](int64_t n) { return (unsigned)((n + kT - 1) / kT); };
    dim3 grid;
    if (MODE == T_WD) grid = dim3((unsigned)d.N, tiles(d.d), tiles(d.m));
    else if (MODE == T_WGU) grid = dim3((unsigned)d.N, tiles(2 * (int64_t)d.m), tiles(d.d));
    else
        grid = dim3((unsigned)ws.max_tiles, tiles(MODE == T_PRE || MODE == T_DH ? d.m : d.d), kSub);
    LaunchScope scope(name, s);
    if (d.act_dtype == PR2_BF16)
        hipLaunchKernelGGL((tile_gemm<MODE, bf16_t>), grid, dim3(256), 0, s, g);
    else
        hipLaunchKernelGGL((tile_gemm<MODE, float>), grid, dim3(256), 0, s, g);
    return hipGetLastError();
}

}  // namespace

int tile_partials(const pr2_moe_desc& d) { return (d.m + kT - 1) / kT; }

hipError_t launch_tile_gate_up(const pr2_moe_desc& d, const void* x, const void* W_gate,
                               const void* W_up, const ReplayWs& ws, void* AU, void* H,
                               hipStream_t s) {
    TileArgs g = tile_args(d, ws);
    g.x = x;
    g.Wg = W_gate;
    g.Wu = W_up;
    g.AU = AU;
    g.H = H;
    return launch_tile<T_PRE>(d, ws, g, H ? "gemm1_tile" : "bwd_preact_tile", s);
}

hipError_t launch_tile_down(const pr2_moe_desc& d, const void* W_down, const float* gate,
                            const ReplayWs& ws, hipStream_t s) {
    TileArgs g = tile_args(d, ws);
    g.Wd = W_down;
    g.gate = gate;
    g.H = ws.H;
    g.O = ws.O;
    return launch_tile<T_DOWN>(d, ws, g, "gemm2_tile", s);
}

hipError_t launch_tile_dh(const pr2_moe_desc& d, const void* dy, const void* W_down,
                          const float* gate, const BwdWs& ws, const void* au_in, hipStream_t s) {
    TileArgs g = tile_args(d, ws.fw);
    g.np = ws.np;
    g.dy = dy;
    g.Wd = W_down;
    g.gate = gate;
    g.AUin = au_in ? au_in : ws.AU;
    g.AU = ws.AU;
    g.H = ws.fw.H;
    g.dgp = ws.dgp;
    return launch_tile<T_DH>(d, ws.fw, g, "bwd_dh_tile", s);
}

hipError_t launch_tile_grads(const pr2_moe_desc& d, const void* x, const void* W_gate,
                             const void* W_up, const void* dy, const BwdWs& ws,
                             const BwdGrads& out, hipStream_t s) {
    TileArgs g = tile_args(d, ws.fw);
    g.x = x;
    g.dy = dy;
    g.Wg = W_gate;
    g.Wu = W_up;
    g.AU = ws.AU;
    g.H = ws.fw.H;
    g.O = ws.fw.O;
    g.dWg = out.dW_gate;
    g.dWu = out.dW_up;
    g.dWd = out.dW_down;
    hipError_t e = launch_tile<T_DX>(d, ws.fw, g, "bwd_dx_tile", s);
    if (e == hipSuccess) e = launch_tile<T_WD>(d, ws.fw, g, "bwd_wd_tile", s);
    if (e == hipSuccess) e = launch_tile<T_WGU>(d, ws.fw, g, "bwd_wgu_tile", s);
    return e;
}

}  // namespace pr2
