// Evolution-predictor training on the feature cache (Sec. 4.2, Eq. pr2_loss;
// Alg. 3 in Appendix D, its predictive-loss steps), for the cached tokens t:
//
//   p_t       = h_t W_r + b_r                  current router (the teacher, no gradient)
//   u_t       = h_old,t A,  b_t = u_t B        predictor residual, W_p = A B
//   standard:  KL(softmax(p_t) || softmax(p_old,t + b_t))
//   delta:     KL(softmax(p_t - p_old,t) || softmax(b_t))   (Appendix G ablation)
//   loss = mean_t KL,  dz_t = (softmax(zhat_t) - target_t) / T
//   dB = sum_t u_t^T dz_t,  dA = sum_t h_old,t^T (dz_t B^T)
//
// p comes from the replay router kernels (exact products, one rounding to fp32).
// Everything after it runs in fp64.  bf16 features of the models' shapes take
// three launches (pred_token, pred_grad, pred_finish; below).  Elsewhere the three
// products u = h_old A, dB = u^T dz and dA = h_old^T w go through one tiled kernel:
// a workgroup forms a 64 x 16 output tile over one slice of the summed index,
// staging both operands through LDS as fp64, and a second kernel adds the slices in
// slice order; the two softmaxes, the KL and dz take one wavefront per token.  All
// sums are deterministic (no atomics).
#include <algorithm>

#include "common.h"

namespace pr2 {
namespace {

constexpr int kMaxVals = kMaxExperts / 64;

__device__ __forceinline__ double wsum(double v) {
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}
__device__ __forceinline__ double wmax(double v) {
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ double to_f64(bf16_t v) { return (double)Act<bf16_t>::to_f32(v); }
__device__ __forceinline__ double to_f64(float v) { return (double)v; }
__device__ __forceinline__ double to_f64(double v) { return v; }

constexpr int kPM = 64, kPN = 16, kPK = 32;     // output tile and staged slice of the sum

// C[m][n] = sum_k a(m, k) b(k, n), operands addressed through strides:
// a(m, k) = a[m*a_m + k*a_k], b(k, n) = b[k*b_k + n*b_n].
struct ProdArgs {
    const void* a;
    int64_t a_m, a_k;
    const void* b;
    int64_t b_k, b_n;
    int M, Nc;
    int64_t K, kslice;
    double* part;       // [slices][M][Nc]
};

// workgroup (m tile, n tile, slice); thread (tm, tn) keeps rows 4tm..4tm+3 of column tn
template <typename TA, typename TB>
__global__ void __launch_bounds__(256) prod_f64_kernel(ProdArgs p) {
    __shared__ double sa[kPK][kPM + 1];
    __shared__ double sb[kPK][kPN];
    const int tid = threadIdx.x;
    const int tn = tid & 15, tm = tid >> 4;
    const int m0 = blockIdx.x * kPM, n0 = blockIdx.y * kPN;
    const int64_t k0 = (int64_t)blockIdx.z * p.kslice;
    const int64_t k1 = min(p.K, k0 + p.kslice);
    const TA* a = (const TA*)p.a;
    const TB* b = (const TB*)p.b;
    const bool a_kfast = p.a_k == 1;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t kc = k0; kc < k1; kc += kPK) {
        for (int e = tid; e < kPM * kPK; e += 256) {
            const int kk = a_kfast ? (e & (kPK - 1)) : e / kPM;
            const int mm = a_kfast ? e / kPK : (e & (kPM - 1));
            const int64_t k = kc + kk;
            const int m = m0 + mm;
            sa[kk][mm] = (m < p.M && k < k1) ? to_f64(a[(int64_t)m * p.a_m + k * p.a_k]) : 0.0;
        }
        for (int e = tid; e < kPN * kPK; e += 256) {
            const int kk = e / kPN, nn = e & (kPN - 1);
            const int64_t k = kc + kk;
            const int n = n0 + nn;
            sb[kk][nn] = (n < p.Nc && k < k1) ? to_f64(b[k * p.b_k + (int64_t)n * p.b_n]) : 0.0;
        }
        __syncthreads();
#pragma unroll 8
        for (int kk = 0; kk < kPK; ++kk) {
            const double bv = sb[kk][tn];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = fma(sa[kk][tm * 4 + i], bv, acc[i]);
        }
        __syncthreads();
    }
    const int n = n0 + tn;
    if (n >= p.Nc) return;
    double* out = p.part + (int64_t)blockIdx.z * p.M * p.Nc;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + tm * 4 + i;
        if (m < p.M) out[(int64_t)m * p.Nc + n] = acc[i];
    }
}

// out[e] = sum over slices of part[s][e], slice order
template <typename OT>
__global__ void __launch_bounds__(256)
sum_slices_kernel(const double* part, int slices, int64_t n, OT* out) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    double acc = 0.0;
    int s = 0;
    for (; s + 8 <= slices; s += 8) {       // eight loads in flight, added in slice order
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = part[(int64_t)(s + i) * n + e];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += v[i];
    }
    for (; s < slices; ++s) acc += part[(int64_t)s * n + e];
    out[e] = (OT)acc;
}

// slices of the summed index: about 1024 workgroups in all, each slice a whole
// number of staged chunks, at most 64 slices
int64_t prod_kslice(int M, int Nc, int64_t K) {
    const int64_t tiles = (int64_t)((M + kPM - 1) / kPM) * ((Nc + kPN - 1) / kPN);
    const int64_t chunks = (K + kPK - 1) / kPK;
    int64_t s = (1024 + tiles - 1) / tiles;
    s = std::max<int64_t>(1, std::min<int64_t>({s, chunks, 64}));
    return std::max<int64_t>(1, (chunks + s - 1) / s) * kPK;
}

int prod_slices(int M, int Nc, int64_t K) {
    return (int)std::max<int64_t>(1, (K + prod_kslice(M, Nc, K) - 1) / prod_kslice(M, Nc, K));
}

template <typename TA, typename TB, typename OT>
hipError_t launch_prod(const TA* a, int64_t a_m, int64_t a_k, const TB* b, int64_t b_k,
                       int64_t b_n, int M, int Nc, int64_t K, double* part, OT* out,
                       hipStream_t s) {
    if (M <= 0 || Nc <= 0) return hipSuccess;
    ProdArgs p{a, a_m, a_k, b, b_k, b_n, M, Nc, K, prod_kslice(M, Nc, K), part};
    const int slices = prod_slices(M, Nc, K);
    dim3 grid((unsigned)((M + kPM - 1) / kPM), (unsigned)((Nc + kPN - 1) / kPN), (unsigned)slices);
    hipLaunchKernelGGL((prod_f64_kernel<TA, TB>), grid, dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)M * Nc;
    hipLaunchKernelGGL(sum_slices_kernel<OT>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       part, slices, n, out);
    return hipGetLastError();
}

// ------------------------------------------------------ three-launch path ----
// bf16 features, rank <= 64, N <= 192, d % 64 == 0 (the models' shapes): three
// launches after the router logits instead of eight, all sums in fp64.  What these
// 16 MB of operands cost is latency: each launch's chain of dependent loads and
// barriers (2048 tokens, d 2048, N 128, r 16: 73 us in eight launches, 36 in three).
// u runs on the vector ALU: its fp64 matrix instructions (16x16x4), issued once in
// about 226 clocks, made the token kernel 27 us instead of 20.
//
// Limits: d % 64 is the token kernel's K step (8 values for each of 8 lane groups);
// the kernel's LDS is sized for r <= 64.  Above 192 columns the logits have no MFMA
// form and take nearly all of the call (2048 tokens, d 2048, N 256, r 16: 1341 us in
// eight launches, 1290 with this path), so it ends where that form ends.  Calls in
// eight launches | in three, us: d 2048, N 128, r 16 51 | 33 at 1 token, 73 | 49 at
// 512, 104 | 60 at 2048, 807 | 464 at 32768; d 2048, N 128, r 1 55 | 43 at 512; d
// 4096, N 128, r 64 112 | 107 at 64, 362 | 206 at 2048; d 1024, N 192, r 32 73 | 40
// at 1, 1026 | 543 at 32768.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
// four floats of a tensor that is only promised to start at a 4-byte boundary (A); the
// load is still one 16-byte instruction
typedef f4 f4_unaligned __attribute__((aligned(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kPTok = 8;            // tokens per workgroup, one wavefront each
// Fewest tokens per slice of the gradient sums, and most slices.  A slice is a serial
// chain of loads and MFMAs, and its partial sums are written and read once.  Whole call
// in us with (tokens, slices) of (64, 64) | (32, 64) | (128, 64) | (64, 32) | (64, 128):
// d 2048, N 128, r 16 43 | 40 | 48 | 43 | 43 at 300 tokens, 60 | 61 | 67 | 60 | 60 at
// 2048 (a response's feature cache, the usual size), 233 | 233 | 233 | 246 | 223 at 16384;
// d 4096, N 128, r 64 136 | 136 | 141 | 136 | 136, 206 | 220 | 207 | 206 | 206 and 1213 |
// 1212 | 1213 | 1196 | 1253 (134 MB of partial sums at 64 slices, and 128 add more).
constexpr int kGradTok = 64;
constexpr int kGradSlices = 64;

// value e (0..7) of 8 consecutive bf16
__device__ __forceinline__ double bf8(u32x4 v, int e) {
    return (double)__uint_as_float(e & 1 ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16);
}

struct TokenArgs {
    const bf16_t* h_old;    // [T, d]
    const float* A;         // [d, r]
    const float* B;         // [r, N]
    const float* p_cur;     // [T, N]
    const float* p_old;     // [T, N]
    int64_t T;
    int d, N, r, kind;
    float* kl_out;          // [T] or null
    double* kl;             // [T]
    double* u;              // [T, r]
    double* dz;             // [T, N]
    double* w;              // [T, r]
};

// Eight tokens: u = h_old A, b = u B, the two softmaxes, KL and dz (one wavefront
// per token), w = dz B^T.  For u a lane keeps 4 tokens x 4 columns of a 16-column
// tile over an eighth of its wavefront's K values, and the 64 parts are added in
// order through LDS.  RT: 16-column tiles of the rank; V64: of 64 experts.
template <int RT, int V64>
__global__ void __launch_bounds__(64 * kPTok) pred_token_kernel(TokenArgs a) {
    constexpr int R = 16 * RT, NP = 64 * V64;
    constexpr int kParts = 8 * kPTok;
    __shared__ __attribute__((aligned(16))) double red[kParts][kPTok * 16];
    __shared__ double red2[4][kPTok * 16];
    __shared__ double su[kPTok][R];
    __shared__ double sz[kPTok][NP];
    __shared__ float sB[R][NP + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * kPTok;
    const int d = a.d, N = a.N, r = a.r;
    const int64_t t = t0 + wave;                    // this wavefront's token
    const int64_t tc = min(t, a.T - 1);

    float pold[V64], pcur[V64];
#pragma unroll
    for (int v = 0; v < V64; ++v) {
        const int64_t e = tc * N + min(64 * v + lane, N - 1);
        pold[v] = a.p_old[e];
        pcur[v] = a.p_cur[e];
    }
    for (int e = tid; e < R * NP; e += 64 * kPTok) {
        const int q = e / NP, j = e % NP;
        sB[q][j] = q < r && j < N ? a.B[(int64_t)q * N + j] : 0.0f;
    }
    const int bt = lane & 1, bq = (lane >> 1) & 3, kg = lane >> 3;
    const bf16_t* hrow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) hrow[i] = a.h_old + min(t0 + 4 * bt + i, a.T - 1) * d;
    const bool vec = r % 4 == 0;
#pragma unroll 1
    for (int qt = 0; qt < RT; ++qt) {
        const int q0 = 16 * qt + 4 * bq;
        double acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
#pragma unroll 2
        for (int k0 = 64 * wave + 8 * kg; k0 < d; k0 += 64 * kPTok) {
            u32x4 h[4];
            f4 av[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = *(const u32x4*)(hrow[i] + k0);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float* p = a.A + (int64_t)(k0 + k) * r;
                av[k] = f4{0.0f, 0.0f, 0.0f, 0.0f};
                if (vec) {
                    if (q0 < r) av[k] = *(const f4_unaligned*)(p + q0);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (q0 + j < r) av[k][j] = p[q0 + j];
                }
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                double x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = bf8(h[i], k);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double y = (double)av[k][j];
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i][j] = fma(x[i], y, acc[i][j]);
                }
            }
        }
        if (qt) __syncthreads();
        double* part = red[wave * 8 + kg];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; j += 2)
                *(d2*)(part + (4 * bt + i) * 16 + 4 * bq + j) = d2{acc[i][j], acc[i][j + 1]};
        __syncthreads();
        {
            const int o = tid & 127, pg = tid >> 7;
            double s = 0.0;
#pragma unroll
            for (int p = 0; p < kParts / 4; ++p) s += red[pg * (kParts / 4) + p][o];
            red2[pg][o] = s;
        }
        __syncthreads();
        if (tid < kPTok * 16) {
            const double s = ((red2[0][tid] + red2[1][tid]) + red2[2][tid]) + red2[3][tid];
            const int tok = tid >> 4, q = 16 * qt + (tid & 15);
            su[tok][q] = s;
            if (t0 + tok < a.T && q < r) a.u[(t0 + tok) * r + q] = s;
        }
    }
    __syncthreads();
    {
        double zh[V64], tl[V64], mz = -INFINITY, mt = -INFINITY;
#pragma unroll
        for (int v = 0; v < V64; ++v) zh[v] = 0.0;
#pragma unroll 4
        for (int q = 0; q < r; ++q) {
            const double uq = su[wave][q];
#pragma unroll
            for (int v = 0; v < V64; ++v) zh[v] = fma(uq, (double)sB[q][64 * v + lane], zh[v]);
        }
#pragma unroll
        for (int v = 0; v < V64; ++v) {
            tl[v] = -INFINITY;
            if (64 * v + lane < N) {
                const double po = (double)pold[v], pc = (double)pcur[v];
                if (a.kind == 0) zh[v] += po;
                tl[v] = a.kind == 0 ? pc : pc - po;
                mz = fmax(mz, zh[v]);
                mt = fmax(mt, tl[v]);
            }
        }
        mz = wmax(mz);
        mt = wmax(mt);
        double ez[V64], et[V64], sumz = 0.0, sumt = 0.0;
#pragma unroll
        for (int v = 0; v < V64; ++v) {
            ez[v] = et[v] = 0.0;
            if (64 * v + lane < N) {
                ez[v] = exp(zh[v] - mz);
                et[v] = exp(tl[v] - mt);
                sumz += ez[v];
                sumt += et[v];
            }
        }
        sumz = wsum(sumz);
        sumt = wsum(sumt);
        // KL = sum_j e_j / sumt * ((t_j - z_j) - shift)
        const double shift = (mt + log(sumt)) - (mz + log(sumz));
        const double iz = 1.0 / (sumz * (double)a.T), it = 1.0 / (sumt * (double)a.T);
        double kl = 0.0;
#pragma unroll
        for (int v = 0; v < V64; ++v) {
            const int j = 64 * v + lane;
            double dzv = 0.0;
            if (j < N) {
                kl += et[v] * ((tl[v] - zh[v]) - shift);
                dzv = ez[v] * iz - et[v] * it;
                if (t < a.T) a.dz[t * N + j] = dzv;
            }
            sz[wave][j] = dzv;
        }
        kl = wsum(kl) / sumt;
        if (lane == 0 && t < a.T) {
            a.kl[t] = kl;
            if (a.kl_out) a.kl_out[t] = (float)kl;
        }
    }
    // w: the token's wavefront, column lane / 4 of each 16, four parts of the sum
    // (the wavefront's own row of sz: LDS operations of one wavefront are in order)
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int qt = 0; qt < RT; ++qt) {
        const int q = 16 * qt + (lane >> 2);
        double s = 0.0;
#pragma unroll 8
        for (int n = 0; n < NP / 4; ++n) {
            const int j = 4 * n + (lane & 3);
            s = fma(sz[wave][j], (double)sB[q][j], s);
        }
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        if ((lane & 3) == 0 && t < a.T && q < r) a.w[t * r + q] = s;
    }
}

struct GradArgs {
    const bf16_t* h_old;
    const double* u;
    const double* dz;
    const double* w;
    int64_t T, tps;         // tokens, tokens per slice
    int d, N, r;
    int na, nb;             // wavefront tasks of dA and dB per slice
    double* pa;             // [slices][d][r]
    double* pb;             // [slices][r][N]
};

// Sums over one slice of the tokens, on v_mfma_f64_16x16x4_f64: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16], its result v is C[l / 16 + 4 v][l % 16].
// dA = h_old^T w: a wavefront takes 128 rows of d (a lane's 16-byte load holds one
// row of eight 16-row tiles) by 16 columns; dB = u^T dz: 16 rows of r by 128 columns.
// (As vector FMAs over 8 x 4 outputs per lane: 24 us against 12, its partial sums
// stored in 32-byte pieces.)
typedef double d4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__global__ void __launch_bounds__(256) pred_grad_kernel(GradArgs a) {
    const int lane = threadIdx.x & 63;
    const int task = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (task >= a.na + a.nb) return;
    const int il = lane & 15, g = lane >> 4;
    const int64_t slice = blockIdx.y;
    const int64_t s0 = slice * a.tps, s1 = min(a.T, s0 + a.tps);
    const int d = a.d, N = a.N, r = a.r;
    const int rt = (r + 15) / 16;
    constexpr int kU = 8, kUB = 4;      // K steps whose loads go out together
    d4 acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = d4{0.0, 0.0, 0.0, 0.0};
    if (task < a.na) {
        const int q = task % rt * 16 + il, i0 = task / rt * 128;
        const bool cin = i0 + 8 * il < d, qin = q < r;
        for (int64_t ts = s0; ts < s1; ts += 4 * kU) {
            u32x4 x[kU];
            double w[kU];
#pragma unroll
            for (int k = 0; k < kU; ++k) {
                const int64_t t = ts + 4 * k + g;
                x[k] = t < s1 && cin ? *(const u32x4*)(a.h_old + t * d + i0 + 8 * il)
                                     : u32x4{0u, 0u, 0u, 0u};
                w[k] = t < s1 && qin ? a.w[t * r + q] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < kU; ++k)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = mfma_f64(bf8(x[k], j), w[k], acc[j]);
        }
        if (!qin) return;
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int i = i0 + 8 * (g + 4 * v) + j;
                if (i < d) a.pa[(slice * d + i) * r + q] = acc[j][v];
            }
    } else {
        const int tb = task - a.na;
        const int q0 = tb % rt * 16, j0 = tb / rt * 128;
        for (int64_t ts = s0; ts < s1; ts += 4 * kUB) {
            double uv[kUB], z[kUB][8];
#pragma unroll
            for (int k = 0; k < kUB; ++k) {
                const int64_t t = ts + 4 * k + g;
                const bool tin = t < s1;
                uv[k] = tin && q0 + il < r ? a.u[t * r + q0 + il] : 0.0;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int c = j0 + 16 * j + il;
                    z[k][j] = tin && c < N ? a.dz[t * N + c] : 0.0;
                }
            }
#pragma unroll
            for (int k = 0; k < kUB; ++k)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = mfma_f64(uv[k], z[k][j], acc[j]);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int q = q0 + g + 4 * v, c = j0 + 16 * j + il;
                if (q < r && c < N) a.pb[(slice * r + q) * N + c] = acc[j][v];
            }
    }
}

// dA and dB: the slices added in order (eight loads in flight); the last
// workgroup: the mean of kl in a fixed order
__global__ void __launch_bounds__(256)
pred_finish_kernel(const double* pa, int64_t na, int ba, const double* pb, int64_t nb, int bb,
                   int slices, float* dA, float* dB, const double* kl, int64_t T, float* loss) {
    __shared__ double s[256];
    const int b = blockIdx.x;
    if (b < ba + bb) {
        const bool first = b < ba;
        const int64_t e = (int64_t)(first ? b : b - ba) * 256 + threadIdx.x;
        const int64_t n = first ? na : nb;
        const double* part = first ? pa : pb;
        if (e >= n) return;
        double acc = 0.0;
        int i = 0;
        for (; i + 8 <= slices; i += 8) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = part[(int64_t)(i + k) * n + e];
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += v[k];
        }
        for (; i < slices; ++i) acc += part[(int64_t)i * n + e];
        (first ? dA : dB)[e] = (float)acc;
        return;
    }
    double acc = 0.0;
    for (int64_t t = threadIdx.x; t < T; t += 256) acc += kl[t];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = (float)(s[0] / (double)T);
}

int grad_slices(int64_t T) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(kGradSlices, (T + kGradTok - 1) / kGradTok));
}

bool pred_three_ok(const pr2_moe_desc& d) {
    return d.act_dtype == PR2_BF16 && d.d % 64 == 0 && d.r <= 64 && d.N <= 192;
}

template <int RT>
void launch_pred_token(const TokenArgs& t, hipStream_t s) {
    const dim3 grid((unsigned)((t.T + kPTok - 1) / kPTok)), block(64 * kPTok);
    if (t.N <= 64) hipLaunchKernelGGL((pred_token_kernel<RT, 1>), grid, block, 0, s, t);
    else if (t.N <= 128) hipLaunchKernelGGL((pred_token_kernel<RT, 2>), grid, block, 0, s, t);
    else hipLaunchKernelGGL((pred_token_kernel<RT, 3>), grid, block, 0, s, t);
}

struct LossArgs {
    const float* p_cur;     // [T, N]
    const float* p_old;     // [T, N]
    const double* u;        // [T, r]
    const float* B;         // [r, N] or null (identity, r == N)
    int64_t T;
    int N, r, kind;
    float* kl_out;          // [T] or null
    double* kl;             // [T]
    double* dz;             // [T, N]
    double* w;              // [T, r]  dz B^T (unused for the identity)
};

constexpr int kLdsB = 4096;      // B entries staged in LDS (r N <= 4096)

// one wavefront per token; B in LDS and the token's u in lanes when they fit
__global__ void __launch_bounds__(256) pred_loss_kernel(LossArgs a) {
    __shared__ float sB[kLdsB];
    const int N = a.N, r = a.r;
    const bool b_lds = a.B && r * N <= kLdsB;
    if (b_lds) {
        for (int e = threadIdx.x; e < r * N; e += 256) sB[e] = a.B[e];
        __syncthreads();
    }
    const float* Bm = b_lds ? sB : a.B;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (t >= a.T) return;
    const int nv = (N + 63) / 64;
    const double* ut = a.u + t * r;
    const bool u_lanes = r <= 64;
    const double ul = (u_lanes && lane < r) ? ut[lane] : 0.0;
    double zh[kMaxVals], tl[kMaxVals];
    double mz = -INFINITY, mt = -INFINITY;
    for (int v = 0; v < nv; ++v) {
        const int j = v * 64 + lane;
        const int jc = j < N ? j : N - 1;       // every lane takes part in the shuffles
        double b = 0.0;
        if (a.B) {
            for (int q = 0; q < r; ++q)
                b = fma(u_lanes ? __shfl(ul, q, 64) : ut[q], (double)Bm[(int64_t)q * N + jc], b);
        } else {
            b = ut[jc];
        }
        zh[v] = -INFINITY;
        tl[v] = -INFINITY;
        if (j < N) {
            const double po = (double)a.p_old[t * N + j];
            const double pc = (double)a.p_cur[t * N + j];
            zh[v] = a.kind == 0 ? po + b : b;
            tl[v] = a.kind == 0 ? pc : pc - po;
            mz = fmax(mz, zh[v]);
            mt = fmax(mt, tl[v]);
        }
    }
    mz = wmax(mz);
    mt = wmax(mt);
    double sz = 0.0, st = 0.0;
    for (int v = 0; v < nv; ++v) {
        if (v * 64 + lane < N) {
            sz += exp(zh[v] - mz);
            st += exp(tl[v] - mt);
        }
    }
    sz = wsum(sz);
    st = wsum(st);
    const double lsz = log(sz), lst = log(st);
    double kl = 0.0;
    for (int v = 0; v < nv; ++v) {
        const int j = v * 64 + lane;
        if (j < N) {
            const double lt = tl[v] - mt - lst;         // log target
            const double lh = zh[v] - mz - lsz;         // log rho_hat
            const double tg = exp(lt);
            kl += tg * (lt - lh);
            const double g = (exp(lh) - tg) / (double)a.T;
            a.dz[t * N + j] = g;
            zh[v] = g;                                  // keep dz for the B^T product
        }
    }
    kl = wsum(kl);
    if (lane == 0) {
        a.kl[t] = kl;
        if (a.kl_out) a.kl_out[t] = (float)kl;
    }
    if (a.B) {
        for (int q = 0; q < r; ++q) {
            double part = 0.0;
            for (int v = 0; v < nv; ++v) {
                const int j = v * 64 + lane;
                if (j < N) part = fma(zh[v], (double)Bm[(int64_t)q * N + j], part);
            }
            part = wsum(part);
            if (lane == (q & 63)) a.w[t * r + q] = part;
        }
    }
}

// loss = mean of kl, fixed-order reduction in one block
__global__ void __launch_bounds__(256) mean_kernel(const double* kl, int64_t T, float* out) {
    __shared__ double s[256];
    double acc = 0.0;
    for (int64_t t = threadIdx.x; t < T; t += 256) acc += kl[t];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = T > 0 ? (float)(s[0] / (double)T) : 0.0f;
}

__global__ void __launch_bounds__(256) fill_f32_kernel(float* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        p[i] = 0.0f;
}

hipError_t fill0(float* p, int64_t n, hipStream_t s) {
    if (!p || n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

}  // namespace

// Partial sums of the three products.  The u product's slice count falls as
// its row tiles grow, so its part is bounded by a size that does not decrease
// with T (slices <= 1024 / tiles + 1 with tiles >= T ntiles / 64, and
// slices <= min(64, K chunks)): a workspace sized for a batch serves every
// smaller one.
size_t predictor_partial_doubles(const pr2_moe_desc& d) {
    const int64_t T = d.T;
    const int64_t ntiles = (d.r + kPN - 1) / kPN;
    const int64_t su_max = std::min<int64_t>(64, std::max<int64_t>(1, (d.d + kPK - 1) / kPK));
    const size_t pu = (size_t)std::min<int64_t>(su_max * T, 1024 * kPM / ntiles + T) * d.r;
    const size_t pb = (size_t)prod_slices(d.r, d.N, T) * (size_t)d.r * d.N;
    const size_t pa = (size_t)prod_slices(d.d, d.r, T) * (size_t)d.d * d.r;
    size_t pm = 0;
    if (pred_three_ok(d))
        pm = (size_t)grad_slices(T) * ((size_t)d.d * d.r + (size_t)d.r * d.N);
    return std::max({pu, pb, pa, pm});
}

hipError_t launch_predictor_zero(const pr2_moe_desc& d, float* kl_out, float* loss_out, float* dA,
                                 float* dB, hipStream_t s) {
    LaunchScope scope("predictor_loss_skip", s);
    hipError_t e;
    if ((e = fill0(kl_out, d.T, s)) != hipSuccess) return e;
    if ((e = fill0(loss_out, 1, s)) != hipSuccess) return e;
    if ((e = fill0(dA, (int64_t)d.d * d.r, s)) != hipSuccess) return e;
    return fill0(dB, (int64_t)d.r * d.N, s);
}

hipError_t launch_predictor_loss(const pr2_moe_desc& d, const void* h, const float* W_r,
                                 const float* b_r, const void* h_old, const float* p_old,
                                 const float* A, const float* B, int kind, float* kl_out,
                                 float* loss_out, float* dA, float* dB, const PredLossWs& ws,
                                 hipStream_t s) {
    hipError_t e = launch_router_logits(d, h, W_r, b_r, ws.p_cur, ws.wsplit, s);
    if (e != hipSuccess) return e;
    const bool bf = d.act_dtype == PR2_BF16;
    if (B && pred_three_ok(d)) {
        const TokenArgs t{(const bf16_t*)h_old, A, B, ws.p_cur, p_old, d.T, d.d, d.N, d.r, kind,
                          kl_out, ws.kl, ws.u, ws.dz, ws.w};
        {
            LaunchScope scope("predictor_token", s);
            switch ((d.r + 15) / 16) {
                case 1: launch_pred_token<1>(t, s); break;
                case 2: launch_pred_token<2>(t, s); break;
                case 3: launch_pred_token<3>(t, s); break;
                default: launch_pred_token<4>(t, s); break;
            }
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const int slices = grad_slices(d.T);
        const int rt = (d.r + 15) / 16;
        const int64_t na = (int64_t)d.d * d.r, nb = (int64_t)d.r * d.N;
        GradArgs g{(const bf16_t*)h_old, ws.u, ws.dz, ws.w, d.T,
                   (d.T + slices - 1) / slices, d.d, d.N, d.r,
                   rt * ((d.d + 127) / 128), rt * ((d.N + 127) / 128), ws.part,
                   ws.part + (size_t)slices * na};
        {
            LaunchScope scope("predictor_grads", s);
            hipLaunchKernelGGL(pred_grad_kernel, dim3((unsigned)((g.na + g.nb + 3) / 4), (unsigned)slices),
                               dim3(256), 0, s, g);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const int ba = (int)((na + 255) / 256), bb = (int)((nb + 255) / 256);
        LaunchScope scope("predictor_finish", s);
        hipLaunchKernelGGL(pred_finish_kernel, dim3((unsigned)(ba + bb + 1)), dim3(256), 0, s, g.pa, na,
                           ba, g.pb, nb, bb, slices, dA, dB, ws.kl, d.T, loss_out);
        return hipGetLastError();
    }
    dim3 tok((unsigned)((d.T + 3) / 4));
    {
        // u = h_old A: (token, column) entries summed over the hidden index
        LaunchScope scope("predictor_proj_u", s);
        e = bf ? launch_prod((const bf16_t*)h_old, d.d, 1, A, d.r, 1, (int)d.T, d.r, d.d, ws.part,
                             ws.u, s)
               : launch_prod((const float*)h_old, d.d, 1, A, d.r, 1, (int)d.T, d.r, d.d, ws.part,
                             ws.u, s);
    }
    if (e != hipSuccess) return e;
    LossArgs a{ws.p_cur, p_old, ws.u, B, d.T, d.N, d.r, kind, kl_out, ws.kl, ws.dz, ws.w};
    {
        LaunchScope scope("predictor_kl", s);
        hipLaunchKernelGGL(pred_loss_kernel, tok, dim3(256), 0, s, a);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    {
        LaunchScope scope("predictor_loss_mean", s);
        hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, s, ws.kl, d.T, loss_out);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (B) {
        // dB[q][j] = sum_t u[t][q] dz[t][j]
        LaunchScope scope("predictor_grad_b", s);
        e = launch_prod(ws.u, 1, d.r, ws.dz, d.N, 1, d.r, d.N, d.T, ws.part, dB, s);
        if (e != hipSuccess) return e;
    }
    // dA[i][q] = sum_t h_old[t][i] g[t][q], g = dz B^T (dz itself for the identity)
    const double* g = B ? ws.w : ws.dz;
    LaunchScope scope("predictor_grad_a", s);
    return bf ? launch_prod((const bf16_t*)h_old, 1, d.d, g, d.r, 1, d.d, d.r, d.T, ws.part, dA, s)
              : launch_prod((const float*)h_old, 1, d.d, g, d.r, 1, d.d, d.r, d.T, ws.part, dA, s);
}

}  // namespace pr2
