// mlp.hip -- learned warm start for the force solve: a per-marker MLP
// (nin -> nh -> nh -> nout, tanh), BF16 weights and GEMM operands with FP32
// accumulation on the matrix cores, FP32 master weights trained with Adam by
// hand-written forward / backward kernels.
//
// The warm start is x0_i = 2 f_{k-1,i} - f_{k-2,i} + MLP(features_i) for the
// force solve of step k (the network corrects the linear extrapolation of
// the force history); the CG iteration it starts still decides convergence
// (ib_force_solve rejects a warm start whose residual exceeds ||b||).
//
// Every matrix product is one kernel family: a workgroup of four wavefronts
// owns a T x T tile (T 64 or 32) of C = A B, operands FP32 in memory with
// either index contiguous, rounded to bf16 as they are staged in LDS.  A
// training step is seven launches: gather + normalise, three forward products
// (bias, tanh and the squared-error gradient in their epilogues), two backward
// products (the tanh derivative in the epilogue), and one launch for the three
// weight gradients and the bias gradients with Adam applied as they are stored.
// 4096 rows of 12-256-256-3: 1.70 -> 0.097 ms a step.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "fft_static.h"
#include "internal.h"

namespace lgfib {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A staged tile holds T outer indices by 4096 / T of k, 4 x 4 values per
// thread; its LDS rows are padded by 8 bytes so that the sixteen rows a quarter
// wavefront reads 8 bytes of start in distinct banks.
template <int T> constexpr int kSlice = 4096 / T;

// What the epilogue does with v = (A B)[m][n]
enum MlpEpi {
    kEpiGrad,       // C[m][n] = v, a weight gradient, and Adam on its weight
    kEpiTanh,       // C = tanh(v + bias[n])
    kEpiBias,       // C = v + bias[n]
    kEpiDenorm,     // C = shift[n] + scale[n] (v + bias[n])
    kEpiMse,        // d = v + bias[n] - H[m][n] (H the targets); C = d / rows, errp[tile] = sum of d^2
    kEpiTanhBack    // C = v (1 - H[m][n]^2)
};

struct MlpGemm {
    const float *A, *B, *bias, *H, *shift, *scale;
    float *C;
    double *errp;
    long lda, ldb, ldc, ldh;   // row strides of A, B, C and H
    int M, N, K;
    float rows;
};

// X[row][col .. col + 3] of a rows x cols array with row stride ld, at addresses
// clamped into the array: every load is unconditional and nothing is done to
// its value here, so the loads of several calls stay in flight together.
// VEC: X is 16-byte aligned and ld a multiple of 4 (the rows may be padded).
template <bool VEC>
__device__ __forceinline__ float4 mlp_ld4(const float *__restrict__ X, long ld, int row, int rows, int col, int cols) {
    const float *p = X + (long)min(row, rows - 1) * ld;
    if constexpr (VEC) return *reinterpret_cast<const float4 *>(p + min(col, (int)ld - 4));
    return make_float4(p[min(col, cols - 1)], p[min(col + 1, cols - 1)], p[min(col + 2, cols - 1)],
                       p[min(col + 3, cols - 1)]);
}
// ... and zero for what lies beyond the array
__device__ __forceinline__ float4 mlp_mask4(float4 v, int row, int rows, int col, int cols) {
    const bool in = row < rows;
    return make_float4(in && col < cols ? v.x : 0.f, in && col + 1 < cols ? v.y : 0.f, in && col + 2 < cols ? v.z : 0.f,
                       in && col + 3 < cols ? v.w : 0.f);
}

// This thread's 4 x 4 piece of the operand tile X (T outer x kSlice k) that
// starts at (o0, k0): r[i] holds k..k+3 of outer index o + i when k is
// contiguous in memory (KC), else outer o..o+3 of k index k + i.  Lanes walk
// the contiguous index.  The outer index ends at O and k at K; mlp_store puts
// zeros for the rest.
template <int T, bool KC> __device__ __forceinline__ void mlp_at(int &c, int &q) {
    constexpr int W = (KC ? kSlice<T> : T) / 4;
    c = ((int)threadIdx.x % W) * 4;
    q = ((int)threadIdx.x / W) * 4;
}
template <int T, bool KC, bool VEC>
__device__ __forceinline__ void mlp_load(const float *__restrict__ X, long ld, int o0, int O, int k0, int K, float4 r[4]) {
    int c, q;
    mlp_at<T, KC>(c, q);
    const int row = KC ? o0 + q : k0 + q, col = KC ? k0 + c : o0 + c;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = mlp_ld4<VEC>(X, ld, row + i, KC ? O : K, col, KC ? K : O);
}

// round to nearest even
__device__ __forceinline__ bf16x4 mlp_bf4(float a, float b, float c, float d) {
    return bf16x4{__builtin_bit_cast(short, (__bf16)a), __builtin_bit_cast(short, (__bf16)b),
                  __builtin_bit_cast(short, (__bf16)c), __builtin_bit_cast(short, (__bf16)d)};
}

template <int T, bool KC>
__device__ __forceinline__ void mlp_store(unsigned short (*S)[kSlice<T> + 4], float4 r[4], int o0, int O, int k0, int K) {
    int c, q;
    mlp_at<T, KC>(c, q);
    if (o0 + T > O || k0 + kSlice<T> > K) {
        const int row = KC ? o0 + q : k0 + q, col = KC ? k0 + c : o0 + c;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = mlp_mask4(r[i], row + i, KC ? O : K, col, KC ? K : O);
    }
    if constexpr (KC) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<bf16x4 *>(&S[q + i][c]) = mlp_bf4(r[i].x, r[i].y, r[i].z, r[i].w);
    } else {
        *reinterpret_cast<bf16x4 *>(&S[c + 0][q]) = mlp_bf4(r[0].x, r[1].x, r[2].x, r[3].x);
        *reinterpret_cast<bf16x4 *>(&S[c + 1][q]) = mlp_bf4(r[0].y, r[1].y, r[2].y, r[3].y);
        *reinterpret_cast<bf16x4 *>(&S[c + 2][q]) = mlp_bf4(r[0].z, r[1].z, r[2].z, r[3].z);
        *reinterpret_cast<bf16x4 *>(&S[c + 3][q]) = mlp_bf4(r[0].w, r[1].w, r[2].w, r[3].w);
    }
}

struct MlpAdam {
    float *p, *m1, *m2;   // null p: gradients only
    float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ void mlp_adam(const MlpAdam &o, long t, float gi) {
    const float a = fmaf(1.f - o.b1, gi, o.b1 * o.m1[t]);
    const float v = fmaf(gi, (1.f - o.b2) * gi, o.b2 * o.m2[t]);
    o.m1[t] = a;
    o.m2[t] = v;
    o.p[t] -= o.lr * (a / o.c1) / (sqrtf(v / o.c2) + o.eps);
}

// One T x T tile of C.  These products are small (a 64-row tile of the
// 12-256-256-3 network is 8 MFLOP) and bound by the latency of their operands,
// not by the matrix cores: K comes in slices of 4096 / T through two LDS
// buffers, one barrier per slice (of LDS only), the sixteen-byte loads of the
// next D = 4 slices in flight in registers while one multiplies.  k runs in order through one accumulator.
// AKC / BKC: k is the contiguous index of A / B.
template <int T, bool AKC, bool BKC, int EPI, bool VEC>
__device__ __forceinline__ void mlp_tile_v(const MlpGemm &g, int m0, int n0, const MlpAdam &opt, long off,
                                           unsigned short (*As)[T][kSlice<T> + 4], unsigned short (*Bs)[T][kSlice<T> + 4]) {
    constexpr int KT = kSlice<T>, F = T / 32;   // wavefront: F x F fragments of 16 x 16
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int wm = (wave / 2) * (T / 2), wn = (wave % 2) * (T / 2);   // wave's part of the tile
    f32x4 acc[F][F];
    for (int i = 0; i < F; ++i)
        for (int j = 0; j < F; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int D = 4;
    float4 ra[D][4], rb[D][4];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        mlp_load<T, AKC, VEC>(g.A, g.lda, m0, g.M, d * KT, g.K, ra[d]);
        mlp_load<T, BKC, VEC>(g.B, g.ldb, n0, g.N, d * KT, g.K, rb[d]);
    }
    // operand layout of v_mfma_f32_16x16x16_bf16: lane l holds
    //   A[row l%16][k 4(l/16)..+3], B[k 4(l/16)..+3][col l%16]
    const int r = lane % 16, kq = 4 * (lane / 16);
    auto stage = [&](int d, int k0) {
        mlp_store<T, AKC>(As[d % 2], ra[d], m0, g.M, k0, g.K);
        mlp_store<T, BKC>(Bs[d % 2], rb[d], n0, g.N, k0, g.K);
        lds_barrier();
    };
    auto multiply = [&](int d, int k0) {
        const int ks = min(KT, g.K - k0);
#pragma unroll
        for (int kk = 0; kk < KT; kk += 16) {
            if (kk >= ks) break;
            bf16x4 a[F], b[F];
#pragma unroll
            for (int i = 0; i < F; ++i) a[i] = *reinterpret_cast<const bf16x4 *>(&As[d % 2][wm + 16 * i + r][kk + kq]);
#pragma unroll
            for (int j = 0; j < F; ++j) b[j] = *reinterpret_cast<const bf16x4 *>(&Bs[d % 2][wn + 16 * j + r][kk + kq]);
#pragma unroll
            for (int i = 0; i < F; ++i)
#pragma unroll
                for (int j = 0; j < F; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    // D slices per round, their successors loaded unconditionally (past the end
    // at clamped addresses): a branch around a load makes the compiler wait for
    // every load in flight.  The last round loads nothing.
    int kd = 0;
    for (; kd + D * KT < g.K; kd += D * KT) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int k0 = kd + d * KT;
            stage(d, k0);
            mlp_load<T, AKC, VEC>(g.A, g.lda, m0, g.M, k0 + D * KT, g.K, ra[d]);
            mlp_load<T, BKC, VEC>(g.B, g.ldb, n0, g.N, k0 + D * KT, g.K, rb[d]);
            multiply(d, k0);
        }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int k0 = kd + d * KT;
        if (k0 >= g.K) break;
        stage(d, k0);
        multiply(d, k0);
    }
    // result layout: lane l holds D[row 4(l/16)+q][col l%16]
    const int c = lane % 16, rq = 4 * (lane / 16);
    double err = 0.0;
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = m0 + wm + 16 * i + rq + q, n = n0 + wn + 16 * j + c;
                if (m >= g.M || n >= g.N) continue;
                const long at = (long)m * g.ldc + n;
                float v = acc[i][j][q];
                if constexpr (EPI == kEpiTanh) v = tanhf(v + g.bias[n]);
                if constexpr (EPI == kEpiBias) v = v + g.bias[n];
                if constexpr (EPI == kEpiDenorm) v = g.shift[n] + g.scale[n] * (v + g.bias[n]);
                if constexpr (EPI == kEpiTanhBack) {
                    const float h = g.H[(long)m * g.ldh + n];
                    v *= 1.f - h * h;
                }
                if constexpr (EPI == kEpiMse) {
                    const float d = (v + g.bias[n]) - g.H[(long)m * g.ldh + n];
                    v = d / g.rows;
                    err += (double)(d * d);
                }
                g.C[at] = v;
                if constexpr (EPI == kEpiGrad)
                    if (opt.p) mlp_adam(opt, off + at, v);
            }
    if constexpr (EPI == kEpiMse) {   // one partial loss per tile, in a fixed order
        __shared__ double sh[4];
        for (int o = 32; o > 0; o >>= 1) err += __shfl_down(err, o);
        if (lane == 0) sh[wave] = err;
        __syncthreads();
        if (tid == 0) g.errp[(long)blockIdx.y * gridDim.x + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    }
}

// sixteen-byte loads where both operands' rows allow them (uniform)
template <int T, bool AKC, bool BKC, int EPI>
__device__ __forceinline__ void mlp_tile(const MlpGemm &g, int m0, int n0, const MlpAdam &opt, long off) {
    const bool va = g.lda % 4 == 0 && (((size_t)g.A) & 15) == 0, vb = g.ldb % 4 == 0 && (((size_t)g.B) & 15) == 0;
    __shared__ __align__(16) unsigned short As[2][T][kSlice<T> + 4];   // [m][k]
    __shared__ __align__(16) unsigned short Bs[2][T][kSlice<T> + 4];   // [n][k]
    if (va && vb) mlp_tile_v<T, AKC, BKC, EPI, true>(g, m0, n0, opt, off, As, Bs);
    else mlp_tile_v<T, AKC, BKC, EPI, false>(g, m0, n0, opt, off, As, Bs);
}

// one product, a T x T tile per workgroup
template <int T, bool BKC, int EPI> __global__ __launch_bounds__(256) void k_mlp_gemm(MlpGemm g) {
    mlp_tile<T, true, BKC, EPI>(g, blockIdx.y * T, blockIdx.x * T, MlpAdam{}, 0);
}

// The three weight gradients G[n][k] = sum_m dZ[m][n] X[m][k] of a step, the
// column sums of dZ (the bias gradients), Adam on all of them and the loss, in
// one launch.  Workgroups 0..first[3]-1 own a T x T tile of a weight gradient,
// the next ones four bias columns each, the last one sums the tiles' losses.
// A tile's sum over the rows stays one chain in row order; 256 x 256 outputs
// give only 16 tiles of 64 (4096 rows: 54 us, what one compute unit can read
// bounds it) but 64 of 32 (29 us), so T = 32 runs while the tiles of 64 would
// leave compute units idle.
struct MlpGrads {
    MlpGemm g[3];
    long off[3], boff[3];   // offsets of the weights and biases in the gradient vector
    int first[4], bfirst[4];   // first workgroup of each product's tiles and bias columns
    int tn[3];              // tiles along N
    float *grad;
    MlpAdam opt;
    const double *errp;
    int nerr;
    double *loss;
};
template <int T> __global__ __launch_bounds__(256) void k_mlp_grads(MlpGrads j) {
    const int t = blockIdx.x, tid = threadIdx.x;
    if (t < j.first[3]) {
        const int w = t < j.first[1] ? 0 : t < j.first[2] ? 1 : 2;
        const int tile = t - j.first[w], bm = tile / j.tn[w], bn = tile % j.tn[w];
        mlp_tile<T, false, false, kEpiGrad>(j.g[w], bm * T, bn * T, j.opt, j.off[w]);
        return;
    }
    if (t < j.bfirst[3]) {   // columns 4 q..+3 of dZ: 256 partial sums each, then a tree
        __shared__ float4 sh[256];
        const int w = t < j.bfirst[1] ? 0 : t < j.bfirst[2] ? 1 : 2;
        const MlpGemm &g = j.g[w];
        const int n0 = (t - j.bfirst[w]) * 4;
        const bool vec = g.lda % 4 == 0 && (((size_t)g.A) & 15) == 0;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        int m = tid;
        for (; m + 768 < g.K; m += 1024) {   // four loads in flight, added in order
            float4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = vec ? mlp_ld4<true>(g.A, g.lda, m + 256 * i, g.K, n0, g.M)
                           : mlp_ld4<false>(g.A, g.lda, m + 256 * i, g.K, n0, g.M);
#pragma unroll
            for (int i = 0; i < 4; ++i) s = make_float4(s.x + v[i].x, s.y + v[i].y, s.z + v[i].z, s.w + v[i].w);
        }
        for (; m < g.K; m += 256) {
            const float4 v = mlp_ld4<false>(g.A, g.lda, m, g.K, n0, g.M);
            s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
        }
        sh[tid] = s;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (tid < h) {
                const float4 a = sh[tid], b = sh[tid + h];
                sh[tid] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
            }
            __syncthreads();
        }
        if (tid < 4 && n0 + tid < g.M) {
            const float gi = reinterpret_cast<const float *>(&sh[0])[tid];
            const long at = j.boff[w] + n0 + tid;
            j.grad[at] = gi;
            if (j.opt.p) mlp_adam(j.opt, at, gi);
        }
        return;
    }
    __shared__ double shd[256];
    double s = 0.0;
    for (int i = tid; i < j.nerr; i += 256) s += j.errp[i];
    shd[tid] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) shd[tid] += shd[tid + h];
        __syncthreads();
    }
    if (tid == 0) *j.loss = shd[0];
}

// normalised inputs xh = (x - in_shift) / in_scale and, when t is given,
// targets th = (t - out_shift) / out_scale, of rows idx (all in order when
// idx is null); rows of xh are ldx apart
__global__ void k_mlp_prep(const float *__restrict__ x, const float *__restrict__ ishift,
                           const float *__restrict__ iscale, float *__restrict__ xh, int ldx, int nin,
                           const float *__restrict__ t, const float *__restrict__ oshift,
                           const float *__restrict__ oscale, float *__restrict__ th, int nout,
                           const int *__restrict__ idx, int M) {
    const int w = nin + (t ? nout : 0);
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (long)M * w) return;
    const long r = e / w;
    const int c = (int)(e - r * w);
    const long src = idx ? idx[r] : r;
    if (c < nin) xh[r * ldx + c] = (x[src * nin + c] - ishift[c]) / iscale[c];
    else th[r * nout + c - nin] = (t[src * nout + c - nin] - oshift[c - nin]) / oscale[c - nin];
}

// features of marker i for the force solve of step k:
//   [n_i (3), U_{k+1} - U_k, U_k - U_{k-1}, U_{k-1} - U_{k-2},
//    f_{k-1,i} (3), f_{k-1,i} - f_{k-2,i} (3)]
__global__ void k_features(const double *__restrict__ normals, double d0, double d1, double d2,
                           const double *__restrict__ f1, const double *__restrict__ f2, float *__restrict__ out,
                           int NL) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NL) return;
    float *o = out + (long)i * 12;
    for (int a = 0; a < 3; ++a) o[a] = (float)normals[3 * i + a];
    o[3] = (float)d0;
    o[4] = (float)d1;
    o[5] = (float)d2;
    for (int a = 0; a < 3; ++a) {
        o[6 + a] = (float)f1[3 * i + a];
        o[9 + a] = (float)(f1[3 * i + a] - f2[3 * i + a]);
    }
}

// x0 = 2 f_{k-1} - f_{k-2} + (shift + scale * o): the network corrects the
// linear extrapolation of the force history
__global__ void k_warm(const double *__restrict__ f1, const double *__restrict__ f2, const float *__restrict__ o,
                       const float *__restrict__ shift, const float *__restrict__ scale, double *__restrict__ x0,
                       int NL) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 3 * NL) return;
    const int a = t % 3;
    x0[t] = (2.0 * f1[t] - f2[t]) + (double)(shift[a] + scale[a] * o[t]);
}

static unsigned nb(long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace lgfib

using namespace lgfib;

struct ib_mlp {
    lgfib_ctx *ctx = nullptr;
    int nin = 0, nh = 0, nout = 0;
    long nparam = 0;
    long oW1 = 0, ob1 = 0, oW2 = 0, ob2 = 0, oW3 = 0, ob3 = 0;
    DevBuf p, g, m1, m2;                  // params, grads, Adam moments (FP32)
    DevBuf in_shift, in_scale, out_shift, out_scale;
    DevBuf xh, th, h1, h2, o, dO, d1, d2, errp, loss;   // activations (grown on demand)
    int cap = 0;
    long step = 0;
};

static int mlp_tiles(int n, int T = 64) { return (n + T - 1) / T; }

// rows of xh and dO are padded to whole 16 bytes, so that the products read
// them in such pieces whatever the width
static int mlp_pad(int n) { return (n + 3) / 4 * 4; }

static int mlp_reserve(ib_mlp *m, int M) {
    if (M <= m->cap) return LGFIB_OK;
    int rc;
    const size_t f = sizeof(float);
    m->cap = 0;   // a buffer that cannot grow is gone
    if ((rc = m->xh.reserve((size_t)M * mlp_pad(m->nin) * f)) || (rc = m->th.reserve((size_t)M * m->nout * f)) ||
        (rc = m->h1.reserve((size_t)M * m->nh * f)) || (rc = m->h2.reserve((size_t)M * m->nh * f)) ||
        (rc = m->o.reserve((size_t)M * m->nout * f)) || (rc = m->dO.reserve((size_t)M * mlp_pad(m->nout) * f)) ||
        (rc = m->d1.reserve((size_t)M * m->nh * f)) || (rc = m->d2.reserve((size_t)M * m->nh * f)) ||
        (rc = m->errp.reserve((size_t)mlp_tiles(M) * mlp_tiles(m->nout) * sizeof(double))))
        return rc;
    m->cap = M;
    return LGFIB_OK;
}

template <bool BKC, int EPI> static int gemm(hipStream_t st, const MlpGemm &g) {
    hipLaunchKernelGGL((k_mlp_gemm<64, BKC, EPI>), dim3(mlp_tiles(g.N), mlp_tiles(g.M)), dim3(256), 0, st, g);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

// C[M][N] = A[M][K] B, B stored [n][k] or, with BKC false in gemm(), [k][n]
static MlpGemm product(const float *A, long lda, const float *B, long ldb, float *C, int M, int N, int K) {
    MlpGemm g{};
    g.A = A;
    g.B = B;
    g.C = C;
    g.lda = lda;
    g.ldb = ldb;
    g.ldc = N;
    g.M = M;
    g.N = N;
    g.K = K;
    return g;
}

// forward up to the last hidden layer: xh, h1 and h2 of rows idx of x (all M
// in order when idx is null); t adds the normalised targets th
static int mlp_hidden(ib_mlp *m, const float *x, const float *t, const int *idx, int M, hipStream_t st) {
    const float *P = m->p.as<float>();
    float *xh = m->xh.as<float>(), *h1 = m->h1.as<float>(), *h2 = m->h2.as<float>();
    hipLaunchKernelGGL(k_mlp_prep, dim3(nb((long)M * (m->nin + (t ? m->nout : 0)))), dim3(256), 0, st, x,
                       m->in_shift.as<float>(), m->in_scale.as<float>(), xh, mlp_pad(m->nin), m->nin, t, m->out_shift.as<float>(),
                       m->out_scale.as<float>(), m->th.as<float>(), m->nout, idx, M);
    LGF_HIP(hipGetLastError());
    int rc;
    // h1 = tanh(xh W1^T + b1), h2 = tanh(h1 W2^T + b2)
    MlpGemm g = product(xh, mlp_pad(m->nin), P + m->oW1, m->nin, h1, M, m->nh, m->nin);
    g.bias = P + m->ob1;
    if ((rc = gemm<true, kEpiTanh>(st, g))) return rc;
    g = product(h1, m->nh, P + m->oW2, m->nh, h2, M, m->nh, m->nh);
    g.bias = P + m->ob2;
    return gemm<true, kEpiTanh>(st, g);
}

// the output layer h2 W3^T + b3 into C
static MlpGemm mlp_out(ib_mlp *m, float *C, int M) {
    MlpGemm g = product(m->h2.as<float>(), m->nh, m->p.as<float>() + m->oW3, m->nh, C, M, m->nout, m->nh);
    g.bias = m->p.as<float>() + m->ob3;
    return g;
}

// forward: x (M x nin) -> o (normalised outputs)
static int mlp_fwd(ib_mlp *m, const float *x, int M, hipStream_t st) {
    int rc = mlp_hidden(m, x, nullptr, nullptr, M, st);
    return rc ? rc : gemm<true, kEpiBias>(st, mlp_out(m, m->o.as<float>(), M));
}

// Gradient of  0.5/M sum_m ||o_m - that_m||^2  (that = normalised targets)
// over rows idx of (x, t) into g, and with lr > 0 one Adam step on it.
static int mlp_grad_step(ib_mlp *m, const float *x, const float *t, const int *idx, int M, float lr, hipStream_t st) {
    const float *P = m->p.as<float>();
    float *h1 = m->h1.as<float>(), *h2 = m->h2.as<float>();
    float *dO = m->dO.as<float>(), *d1 = m->d1.as<float>(), *d2 = m->d2.as<float>();
    const int nh = m->nh, nout = m->nout, nin = m->nin;
    int rc = mlp_hidden(m, x, t, idx, M, st);
    if (rc) return rc;
    MlpGemm g = mlp_out(m, dO, M);   // dO = (o - that) / M
    g.H = m->th.as<float>();
    g.ldh = nout;
    g.ldc = mlp_pad(nout);
    g.rows = (float)M;
    g.errp = m->errp.as<double>();
    if ((rc = gemm<true, kEpiMse>(st, g))) return rc;
    // dZ2 = (dO W3) (1 - h2^2), dZ1 = (dZ2 W2) (1 - h1^2)
    g = product(dO, mlp_pad(nout), P + m->oW3, nh, d2, M, nh, nout);
    g.H = h2;
    g.ldh = nh;
    if ((rc = gemm<false, kEpiTanhBack>(st, g))) return rc;
    g = product(d2, nh, P + m->oW2, nh, d1, M, nh, nh);
    g.H = h1;
    g.ldh = nh;
    if ((rc = gemm<false, kEpiTanhBack>(st, g))) return rc;
    // dW[n][k] = sum_m dZ[m][n] X[m][k], db[n] = sum_m dZ[m][n]
    MlpGrads j{};
    const float *dz[3] = {d1, d2, dO}, *xs[3] = {m->xh.as<float>(), h1, h2};
    const int rows[3] = {nh, nh, nout}, cols[3] = {nin, nh, nh}, ldz[3] = {nh, nh, mlp_pad(nout)},
              ldx[3] = {mlp_pad(nin), nh, nh};
    const long off[3] = {m->oW1, m->oW2, m->oW3}, boff[3] = {m->ob1, m->ob2, m->ob3};
    int tiles64 = 0;
    for (int w = 0; w < 3; ++w) tiles64 += mlp_tiles(rows[w]) * mlp_tiles(cols[w]);
    const int T = tiles64 < m->ctx->num_cu ? 32 : 64;
    for (int w = 0; w < 3; ++w) {
        j.g[w] = product(dz[w], ldz[w], xs[w], ldx[w], m->g.as<float>() + off[w], rows[w], cols[w], M);
        j.off[w] = off[w];
        j.boff[w] = boff[w];
        j.tn[w] = mlp_tiles(cols[w], T);
        j.first[w + 1] = j.first[w] + mlp_tiles(rows[w], T) * j.tn[w];
    }
    j.bfirst[0] = j.first[3];
    for (int w = 0; w < 3; ++w) j.bfirst[w + 1] = j.bfirst[w] + mlp_tiles(rows[w], 4);
    j.grad = m->g.as<float>();
    if (lr > 0.f) {
        const float b1 = 0.9f, b2 = 0.999f;
        m->step += 1;
        j.opt = MlpAdam{m->p.as<float>(), m->m1.as<float>(), m->m2.as<float>(), lr, b1, b2, 1e-8f,
                        1.f - powf(b1, (float)m->step), 1.f - powf(b2, (float)m->step)};
    }
    j.errp = m->errp.as<double>();
    j.nerr = mlp_tiles(M) * mlp_tiles(nout);
    j.loss = m->loss.as<double>();
    if (T == 32) hipLaunchKernelGGL(k_mlp_grads<32>, dim3(j.bfirst[3] + 1), dim3(256), 0, st, j);
    else hipLaunchKernelGGL(k_mlp_grads<64>, dim3(j.bfirst[3] + 1), dim3(256), 0, st, j);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

extern "C" int ib_mlp_create(lgfib_ctx *ctx, int nin, int nh, int nout, const float *params, const float *in_shift,
                             const float *in_scale, const float *out_shift, const float *out_scale, ib_mlp **out) {
    if (!out) return fail(LGFIB_EINVAL, "ib_mlp_create: null output");
    *out = nullptr;
    if (!ctx || !params || !in_shift || !in_scale || !out_shift || !out_scale)
        return fail(LGFIB_EINVAL, "ib_mlp_create: null argument");
    if (nin < 1 || nin > 4096 || nh < 1 || nh > 4096 || nout < 1 || nout > 4096)
        return fail(LGFIB_EINVAL, "ib_mlp_create: layer widths must lie in [1, 4096]");
    for (int i = 0; i < nin; ++i)
        if (!(in_scale[i] != 0.f)) return fail(LGFIB_EINVAL, "ib_mlp_create: zero input scale");
    for (int i = 0; i < nout; ++i)
        if (!(out_scale[i] != 0.f)) return fail(LGFIB_EINVAL, "ib_mlp_create: zero output scale");
    LGF_HIP(hipSetDevice(ctx->device));
    auto m = std::make_unique<ib_mlp>();
    m->ctx = ctx;
    m->nin = nin;
    m->nh = nh;
    m->nout = nout;
    m->oW1 = 0;
    m->ob1 = m->oW1 + (long)nh * nin;
    m->oW2 = m->ob1 + nh;
    m->ob2 = m->oW2 + (long)nh * nh;
    m->oW3 = m->ob2 + nh;
    m->ob3 = m->oW3 + (long)nout * nh;
    m->nparam = m->ob3 + nout;
    const size_t pb = (size_t)m->nparam * sizeof(float);
    int rc;
    if ((rc = m->p.reserve(pb)) || (rc = m->g.reserve(pb)) || (rc = m->m1.reserve(pb)) || (rc = m->m2.reserve(pb)) ||
        (rc = m->in_shift.reserve(nin * 4)) || (rc = m->in_scale.reserve(nin * 4)) ||
        (rc = m->out_shift.reserve(nout * 4)) || (rc = m->out_scale.reserve(nout * 4)) || (rc = m->loss.reserve(8)))
        return rc;
    LGF_HIP(hipMemcpy(m->p.p, params, pb, hipMemcpyHostToDevice));
    LGF_HIP(hipMemset(m->m1.p, 0, pb));
    LGF_HIP(hipMemset(m->m2.p, 0, pb));
    LGF_HIP(hipMemcpy(m->in_shift.p, in_shift, nin * 4, hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(m->in_scale.p, in_scale, nin * 4, hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(m->out_shift.p, out_shift, nout * 4, hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(m->out_scale.p, out_scale, nout * 4, hipMemcpyHostToDevice));
    *out = m.release();
    return LGFIB_OK;
}

extern "C" void ib_mlp_destroy(ib_mlp *m) {
    if (!m) return;
    (void)hipSetDevice(m->ctx->device);
    (void)hipDeviceSynchronize();
    delete m;
}

extern "C" int ib_mlp_get_params(ib_mlp *m, float *host, int64_t n) {
    if (!m || !host) return fail(LGFIB_EINVAL, "ib_mlp_get_params: null argument");
    if (n != m->nparam) return fail(LGFIB_EINVAL, "ib_mlp_get_params: count must be " + std::to_string(m->nparam));
    LGF_HIP(hipSetDevice(m->ctx->device));
    LGF_HIP(hipMemcpy(host, m->p.p, (size_t)n * 4, hipMemcpyDeviceToHost));
    return LGFIB_OK;
}

extern "C" int ib_mlp_forward(lgfib_ctx *ctx, ib_mlp *m, const float *x, int M, float *y, lgfib_stream_t stream) {
    if (!ctx || !m || m->ctx != ctx || !x || !y || M < 0) return fail(LGFIB_EINVAL, "ib_mlp_forward: bad argument");
    if (M == 0) return LGFIB_OK;
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if ((rc = mlp_reserve(m, M)) || (rc = mlp_hidden(m, x, nullptr, nullptr, M, st))) return rc;
    MlpGemm g = mlp_out(m, y, M);
    g.shift = m->out_shift.as<float>();
    g.scale = m->out_scale.as<float>();
    return gemm<true, kEpiDenorm>(st, g);
}

extern "C" int ib_mlp_grad(lgfib_ctx *ctx, ib_mlp *m, const float *x, const float *t, int M, float *grad_host,
                           double *loss) {
    if (!ctx || !m || m->ctx != ctx || !x || !t || M < 1) return fail(LGFIB_EINVAL, "ib_mlp_grad: bad argument");
    LGF_HIP(hipSetDevice(ctx->device));
    int rc;
    if ((rc = mlp_reserve(m, M)) || (rc = mlp_grad_step(m, x, t, nullptr, M, 0.f, nullptr))) return rc;
    LGF_HIP(hipDeviceSynchronize());
    if (grad_host) LGF_HIP(hipMemcpy(grad_host, m->g.p, (size_t)m->nparam * 4, hipMemcpyDeviceToHost));
    if (loss) {
        double e = 0.0;
        LGF_HIP(hipMemcpy(&e, m->loss.p, 8, hipMemcpyDeviceToHost));
        *loss = 0.5 * e / M;
    }
    return LGFIB_OK;
}

extern "C" int ib_mlp_train_step(lgfib_ctx *ctx, ib_mlp *m, const float *x, const float *t, int M, float lr,
                                 lgfib_stream_t stream) {
    if (!ctx || !m || m->ctx != ctx || !x || !t || M < 1 || !(lr > 0.f))
        return fail(LGFIB_EINVAL, "ib_mlp_train_step: bad argument");
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if ((rc = mlp_reserve(m, M))) return rc;
    return mlp_grad_step(m, x, t, nullptr, M, lr, st);
}

extern "C" int ib_mlp_last_loss(ib_mlp *m, int M, double *loss) {
    if (!m || !loss || M < 1) return fail(LGFIB_EINVAL, "ib_mlp_last_loss: bad argument");
    LGF_HIP(hipSetDevice(m->ctx->device));
    double e = 0.0;
    LGF_HIP(hipMemcpy(&e, m->loss.p, 8, hipMemcpyDeviceToHost));
    *loss = 0.5 * e / M;
    return LGFIB_OK;
}

extern "C" int ib_mlp_features(lgfib_ctx *ctx, const double *normals, const double *ustate, const double *f1,
                               const double *f2, int NL, float *feats, lgfib_stream_t stream) {
    if (!ctx || !normals || !ustate || !f1 || !f2 || !feats || NL < 0)
        return fail(LGFIB_EINVAL, "ib_mlp_features: bad argument");
    if (NL == 0) return LGFIB_OK;
    LGF_HIP(hipSetDevice(ctx->device));
    hipLaunchKernelGGL(k_features, dim3(nb(NL)), dim3(256), 0, (hipStream_t)stream, normals, ustate[0] - ustate[1],
                       ustate[1] - ustate[2], ustate[2] - ustate[3], f1, f2, feats, NL);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

extern "C" int ib_mlp_warmstart(lgfib_ctx *ctx, ib_mlp *m, const float *feats, const double *f1, const double *f2,
                                int NL, double *x0, lgfib_stream_t stream) {
    if (!ctx || !m || m->ctx != ctx || !feats || !f1 || !f2 || !x0 || NL < 0)
        return fail(LGFIB_EINVAL, "ib_mlp_warmstart: bad argument");
    if (m->nout != 3 || m->nin != 12) return fail(LGFIB_EINVAL, "ib_mlp_warmstart: network must map 12 -> 3");
    if (NL == 0) return LGFIB_OK;
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    int rc;
    if ((rc = mlp_reserve(m, NL)) || (rc = mlp_fwd(m, feats, NL, st))) return rc;
    hipLaunchKernelGGL(k_warm, dim3(nb(3L * NL)), dim3(256), 0, st, f1, f2, m->o.as<float>(),
                       m->out_shift.as<float>(), m->out_scale.as<float>(), x0, NL);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

// splitmix64: a counter-based generator for the epoch permutations
static uint64_t splitmix64(uint64_t &x) {
    uint64_t z = (x += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

extern "C" int ib_mlp_train(lgfib_ctx *ctx, ib_mlp *m, const float *x, const float *t, int M, int epochs, int batch,
                            float lr, uint64_t seed, double *final_loss) {
    if (!ctx || !m || m->ctx != ctx || !x || !t || M < 1 || epochs < 0 || batch < 1 || !(lr > 0.f))
        return fail(LGFIB_EINVAL, "ib_mlp_train: bad argument");
    LGF_HIP(hipSetDevice(ctx->device));
    batch = std::min(batch, M);
    DevBuf bidx;
    int rc;
    if ((rc = bidx.reserve((size_t)M * 4)) || (rc = mlp_reserve(m, batch))) return rc;
    std::vector<int> perm(M);
    uint64_t st = seed;
    double last = 0.0;
    for (int e = 0; e < epochs; ++e) {
        for (int i = 0; i < M; ++i) perm[i] = i;
        for (int i = M - 1; i > 0; --i) std::swap(perm[i], perm[splitmix64(st) % (uint64_t)(i + 1)]);
        LGF_HIP(hipMemcpy(bidx.p, perm.data(), (size_t)M * 4, hipMemcpyHostToDevice));
        for (int b0 = 0; b0 + batch <= M; b0 += batch) {
            if ((rc = mlp_grad_step(m, x, t, bidx.as<int>() + b0, batch, lr, nullptr))) return rc;
        }
        if ((rc = ib_mlp_last_loss(m, batch, &last))) return rc;
    }
    LGF_HIP(hipDeviceSynchronize());
    if (final_loss) *final_loss = last;
    return LGFIB_OK;
}
