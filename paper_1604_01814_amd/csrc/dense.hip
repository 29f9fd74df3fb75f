// dense.hip -- the dense force solve of Sec. 3.2: the Schur complement C is
// factored once (C = L L^T, FP64) and its inverse factor W = L^{-1} kept, so
// that every later solve is f = W^T (W b), two triangular matrix-vector
// products that stream W from HBM.
//
// Factorisation: recursive on halves, so that all but the 64 x 64 diagonal
// leaves is matrix multiplication on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64).  For A = [A11 .; A21 A22] with L11 = chol(A11),
// W11 = L11^{-1}:
//   L21 = A21 W11^T,   A22 <- A22 - L21 L21^T,   L22 = chol(A22),
//   W21 = -W22 (L21 W11).
// Each leaf is factored and inverted by one workgroup in LDS.
// Matrices are row-major doubles with a leading dimension; only the lower
// triangle of A is read.
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"

namespace lgfib {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kLeaf = 64;   // leaf order of the recursive factorisation
constexpr int kKT = 32;     // K slice staged in LDS per GEMM step (16 and 64 measured slower)

// C = alpha op(A) op(B) + beta C with op(A)(m, k) = A[m lda + k] and
// op(B)(k, n) = TB ? B[n ldb + k] : B[k ldb + n].  Tile (32 FM)^2 per
// workgroup of four waves, each wave (16 FM)^2 as FM x FM blocks of 16 x 16.
// tri names the operand that is lower triangular (zero above its diagonal), whose
// zero part a tile then skips along k: kTriBtLower, op(B)(k, n) = B[n][k]
// with k <= n; kTriBLower, op(B)(k, n) = B[k][n] with k >= n; kTriALower,
// op(A)(m, k) = A[m][k] with k <= m.  The skipped entries must be zero.
// A tile inside the matrices with whole slices (EDGE = false) takes its loads
// at a uniform base plus a constant 32-bit offset a thread, without the clamps
// of the edge form.  Bound by the matrix cores, which the counters show three
// quarters busy while a tile runs (two workgroups a CU; three with one buffer
// or half slices measured the same or slower).
template <int FM, bool TB, bool EDGE, typename Lds>
__device__ __forceinline__ void gemm_f64_tile(Lds &As, Lds &Bs, int m0, int n0, int kb, int ke, int M, int N,
                                              double alpha, const double *__restrict__ A, long lda,
                                              const double *__restrict__ Bm, long ldb, double beta,
                                              double *__restrict__ C, long ldc) {
    constexpr int T = 32 * FM;              // tile edge
    constexpr int PER = T * kKT / 256;      // staged values per thread and operand
    constexpr int RS = 256 / kKT, KS = 256 / T;   // rows (of k for a plain B) a step of the 256 threads covers
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int wm = (wave / 2) * 16 * FM, wn = (wave % 2) * 16 * FM;
    f64x4 acc[FM][FM];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    double ra[PER], rb[PER];
    const unsigned va = (unsigned)((tid / kKT) * lda + tid % kKT);
    const unsigned vb = (unsigned)(TB ? (tid / kKT) * ldb + tid % kKT : (tid / T) * ldb + tid % T);
    // slice k0 .. k0 + kKT - 1 into registers.  Edge form: loads are clamped
    // into the matrices, so they need no branch; rows of A past M and columns
    // of B past N only reach outputs that are not stored, and entries at
    // k >= ke are zeroed in A alone, which removes their products.
    auto fetch = [&](int k0) {
        if constexpr (!EDGE) {
            k0 = min(k0, ke - kKT);   // past the last slice: read it again, unused
            const double *a0 = A + (long)m0 * lda + k0;
            const double *b0 = TB ? Bm + (long)n0 * ldb + k0 : Bm + (long)k0 * ldb + n0;
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                ra[q] = (a0 + q * RS * lda)[va];
                rb[q] = (b0 + q * (TB ? RS : KS) * ldb)[vb];
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + 256 * q;
            {
                const int mm = e / kKT, kk = e % kKT, m = m0 + mm, k = k0 + kk;
                const double v = A[(long)min(m, M - 1) * lda + min(k, ke - 1)];
                ra[q] = k < ke ? v : 0.0;
            }
            if (TB) {
                const int nn = e / kKT, kk = e % kKT, n = n0 + nn, k = k0 + kk;
                rb[q] = Bm[(long)min(n, N - 1) * ldb + min(k, ke - 1)];
            } else {
                const int kk = e / T, nn = e % T, n = n0 + nn, k = k0 + kk;
                rb[q] = Bm[(long)min(k, ke - 1) * ldb + min(n, N - 1)];
            }
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + 256 * q;
            As[buf][e / kKT][e % kKT] = ra[q];
            if (TB)
                Bs[buf][e / kKT][e % kKT] = rb[q];
            else
                Bs[buf][e % T][e / T] = rb[q];
        }
    };
    fetch(kb);
    stage(0);
    __syncthreads();
    // operand layout of v_mfma_f64_16x16x4f64: lane l holds A[row l%16][k l/16]
    // and B[k l/16][col l%16]; the result D[row l/16 + 4q][col l%16] in acc[q]
    // (rows interleaved, unlike the 16x16x16 BF16 form)
    const int r = lane % 16, kq = lane / 16;
    const int nslice = (ke - kb + kKT - 1) / kKT;
    for (int s = 0; s < nslice; ++s) {
        const int buf = s & 1;
        fetch(kb + (s + 1) * kKT);   // after the last slice: not used
#pragma unroll
        for (int ks = 0; ks < kKT; ks += 4) {
            double a[FM], b[FM];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = As[buf][wm + 16 * i + r][ks + kq];
#pragma unroll
            for (int j = 0; j < FM; ++j) b[j] = Bs[buf][wn + 16 * j + r][ks + kq];
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        stage(buf ^ 1);
        __syncthreads();
    }
    const int c = lane % 16, rq = lane / 16;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int m = m0 + wm + 16 * i + rq + 4 * q, n = n0 + wn + 16 * j + c;
                if (m < M && n < N) {
                    double v = alpha * acc[i][j][q];
                    if (beta != 0.0) v += beta * C[(long)m * ldc + n];
                    C[(long)m * ldc + n] = v;
                }
            }
}

template <int FM, bool TB>
__global__ __launch_bounds__(256) void k_gemm_f64(int M, int N, int K, double alpha, const double *__restrict__ A,
                                                  long lda, const double *__restrict__ Bm, long ldb, double beta,
                                                  double *__restrict__ C, long ldc, int tri) {
    constexpr int T = 32 * FM;
    // two LDS buffers: slice s + 1 is staged while slice s is multiplied
    __shared__ double As[2][T][kKT + 1];    // [m][k]
    __shared__ double Bs[2][T][kKT + 1];    // [n][k]
    // tiles with the longest k range first, so that the last ones to finish are
    // short ones: by falling m, falling n or rising n (a factor of
    // 6600 unknowns with the inner form: 11.5 instead of 11.9 ms)
    int bx = blockIdx.x, by = blockIdx.y;
    if (tri == kTriALower) {
        by = gridDim.y - 1 - by;
    } else {
        const int id = by * gridDim.x + bx;
        bx = id / gridDim.y;
        by = id % gridDim.y;
        if (tri == kTriBtLower) bx = gridDim.x - 1 - bx;
    }
    const int m0 = by * T, n0 = bx * T;
    // k range of the tile (tile edges are multiples of kKT)
    const int kb = tri == kTriBLower ? min(n0, K) : 0;
    const int ke = tri == kTriBtLower ? min(n0 + T, K) : tri == kTriALower ? min(m0 + T, K) : K;
    // offsets of the inner form: 32 bits for the rows one step covers
    const bool inner = m0 + T <= M && n0 + T <= N && ke > kb && (ke - kb) % kKT == 0 && max(lda, ldb) < (1l << 24);
    if (inner)
        gemm_f64_tile<FM, TB, false>(As, Bs, m0, n0, kb, ke, M, N, alpha, A, lda, Bm, ldb, beta, C, ldc);
    else
        gemm_f64_tile<FM, TB, true>(As, Bs, m0, n0, kb, ke, M, N, alpha, A, lda, Bm, ldb, beta, C, ldc);
}

int gemm_f64(int M, int N, int K, double alpha, const double *A, long lda, const double *B, long ldb, bool tb,
             double beta, double *C, long ldc, int tri, hipStream_t st) {
    if (M <= 0 || N <= 0) return LGFIB_OK;
    if (K <= 0) return fail(LGFIB_EINVAL, "gemm_f64: empty inner dimension");
    // 64-edge tiles for every product: the 128-edge form (FM = 4) measured
    // slower even on the 3300-edge products of the top split (fewer
    // workgroups in flight)
    constexpr int T = 64;
    const dim3 grid((N + T - 1) / T, (M + T - 1) / T);
    if (tb)
        hipLaunchKernelGGL((k_gemm_f64<2, true>), grid, dim3(256), 0, st, M, N, K, alpha, A, lda, B, ldb, beta, C,
                           ldc, tri);
    else
        hipLaunchKernelGGL((k_gemm_f64<2, false>), grid, dim3(256), 0, st, M, N, K, alpha, A, lda, B, ldb, beta, C,
                           ldc, tri);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

// 1 / sqrt(d) to double precision: the hardware estimate and two Newton
// steps y <- y + y (1 - d y^2) / 2 (NaN for d < 0, infinity for d = 0)
__device__ __forceinline__ double rsqrt_f64(double d) {
    double y = __builtin_amdgcn_rsq(d);
#pragma unroll
    for (int it = 0; it < 2; ++it) y = fma(0.5 * y, fma(-d, y * y, 1.0), y);
    return y;
}

// Leaf: Cholesky factor L and its inverse W = L^{-1} of an n x n block
// (n <= kLeaf) by one workgroup of four wavefronts (rows n..kLeaf-1 padded with
// the identity, whose factor is the identity).  The leaves form a serial chain
// of n steps, so a leaf is bound by the latency of a step, and the fewer of
// them cross a workgroup barrier the better: the block is taken in panels of
// 16 columns.  Of panel p,
//   one wavefront factors and inverts the 16 x 16 diagonal block in registers
//     (lane i holds row i; a column is spread by lane reads, no barrier),
//   L_ip = A_ip W_pp^T for the blocks below it, one wavefront each, and
//   A_ij -= L_ip L_jp^T for the blocks to its right, on the matrix cores;
// then, for i - j = 1, 2, 3, W_ij = -W_ii sum_k L_ik W_kj, whose inner sum comes
// out of the matrix cores in the operand layout of the outer product.  14
// barriers a leaf.  The form with one column of all 64 rows per barrier took
// 43 us (128 barriers), this one 23; a 128-row node 107 -> 65 us.
// A pivot that is not positive sets *bad; the factor then holds NaN.
// On return, ls holds the factor and wv its inverse (row stride kLP, zeros
// above the diagonal, the identity in the padding).
constexpr int kLeafThreads = 256;
constexpr int kLP = kLeaf + 1;   // row stride of the LDS tiles
constexpr int kPan = 16;         // panel width: one MFMA block

__device__ __forceinline__ double lane_read(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Factor and inverse of the diagonal block at d (in ls), inverse to w (in wv),
// by one wavefront; its four groups of sixteen lanes do the same.
__device__ __forceinline__ void chol16(double *__restrict__ d, double *__restrict__ w, int *__restrict__ bad) {
    const int i = threadIdx.x % kPan;
    double r[kPan], ip[kPan], x[kPan];
#pragma unroll
    for (int k = 0; k < kPan; ++k) r[k] = d[i * kLP + k];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < kPan; ++k) {
        const double piv = lane_read(r[k], k);
        ok = ok && piv > 0.0;
        ip[k] = rsqrt_f64(piv);
        r[k] *= ip[k];   // L[i][k]; rows above k hold garbage that nothing reads
#pragma unroll
        for (int j = k + 1; j < kPan; ++j) r[j] = fma(-r[k], lane_read(r[k], j), r[j]);
    }
    // column i of the inverse: L x = e_i
#pragma unroll
    for (int k = 0; k < kPan; ++k) x[k] = k == i ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < kPan; ++k) {
        x[k] *= ip[k];
#pragma unroll
        for (int j = k + 1; j < kPan; ++j) x[j] = fma(-lane_read(r[k], j), x[k], x[j]);
    }
    if (threadIdx.x < kPan) {
#pragma unroll
        for (int k = 0; k < kPan; ++k) {
            d[i * kLP + k] = k <= i ? r[k] : 0.0;
            w[k * kLP + i] = x[k];
        }
        if (i == 0 && !ok) *bad = 1;
    }
}

// acc += X Y^T for 16 x 16 blocks in LDS
__device__ __forceinline__ f64x4 mm16_nt(const double *__restrict__ X, const double *__restrict__ Y, f64x4 acc) {
    const int r = threadIdx.x % 16, kq = (threadIdx.x % 64) / 16;
#pragma unroll
    for (int ks = 0; ks < kPan; ks += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[r * kLP + ks + kq], Y[r * kLP + ks + kq], acc, 0, 0, 0);
    return acc;
}
// acc += X Y
__device__ __forceinline__ f64x4 mm16_nn(const double *__restrict__ X, const double *__restrict__ Y, f64x4 acc) {
    const int r = threadIdx.x % 16, kq = (threadIdx.x % 64) / 16;
#pragma unroll
    for (int ks = 0; ks < kPan; ks += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[r * kLP + ks + kq], Y[(ks + kq) * kLP + r], acc, 0, 0, 0);
    return acc;
}

__device__ __forceinline__ void leaf_run(double *__restrict__ A, long lda, double *__restrict__ W, long ldw, int n,
                                         int *__restrict__ bad, double *__restrict__ ls, double *__restrict__ wv) {
    constexpr int L = kLeaf, LP = kLP, NP = kLeaf / kPan;
    const int t = threadIdx.x, wave = t / 64, c = t % 16, rq = (t % 64) / 16;
    auto at = [](double *p, int i, int j) { return p + i * kPan * kLP + j * kPan; };
#pragma unroll
    for (int q = 0; q < L * L / kLeafThreads; ++q) {
        const int e = t + q * kLeafThreads, i = e / L, j = e % L;
        ls[i * LP + j] = i < n ? (j <= i ? A[(long)i * lda + j] : 0.0) : (j == i ? 1.0 : 0.0);
        wv[i * LP + j] = 0.0;
    }
    __syncthreads();
#pragma unroll 1
    for (int p = 0; p < NP; ++p) {
        if (wave == 0) chol16(at(ls, p, p), at(wv, p, p), bad);
        __syncthreads();
        if (p + 1 == NP) break;
        if (p + 1 + wave < NP) {   // this wavefront alone reads and writes its block
            double *x = at(ls, p + 1 + wave, p);
            const f64x4 v = mm16_nt(x, at(wv, p, p), f64x4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int q = 0; q < 4; ++q) x[(rq + 4 * q) * LP + c] = v[q];
        }
        __syncthreads();
        const int m = NP - 1 - p;   // blocks (i, j), p < j <= i
        for (int e = wave; e < m * (m + 1) / 2; e += 4) {
            const int i = e >= 3 ? 2 : e >= 1 ? 1 : 0, j = e - i * (i + 1) / 2;
            double *x = at(ls, p + 1 + i, p + 1 + j);
            const f64x4 v = mm16_nt(at(ls, p + 1 + i, p), at(ls, p + 1 + j, p), f64x4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int q = 0; q < 4; ++q) x[(rq + 4 * q) * LP + c] -= v[q];
        }
        __syncthreads();
    }
#pragma unroll 1
    for (int dd = 1; dd < NP; ++dd) {
        if (wave + dd < NP) {
            const int j = wave, i = wave + dd;
            f64x4 sum{0.0, 0.0, 0.0, 0.0}, v{0.0, 0.0, 0.0, 0.0};
            for (int k = j; k < i; ++k) sum = mm16_nn(at(ls, i, k), at(wv, k, j), sum);
            // sum[q] is row rq + 4 q, column c: the operand of k step q
            const double *x = at(wv, i, i);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v = __builtin_amdgcn_mfma_f64_16x16x4f64(x[c * LP + 4 * q + rq], sum[q], v, 0, 0, 0);
            double *y = at(wv, i, j);
#pragma unroll
            for (int q = 0; q < 4; ++q) y[(rq + 4 * q) * LP + c] = -v[q];
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < L * L / kLeafThreads; ++q) {   // rows of L, and of W with zeros above the diagonal
        const int e = t + q * kLeafThreads, i = e / L, j = e % L;
        if (i < n && j <= i) A[(long)i * lda + j] = ls[i * LP + j];
        if (i < n && j < n) W[(long)i * ldw + j] = j <= i ? wv[i * LP + j] : 0.0;
    }
}

__global__ __launch_bounds__(kLeafThreads) void k_chol_leaf(double *__restrict__ A, long lda, double *__restrict__ W,
                                                            long ldw, int n, int *__restrict__ bad) {
    __shared__ double ls[kLeaf * kLP], wv[kLeaf * kLP];
    leaf_run(A, lda, W, ldw, n, bad, ls, wv);
}

// C = X Y^T for 64 x 64 tiles in LDS (row stride kLP): C[i][j] = sum_k
// X(i, k) Y[j][k], with X(i, k) = X[i][k], or X[k][i] when XT.  Wave w of
// four takes the 32 x 32 quadrant (w / 2, w % 2) as 2 x 2 FP64 MFMA blocks;
// out(i, j, v) receives each result.
template <bool XT, class Out>
__device__ __forceinline__ void mm64(const double *__restrict__ X, const double *__restrict__ Y, Out out) {
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wm = (wave / 2) * 32, wn = (wave % 2) * 32;
    const int r = lane % 16, kq = lane / 16;
    f64x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k0 = 0; k0 < kLeaf; k0 += 4) {
        const int k = k0 + kq;
        double a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = XT ? X[k * kLP + wm + 16 * i + r] : X[(wm + 16 * i + r) * kLP + k];
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = Y[(wn + 16 * j + r) * kLP + k];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // result D[row l/16 + 4q][col l%16] in acc[q]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) out(wm + 16 * i + kq + 4 * q, wn + 16 * j + r, acc[i][j][q]);
}

// One node of the recursion with n1 = kLeaf, n2 = n - kLeaf <= kLeaf, in one
// workgroup: the leaf of A11, L21 = A21 W11^T, A22 -= L21 L21^T, the leaf of
// A22, then W21 = -W22 (L21 W11), formed as -W22 (W11^T L21^T)^T.  The same
// steps as the recursion below a node of this size, without its launches.
__global__ __launch_bounds__(kLeafThreads) void k_chol_node(double *__restrict__ A, long lda, double *__restrict__ W,
                                                            long ldw, int n, int *__restrict__ bad) {
    constexpr int L = kLeaf, LP = kLP;
    __shared__ double Wb[L * LP];   // W11
    __shared__ double Xb[L * LP];   // A21, then L21
    __shared__ double Tb[L * LP];   // the leaves' factors, then S^T = (L21 W11)^T
    __shared__ double Vb[L * LP];   // W22
    const int t = threadIdx.x, n2 = n - L;
    double *A21 = A + (long)L * lda, *A22 = A21 + L, *W21 = W + (long)L * ldw, *W22 = W21 + L;
    leaf_run(A, lda, W, ldw, L, bad, Tb, Wb);
    for (int e = t; e < L * L; e += kLeafThreads) {
        const int i = e / L, j = e % L;
        Xb[i * LP + j] = i < n2 ? A21[(long)i * lda + j] : 0.0;
    }
    __syncthreads();
    // L21 = A21 W11^T, kept in registers until every wave has read A21
    double l21[16];
    int li[16], lj[16], nl = 0;
    mm64<false>(Xb, Wb, [&](int i, int j, double v) {
        li[nl] = i;
        lj[nl] = j;
        l21[nl++] = v;
    });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        Xb[li[q] * LP + lj[q]] = l21[q];
        if (li[q] < n2) A21[(long)li[q] * lda + lj[q]] = l21[q];
    }
    __syncthreads();
    // A22 -= L21 L21^T on and below the diagonal
    mm64<false>(Xb, Xb, [&](int i, int j, double v) {
        if (i < n2 && j <= i) A22[(long)i * lda + j] -= v;
    });
    __syncthreads();
    leaf_run(A22, lda, W22, ldw, n2, bad, Tb, Vb);
    __syncthreads();   // Tb has been read
    // S^T = W11^T L21^T
    mm64<true>(Wb, Xb, [&](int i, int j, double v) { Tb[i * LP + j] = v; });
    __syncthreads();
    // W21 = -W22 S
    mm64<false>(Vb, Tb, [&](int i, int j, double v) {
        if (i < n2) W21[(long)i * ldw + j] = -v;
    });
}

// What follows from L21 = S at one level of the recursion, in one launch: A22 -=
// S S^T (tiles on and below the diagonal), T = S W11 (T nullable) and S copied to
// A21.  Three launches of their own leave most of the chip idle on the small
// levels, where a product is bound by its latency
// (factor of 6600 unknowns: 11.5 -> 10.2 ms).
__global__ __launch_bounds__(256) void k_chol_trail(int n1, int n2, const double *__restrict__ S, long lds,
                                                    double *__restrict__ A21, double *__restrict__ A22, long lda,
                                                    const double *__restrict__ W11, long ldw, double *__restrict__ T,
                                                    long ldt) {
    constexpr int E = 64;
    __shared__ double As[2][E][kKT + 1];
    __shared__ double Bs[2][E][kKT + 1];
    const int t1 = (n1 + E - 1) / E, t2 = (n2 + E - 1) / E;
    int id = blockIdx.x;
    if (id < t2 * (t2 + 1) / 2) {
        int r = (int)((sqrtf(8.0f * id + 1.0f) - 1.0f) * 0.5f);
        while (r * (r + 1) / 2 > id) --r;
        while ((r + 1) * (r + 2) / 2 <= id) ++r;
        const int m0 = r * E, n0 = (id - r * (r + 1) / 2) * E;
        if (m0 + E <= n2)   // then n0 + E <= n2; n1 is a multiple of the slice
            gemm_f64_tile<2, true, false>(As, Bs, m0, n0, 0, n1, n2, n2, -1.0, S, lds, S, lds, 1.0, A22, lda);
        else
            gemm_f64_tile<2, true, true>(As, Bs, m0, n0, 0, n1, n2, n2, -1.0, S, lds, S, lds, 1.0, A22, lda);
        return;
    }
    id -= t2 * (t2 + 1) / 2;
    if (T && id < t1 * t2) {   // long contractions first: k runs from n0 to n1
        const int m0 = id % t2 * E, n0 = id / t2 * E;
        if (m0 + E <= n2)
            gemm_f64_tile<2, false, false>(As, Bs, m0, n0, n0, n1, n2, n1, 1.0, S, lds, W11, ldw, 0.0, T, ldt);
        else
            gemm_f64_tile<2, false, true>(As, Bs, m0, n0, n0, n1, n2, n1, 1.0, S, lds, W11, ldw, 0.0, T, ldt);
        return;
    }
    if (T) id -= t1 * t2;
    const int m0 = id % t2 * E, c = id / t2 * E + threadIdx.x % E, m1 = min(m0 + E, n2);
    for (int m = m0 + threadIdx.x / E; m < m1; m += 256 / E) A21[m * lda + c] = S[m * lds + c];
}

__global__ void k_zero2d(double *__restrict__ dst, long ldd, int rows, int cols) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)rows * cols) return;
    dst[(long)(t / cols) * ldd + t % cols] = 0.0;
}

static inline unsigned nblk256(long n) { return (unsigned)((n + 255) / 256); }

// Workspace of the recursion: S, L21 of a level until it is in place, and T, per
// depth with chol_early(n1), L21 W11 until the level's W22 is known (at the other
// depths, and with null T, it is formed in S only then)
struct CholWs {
    double *S, *T;
};
// The early product fills up a launch that is too small by itself, so it gains on
// the small levels: 11.2 ms without any for a factor of 6600 unknowns, 10.1 with
// those up to 24 MiB (n1 <= 1773), 10.0 with all; 12,000 34.2 and 33.9 ms with all,
// 16,000 68.7 and 68.3.  The context keeps the workspace, and all of T would be
// n^2 / 3 values beside the n^2 / 4 of S; so it is at most 32 MiB.
constexpr size_t kEarlyMax = (size_t)3 << 20;   // values at one depth
static bool chol_early(size_t n1) { return n1 * n1 <= kEarlyMax; }

// factor the n x n block at A (lower) into L (in place) and W = L^{-1}
static int chol_rec(lgfib_ctx *ctx, int n, double *A, long lda, double *W, long ldw, CholWs ws, int *bad,
                    hipStream_t st) {
    int rc;
    if (n <= kLeaf) {
        ProfScope ps(ctx, "k_chol_leaf", st);
        hipLaunchKernelGGL(k_chol_leaf, dim3(1), dim3(kLeafThreads), 0, st, A, lda, W, ldw, n, bad);
        LGF_HIP(hipGetLastError());
        return LGFIB_OK;
    }
    if (n <= 2 * kLeaf) {
        ProfScope ps(ctx, "k_chol_node", st);
        hipLaunchKernelGGL(k_chol_node, dim3(1), dim3(kLeafThreads), 0, st, A, lda, W, ldw, n, bad);
        LGF_HIP(hipGetLastError());
        return LGFIB_OK;
    }
    const int n1 = kLeaf * ((n + 2 * kLeaf - 1) / (2 * kLeaf)), n2 = n - n1;
    const long lds = n1;
    double *A21 = A + (long)n1 * lda, *A22 = A21 + n1, *W21 = W + (long)n1 * ldw, *W22 = W21 + n1;
    double *early = chol_early(n1) ? ws.T : nullptr;
    const CholWs inner{ws.S, early ? early + n2 * lds : ws.T};
    if ((rc = chol_rec(ctx, n1, A, lda, W, ldw, inner, bad, st))) return rc;
    {
        ProfScope ps(ctx, "k_gemm_f64", st);
        // S = L21 = A21 W11^T
        if ((rc = gemm_f64(n2, n1, n1, 1.0, A21, lda, W, ldw, true, 0.0, ws.S, lds, kTriBtLower, st)))
            return rc;
        const unsigned t1 = n1 / 64, t2 = (n2 + 63) / 64;
        hipLaunchKernelGGL(k_chol_trail, dim3(t2 * (t2 + 1) / 2 + (early ? 2 : 1) * t1 * t2), dim3(256), 0, st, n1, n2,
                           ws.S, lds, A21, A22, lda, W, ldw, early, lds);
        LGF_HIP(hipGetLastError());
    }
    if ((rc = chol_rec(ctx, n2, A22, lda, W22, ldw, inner, bad, st))) return rc;
    {
        ProfScope ps(ctx, "k_gemm_f64", st);
        // W21 = -W22 (L21 W11)
        const double *T = early;
        if (!T) {
            if ((rc = gemm_f64(n2, n1, n1, 1.0, A21, lda, W, ldw, false, 0.0, ws.S, lds, kTriBLower, st)))
                return rc;
            T = ws.S;
        }
        if ((rc = gemm_f64(n2, n1, n2, -1.0, W22, ldw, T, lds, false, 0.0, W21, ldw, kTriALower, st)))
            return rc;
    }
    return LGFIB_OK;
}

int chol_factor_f64(lgfib_ctx *ctx, int n, double *A, long lda, double *W, long ldw, hipStream_t st) {
    if (n == 0) return LGFIB_OK;
    int rc;
    // S, then T of the depths: half the order of the depth above, rounded up to leaves
    size_t ns = 0, nt = 0;
    for (size_t m = n; m > 2 * kLeaf;) {
        const size_t n1 = kLeaf * ((m + 2 * kLeaf - 1) / (2 * kLeaf));
        if (!ns) ns = (m - n1) * n1;
        if (chol_early(n1)) nt += n1 * n1;
        m = n1;
    }
    CholWs ws{nullptr, nullptr};
    if (ns) {   // without room for T its products are formed in S
        if (ctx->dense_ws.reserve((ns + nt) * sizeof(double)) == LGFIB_OK)
            ws.T = ctx->dense_ws.as<double>() + ns;
        else if ((rc = ctx->dense_ws.reserve(ns * sizeof(double))))
            return rc;
        ws.S = ctx->dense_ws.as<double>();
    }
    if ((rc = ctx->dense_flag.reserve(sizeof(int)))) return rc;
    LGF_HIP(hipMemsetAsync(ctx->dense_flag.p, 0, sizeof(int), st));
    // the strict upper blocks of W are never written by the recursion
    hipLaunchKernelGGL(k_zero2d, dim3(nblk256((long)n * n)), dim3(256), 0, st, W, ldw, n, n);
    LGF_HIP(hipGetLastError());
    if ((rc = chol_rec(ctx, n, A, lda, W, ldw, ws, ctx->dense_flag.as<int>(), st))) return rc;
    int bad = 0;
    LGF_HIP(hipMemcpyAsync(&bad, ctx->dense_flag.p, sizeof(int), hipMemcpyDeviceToHost, st));
    LGF_HIP(hipStreamSynchronize(st));
    if (bad) return fail(LGFIB_ENOTSPD, "Cholesky factorisation: the matrix is not positive definite");
    return LGFIB_OK;
}

// y = W b, W lower triangular: one wavefront per row, j <= i
__global__ __launch_bounds__(256) void k_trmv_rows(const double *__restrict__ W, long ldw, const double *__restrict__ b,
                                                   double *__restrict__ y, int n) {
    const int row = blockIdx.x * 4 + threadIdx.x / 64, lane = threadIdx.x % 64;
    if (row >= n) return;
    const double *w = W + (long)row * ldw;
    double s = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;   // four loads in flight per lane
    int j = lane;
    // unrolled twice so that eight loads per lane are in flight (the
    // accumulation order is that of the plain loop)
#pragma unroll 2
    for (; j + 192 <= row; j += 256) {
        s += w[j] * b[j];
        s1 += w[j + 64] * b[j + 64];
        s2 += w[j + 128] * b[j + 128];
        s3 += w[j + 192] * b[j + 192];
    }
    for (; j <= row; j += 64) s += w[j] * b[j];
    s += (s1 + s2) + s3;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) y[row] = s;
}

constexpr int kColChunks = 32;   // row chunks of the transposed product

// part[r][j] = sum over rows i of chunk r with i >= j of W[i][j] y[i]
__global__ __launch_bounds__(256) void k_trmv_cols(const double *__restrict__ W, long ldw, const double *__restrict__ y,
                                                   double *__restrict__ part, int n, int rows_per) {
    const int j = blockIdx.x * 256 + threadIdx.x, r = blockIdx.y;
    const int j0 = blockIdx.x * 256;
    const int i0 = max(r * rows_per, j0), i1 = min((r + 1) * rows_per, n);
    double s = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    if (j < n) {
        const double *wc = W + j;
        int i = i0;
        // (unrolling this loop twice measured slower: 0.065 -> 0.069 ms for
        // the three solve kernels at 6600 unknowns)
        for (; i + 3 < i1; i += 4) {   // entries above the diagonal are not part of W
            const double w0 = wc[(long)i * ldw], w1 = wc[(long)(i + 1) * ldw], w2 = wc[(long)(i + 2) * ldw],
                         w3 = wc[(long)(i + 3) * ldw];
            s += (i >= j ? w0 : 0.0) * y[i];
            s1 += (i + 1 >= j ? w1 : 0.0) * y[i + 1];
            s2 += (i + 2 >= j ? w2 : 0.0) * y[i + 2];
            s3 += (i + 3 >= j ? w3 : 0.0) * y[i + 3];
        }
        for (; i < i1; ++i) s += (i >= j ? wc[(long)i * ldw] : 0.0) * y[i];
        part[(long)r * n + j] = s + ((s1 + s2) + s3);
    }
}

// the partial sums added in chunk order; a compile-time count lets every
// load be issued before the first add
__global__ void k_sum_parts(const double *__restrict__ part, double *__restrict__ x, int n) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    double v[kColChunks];
#pragma unroll
    for (int r = 0; r < kColChunks; ++r) v[r] = part[(long)r * n + j];
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < kColChunks; ++r) s += v[r];
    x[j] = s;
}

int chol_solve_f64(lgfib_ctx *ctx, int n, const double *W, long ldw, const double *b, double *x, hipStream_t st) {
    if (n == 0) return LGFIB_OK;
    int rc;
    if ((rc = ctx->dense_solve_ws.reserve((size_t)(kColChunks + 1) * n * sizeof(double)))) return rc;
    double *y = ctx->dense_solve_ws.as<double>(), *part = y + n;
    {
        ProfScope ps(ctx, "k_trmv_rows", st);
        hipLaunchKernelGGL(k_trmv_rows, dim3((n + 3) / 4), dim3(256), 0, st, W, ldw, b, y, n);
        LGF_HIP(hipGetLastError());
    }
    {
        ProfScope ps(ctx, "k_trmv_cols", st);
        const int rows_per = (n + kColChunks - 1) / kColChunks;
        hipLaunchKernelGGL(k_trmv_cols, dim3((n + 255) / 256, kColChunks), dim3(256), 0, st, W, ldw, y, part, n,
                           rows_per);
        LGF_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_sum_parts, dim3((n + 255) / 256), dim3(256), 0, st, part, x, n);
        LGF_HIP(hipGetLastError());
    }
    return LGFIB_OK;
}

}  // namespace lgfib

using namespace lgfib;

static bool overlaps(const void *a, size_t na, const void *b, size_t nb) {
    const char *pa = (const char *)a, *pb = (const char *)b;
    return pa < pb + nb && pb < pa + na;
}

extern "C" int ib_chol_factor(lgfib_ctx *ctx, int n, double *A, int lda, double *W, int ldw, lgfib_stream_t stream) {
    if (!ctx) return fail(LGFIB_EINVAL, "ib_chol_factor: null context");
    if (n < 0 || lda < std::max(n, 1) || ldw < std::max(n, 1))
        return fail(LGFIB_EINVAL, "ib_chol_factor: need n >= 0 and leading dimensions >= n");
    if (n > 0 && (!A || !W)) return fail(LGFIB_EINVAL, "ib_chol_factor: null matrix");
    if (n > 0 && overlaps(A, ((size_t)(n - 1) * lda + n) * 8, W, ((size_t)(n - 1) * ldw + n) * 8))
        return fail(LGFIB_EINVAL, "ib_chol_factor: A and W overlap");
    LGF_HIP(hipSetDevice(ctx->device));
    return chol_factor_f64(ctx, n, A, lda, W, ldw, (hipStream_t)stream);
}

extern "C" int ib_chol_solve(lgfib_ctx *ctx, int n, const double *W, int ldw, const double *b, double *x,
                             lgfib_stream_t stream) {
    if (!ctx) return fail(LGFIB_EINVAL, "ib_chol_solve: null context");
    if (n < 0 || ldw < std::max(n, 1)) return fail(LGFIB_EINVAL, "ib_chol_solve: need n >= 0 and ldw >= n");
    if (n > 0 && (!W || !b || !x)) return fail(LGFIB_EINVAL, "ib_chol_solve: null pointer");
    LGF_HIP(hipSetDevice(ctx->device));
    return chol_solve_f64(ctx, n, W, ldw, b, x, (hipStream_t)stream);
}
