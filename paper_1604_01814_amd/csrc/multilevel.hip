// multilevel.hip -- multilevel interpolation evaluator of the lattice
// convolution u = dx^2 G * f (Sec. 2.2, Eq. dpoisson_conv), FP64.
//
// The paper evaluates these convolutions with a kernel-independent,
// interpolation-based multipole method on the block grid and gives no steps;
// the method here is a block tree with p^3 lattice nodes per cluster:
//
//   P2M   per source block: node charges M_a = sum_cells S_a(x) f(x), S_a the
//         tensor Lagrange basis of the block's nodes;
//   M2M   per parent cluster: M_a = sum over children and their nodes of the
//         parent's basis at the child node times the child's charge;
//   M2L   per pair of clusters (target c, source s) on a level's interaction
//         list: Phi_b(c) += sum_a G(y_b - x_a) M_a(s); the pairs are grouped
//         by the displacement D = c - s, and each group is a GEMM of its
//         p^3 x p^3 node matrix with the gathered charges on the matrix
//         cores, tiles of 128 pairs added atomically into Phi (one target
//         receives several displacements);
//   L2L   per target cluster below the top, level by level downwards: Phi(c) +=
//         parent's Phi interpolated at c's nodes (after M2L, which starts from
//         zeroed Phi and takes the pairs of every level in one launch);
//   leaf  per target block: L2P (Phi interpolated at the cells) plus the exact
//         sum over the neighbouring source blocks.  For B = 8 that sum runs on
//         the matrix cores, in the even and odd parts of the blocks along each
//         axis (k_ml_near below); for B = 4 in the leaf kernel, the kernel's
//         2B x 2B x 2B corner held in LDS, one thread owning one x-row of B
//         target cells (B^2 FMAs per 3B/2 loads).
//
// Interaction lists: at the top level every non-neighbour pair; below it the
// children of the parent's neighbours (and the parent) that are not
// neighbours.  Every block pair is counted once, at the finest level where
// the two are apart, or in the leaf sum if they are neighbours.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "conv_common.h"
#include "internal.h"

namespace lgfib {
namespace {

constexpr int kTopSpan = 4;   // top level: at most this many clusters per axis
constexpr int kNearTile = 128;   // pairs (and output columns) per MFMA tile
constexpr int kNearKT = 16;      // contraction terms staged in LDS per step
// Zero axes from which a neighbour product (edge 512 / 2^axes) is cut into
// tiles of 64 columns: edge 128 in one tile of 128 leaves too few workgroups
// (sphere shell of 2.1e5 points: 1.29 ms, against 1.22 with tiles of 64)
constexpr int kNearNarrow = 2;

struct CKey {
    int32_t x, y, z;
    bool operator==(const CKey &o) const { return x == o.x && y == o.y && z == o.z; }
};
struct CKeyHash {
    size_t operator()(const CKey &k) const {
        uint64_t h = 1469598103934665603ull;
        for (int32_t v : {k.x, k.y, k.z}) {
            h ^= (uint32_t)v;
            h *= 1099511628211ull;
        }
        return (size_t)h;
    }
};
using CMap = std::unordered_map<CKey, int, CKeyHash>;

inline CKey parent_of(const CKey &c) { return {c.x >> 1, c.y >> 1, c.z >> 1}; }   // floor(c / 2)
inline int octant_of(const CKey &c) { return (c.x & 1) | ((c.y & 1) << 1) | ((c.z & 1) << 2); }
inline bool adjacent(const CKey &a, const CKey &b) {
    return std::abs(a.x - b.x) <= 1 && std::abs(a.y - b.y) <= 1 && std::abs(a.z - b.z) <= 1;
}

// rounded Chebyshev nodes of a cluster side of L cells (empty if two coincide)
std::vector<int> cluster_nodes(int L, int p) {
    std::vector<int> t(p);
    for (int j = 0; j < p; ++j)
        t[j] = (int)std::floor((L - 1) / 2.0 * (1.0 - std::cos(M_PI * (2 * j + 1) / (2.0 * p))) + 0.5);
    for (int j = 1; j < p; ++j)
        if (t[j] <= t[j - 1]) return {};
    return t;
}

double lagrange(const std::vector<int> &t, int j, double x) {
    double w = 1.0;
    for (int k = 0; k < (int)t.size(); ++k)
        if (k != j) w *= (x - t[k]) / (double)(t[j] - t[k]);
    return w;
}

// ---------------------------------------------------------------- kernels

template <int P, int B>
__global__ __launch_bounds__(256) void k_ml_p2m(const double *__restrict__ f, const double *__restrict__ W0,
                                                 double *__restrict__ M) {
    constexpr int P3 = P * P * P, B3 = B * B * B;
    __shared__ double fs[B3];
    __shared__ double w[P * B];
    const int s = xcd_remap(blockIdx.x, gridDim.x);
    for (int i = threadIdx.x; i < B3; i += blockDim.x) fs[i] = f[(size_t)s * B3 + i];
    for (int i = threadIdx.x; i < P * B; i += blockDim.x) w[i] = W0[i];
    __syncthreads();
    const int a = threadIdx.x;
    if (a >= P3) return;
    const int ax = a % P, ay = (a / P) % P, az = a / (P * P);
    double acc = 0.0;
    for (int z = 0; z < B; ++z)
        for (int y = 0; y < B; ++y) {
            const double wzy = w[az * B + z] * w[ay * B + y];
            double r = 0.0;
#pragma unroll
            for (int x = 0; x < B; ++x) r += w[ax * B + x] * fs[(z * B + y) * B + x];
            acc += wzy * r;
        }
    M[(size_t)s * P3 + a] = acc;
}

// Wup: [2][P][P], Wup[o][j][k] = basis j of the parent at node k of a child
// whose offset in the parent is o (0 or 1) child sides.
template <int P>
__global__ __launch_bounds__(256) void k_ml_m2m(const double *__restrict__ Mc, const int *__restrict__ kids,
                                                 const double *__restrict__ Wup, double *__restrict__ Mp) {
    constexpr int P3 = P * P * P;
    __shared__ double w[2 * P * P];
    __shared__ double mc[8 * P3];
    const int c = xcd_remap(blockIdx.x, gridDim.x);
    for (int i = threadIdx.x; i < 2 * P * P; i += blockDim.x) w[i] = Wup[i];
    for (int i = threadIdx.x; i < 8 * P3; i += blockDim.x) {
        const int k = kids[c * 8 + i / P3];
        mc[i] = k >= 0 ? Mc[(size_t)k * P3 + i % P3] : 0.0;
    }
    __syncthreads();
    const int a = threadIdx.x;
    if (a >= P3) return;
    const int ax = a % P, ay = (a / P) % P, az = a / (P * P);
    double acc = 0.0;
    for (int o = 0; o < 8; ++o) {
        if (kids[c * 8 + o] < 0) continue;
        const double *wx = w + (o & 1) * P * P + ax * P;
        const double *wy = w + ((o >> 1) & 1) * P * P + ay * P;
        const double *wz = w + (o >> 2) * P * P + az * P;
        const double *m = mc + o * P3;
        for (int kz = 0; kz < P; ++kz)
            for (int ky = 0; ky < P; ++ky) {
                const double wzy = wz[kz] * wy[ky];
                double r = 0.0;
#pragma unroll
                for (int kx = 0; kx < P; ++kx) r += wx[kx] * m[(kz * P + ky) * P + kx];
                acc += wzy * r;
            }
    }
    Mp[(size_t)c * P3 + a] = acc;
}

template <int P>
__global__ __launch_bounds__(256) void k_ml_l2l(const double *__restrict__ Phip, const int *__restrict__ par,
                                                 const double *__restrict__ Wup, double *__restrict__ Phi) {
    constexpr int P3 = P * P * P;
    __shared__ double w[2 * P * P];
    __shared__ double pp[P3];
    const int c = xcd_remap(blockIdx.x, gridDim.x);
    const int pr = par[2 * c], o = par[2 * c + 1];
    for (int i = threadIdx.x; i < 2 * P * P; i += blockDim.x) w[i] = Wup[i];
    for (int i = threadIdx.x; i < P3; i += blockDim.x) pp[i] = Phip[(size_t)pr * P3 + i];
    __syncthreads();
    const int b = threadIdx.x;
    if (b >= P3) return;
    const int bx = b % P, by = (b / P) % P, bz = b / (P * P);
    const double *wx = w + (o & 1) * P * P;
    const double *wy = w + ((o >> 1) & 1) * P * P;
    const double *wz = w + (o >> 2) * P * P;
    double acc = 0.0;
    for (int kz = 0; kz < P; ++kz)
        for (int ky = 0; ky < P; ++ky) {
            const double wzy = wz[kz * P + bz] * wy[ky * P + by];
            double r = 0.0;
#pragma unroll
            for (int kx = 0; kx < P; ++kx) r += wx[kx * P + bx] * pp[(kz * P + ky) * P + kx];
            acc += wzy * r;
        }
    Phi[(size_t)c * P3 + b] += acc;
}

template <int P, typename R>
__global__ __launch_bounds__(256) void k_ml_kmat(const double *__restrict__ tab, int e1, int e2,
                                                  const int4 *__restrict__ dinfo, const int *__restrict__ nodes,
                                                  R *__restrict__ K) {
    constexpr int P3 = P * P * P;
    const int d = blockIdx.x;
    const int4 in = dinfo[d];
    const int *t = nodes + in.w * P;
    for (int i = threadIdx.x; i < P3 * P3; i += blockDim.x) {
        const int b = i / P3, a = i % P3;   // target node b, source node a
        const int ox = abs(in.x + t[b % P] - t[a % P]);
        const int oy = abs(in.y + t[(b / P) % P] - t[(a / P) % P]);
        const int oz = abs(in.z + t[b / (P * P)] - t[a / (P * P)]);
        K[(size_t)d * P3 * P3 + i] = (R)tab[((size_t)oz * (e2 + 1) + oy) * (e1 + 1) + ox];
    }
}

// p = 0 and, where given, *flag = 0
__global__ void k_ml_zero(double *__restrict__ p, size_t n, int *__restrict__ flag) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
    if (i == 0 && flag) *flag = 0;
}

// exact sum of one neighbouring source block into a row of B target cells;
// DX = source block x - target block x, so the x offsets are compile-time
template <int B, int DX>
__device__ __forceinline__ void near_rows(const double *__restrict__ fs, const double *g, int ty, int tz, int DY,
                                          int DZ, double (&acc)[B]) {
    constexpr int G2 = 2 * B;
    for (int sz = 0; sz < B; ++sz) {
        const int dz = abs(tz - sz - B * DZ);
        for (int sy = 0; sy < B; ++sy) {
            const int dy = abs(ty - sy - B * DY);
            const double *gr = g + (dz * G2 + dy) * G2;
            double gv[G2], fv[B];
#pragma unroll
            for (int i = 0; i < G2; ++i) gv[i] = gr[i];
#pragma unroll
            for (int i = 0; i < B; ++i) fv[i] = fs[(sz * B + sy) * B + i];
#pragma unroll
            for (int tx = 0; tx < B; ++tx)
#pragma unroll
                for (int sx = 0; sx < B; ++sx) {
                    const int d = tx - sx - B * DX;
                    acc[tx] += gv[d < 0 ? -d : d] * fv[sx];
                }
        }
    }
}

// near: CSR over target blocks of int2 (source block, 9 (dz+1) + 3 (dy+1) + dx+1)
template <int P, int B, bool NEAR>
__global__ __launch_bounds__(256) void k_ml_leaf(const double *__restrict__ f, const double *__restrict__ tab, int e1,
                                                  int e2, int e3, const int *__restrict__ near_off,
                                                  const int2 *__restrict__ near_ent, const double *__restrict__ Phi0,
                                                  const double *__restrict__ W0, double scale, double *__restrict__ u,
                                                  int ntgt) {
    constexpr int P3 = P * P * P, B3 = B * B * B, R = B * B, TB = 256 / R, G2 = 2 * B;
    __shared__ double g[G2 * G2 * G2];
    __shared__ double w[P * B];
    __shared__ double ph[TB * P3];
    for (int i = threadIdx.x; i < G2 * G2 * G2; i += blockDim.x) {
        const int x = i % G2, y = (i / G2) % G2, z = i / (G2 * G2);
        g[i] = (x <= e1 && y <= e2 && z <= e3) ? tab[((size_t)z * (e2 + 1) + y) * (e1 + 1) + x] : 0.0;
    }
    for (int i = threadIdx.x; i < P * B; i += blockDim.x) w[i] = W0[i];
    const int wg = xcd_remap(blockIdx.x, gridDim.x);
    const int lb = threadIdx.x / R;
    int t = wg * TB + lb;
    if (R % 64 == 0) t = __builtin_amdgcn_readfirstlane(t);
    const int row = threadIdx.x % R;
    if (t < ntgt)
        for (int i = row; i < P3; i += R) ph[lb * P3 + i] = Phi0[(size_t)t * P3 + i];
    __syncthreads();
    if (t >= ntgt) return;
    const int ty = row % B, tz = row / B;
    double acc[B];
#pragma unroll
    for (int i = 0; i < B; ++i) acc[i] = 0.0;
    const double *p = ph + lb * P3;
    for (int bz = 0; bz < P; ++bz)
        for (int by = 0; by < P; ++by) {
            const double wzy = w[bz * B + tz] * w[by * B + ty];
#pragma unroll
            for (int bx = 0; bx < P; ++bx) {
                const double c = wzy * p[(bz * P + by) * P + bx];
#pragma unroll
                for (int tx = 0; tx < B; ++tx) acc[tx] += c * w[bx * B + tx];
            }
        }
    const int e0 = NEAR ? near_off[t] : 0, e1n = NEAR ? near_off[t + 1] : 0;
    for (int e = e0; e < e1n; ++e) {
        const int2 en = near_ent[e];
        const double *fs = f + (size_t)en.x * B3;
        const int DX = en.y % 3 - 1, DY = (en.y / 3) % 3 - 1, DZ = en.y / 9 - 1;
        if (DX < 0) near_rows<B, -1>(fs, g, ty, tz, DY, DZ, acc);
        else if (DX == 0) near_rows<B, 0>(fs, g, ty, tz, DY, DZ, acc);
        else near_rows<B, 1>(fs, g, ty, tz, DY, DZ, acc);
    }
    double *ur = u + (size_t)t * B3 + (size_t)row * B;
#pragma unroll
    for (int tx = 0; tx < B; ++tx) ur[tx] = scale * acc[tx];
}

// ---- exact neighbour sum of 8^3 blocks on the matrix cores
//
// For a neighbour displacement D (source block - target block) the sum is a
// dense 512 x 512 matrix K_D[i][j] = G(x_i - y_j), i a target cell, j a source
// cell, applied to every pair with that displacement.  G is even along each
// axis, so along an axis where D is zero K_D commutes with the reflection of
// the block: split into the even and odd part along every axis,
//   T f = (f(h) + f(7 - h), f(h) - f(7 - h)), h < 4,   T^{-1} = T^T / 2,
// K'_D = T K_D T^{-1} has no entries between the two parities of such an axis.
// With z zero axes the 512 x 512 product falls into 2^z products of edge
// 512 / 2^z: an eighth of the work for the block itself, a quarter for the six
// face neighbours, half for the twelve edge neighbours.  T is additions only.
// The folded order is [parity px + 2 py + 4 pz][hx + 4 hy + 16 hz], so that the
// rows of one product are whole 64-value chunks.

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// axes along which displacement code 9 (DZ + 1) + 3 (DY + 1) + DX + 1 is zero
__host__ __device__ inline int near_zero_axes(int code) {
    return (code % 3 == 1 ? 1 : 0) | ((code / 3) % 3 == 1 ? 2 : 0) | (code / 9 == 1 ? 4 : 0);
}
// parity chunks of product `sub` of a displacement with zero axes zmask, four
// bits each: the parities whose bits in zmask spell sub
__host__ __device__ inline unsigned near_chunks(int zmask, int sub) {
    unsigned out = 0;
    int n = 0;
    for (int pi = 0; pi < 8; ++pi) {
        int key = 0, b = 0;
        for (int a = 0; a < 3; ++a)
            if (zmask >> a & 1) key |= (pi >> a & 1) << b++;
        if (key == sub) out |= (unsigned)pi << (4 * n++);
    }
    return out;
}

// K'_D, product by product: product sub of code at code * 512^2 + sub * N^2, row
// length N = 512 / 2^z.  One workgroup per (row of the folded target, code).  An
// entry is a signed sum over the 64 images of its two cells, which falls into
// one axis after the other: 8192 and 4096 terms a row for x and y and four an
// entry for z, instead of 64 (all 27 codes: 143 -> 73 us).
template <typename R>
__global__ __launch_bounds__(256) void k_ml_near_mats(const double *__restrict__ tab, int e1, int e2, int e3,
                                                       R *__restrict__ Kn) {
    __shared__ double fx[16 * 16 * 8];   // [target and source z][target and source y][px sx]
    __shared__ double fy[16 * 8 * 8];    // [target and source z][py sy][px sx]
    const int code = blockIdx.y, zm = near_zero_axes(code), z = __popc(zm), N = 512 >> z;
    const int sub = blockIdx.x / N, i = blockIdx.x % N, t = threadIdx.x;
    const unsigned ch = near_chunks(zm, sub);
    const int DX = code % 3 - 1, DY = (code / 3) % 3 - 1, DZ = code / 9 - 1;
    const int pt = ch >> (4 * (i / 64)) & 7, tx = i & 3, ty = (i >> 2) & 3, tz = (i >> 4) & 3;
    // places of an axis: target image 8 a + source cell; a = 0, 1 is cell t, 7 - t
    for (int e = t; e < 16 * 16 * 8; e += 256) {
        const int ps = e >> 2 & 1, sx = e & 3, y = e >> 3 & 15, zz = e >> 7;
        const int dy = abs((y & 8 ? 7 - ty : ty) - (y & 7) - 8 * DY), dz = abs((zz & 8 ? 7 - tz : tz) - (zz & 7) - 8 * DZ);
        const double *row = tab + ((size_t)dz * (e2 + 1) + dy) * (e1 + 1);
        double v = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) {
                const int dx = abs((a ? 7 - tx : tx) - (b ? 7 - sx : sx) - 8 * DX);
                const double g = dx <= e1 && dy <= e2 && dz <= e3 ? row[dx] : 0.0;
                v += (a & pt) ^ (b & ps) ? -g : g;
            }
        fx[e] = v;
    }
    __syncthreads();
    for (int e = t; e < 16 * 8 * 8; e += 256) {
        const int x = e & 7, sy = e >> 3 & 3, ps = e >> 5 & 1, zz = e >> 6;
        double v = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) {
                const double g = fx[(zz * 16 + 8 * a + (b ? 7 - sy : sy)) * 8 + x];
                v += (a & pt >> 1) ^ (b & ps) ? -g : g;
            }
        fy[e] = v;
    }
    __syncthreads();
    for (int j = t; j < N; j += 256) {
        const int ps = ch >> (4 * (j / 64)) & 7, sz = (j >> 4) & 3;
        const int xy = ((ps >> 1 & 1) * 4 + ((j >> 2) & 3)) * 8 + (ps & 1) * 4 + (j & 3);
        double v = 0.0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) {
                const double g = fy[(8 * a + (b ? 7 - sz : sz)) * 64 + xy];
                v += (a & pt >> 2) ^ (b & ps >> 2) ? -g : g;
            }
        Kn[((size_t)code * 512 + (size_t)sub * N * N / 512) * 512 + (size_t)i * N + j] = (R)(0.125 * v);
    }
}

// One butterfly of T along an axis of stride s (in cells) for a block in LDS
__device__ __forceinline__ void near_fold_axis(double *b, int s, bool inverse) {
    // 256 pairs (h, 7 - h) of the axis, one per thread: h < 4 and 64 lines
    const int t = threadIdx.x, h = t & 3, line = t >> 2;
    const int base = s == 1 ? line * 8 : s == 8 ? (line >> 3) * 64 + (line & 7) : line;
    // forward: even parts to places 0..3, odd parts to 4..7; inverse: back
    const double x = b[base + h * s], y = b[base + (inverse ? 4 + h : 7 - h) * s];
    __syncthreads();
    b[base + h * s] = x + y;
    b[base + (inverse ? 7 - h : 4 + h) * s] = x - y;
    __syncthreads();
}
// place of the folded block's cell c (axis places 0..7) in the folded order
__device__ __forceinline__ int near_place(int c) {
    const int x = c & 7, y = (c >> 3) & 7, z = c >> 6;
    return (((x >> 2) | (y >> 2) << 1 | (z >> 2) << 2) << 6) | (x & 3) | (y & 3) << 2 | (z & 3) << 4;
}
// Fp = T f for every source block, and zeros in every target block of Yp.
// bad[s]: a folded value of block s is no finite R (an infinity or NaN in f, or
// a sum of finite cells that overflows); bad[nsrc]: of any block
template <typename R>
__global__ __launch_bounds__(256) void k_ml_fold(const double *__restrict__ f, double *__restrict__ Fp,
                                                  double *__restrict__ Yp, int *__restrict__ bad, int nsrc, int ntgt) {
    __shared__ double b[512];
    const int t = threadIdx.x, s = blockIdx.x;
    if (s < ntgt)
        for (int c = t; c < 512; c += 256) Yp[(size_t)s * 512 + c] = 0.0;
    if (s >= nsrc) return;
    for (int c = t; c < 512; c += 256) b[c] = f[(size_t)s * 512 + c];
    __syncthreads();
    near_fold_axis(b, 1, false);
    near_fold_axis(b, 8, false);
    near_fold_axis(b, 64, false);
    bool fin = true;
    for (int c = t; c < 512; c += 256) {
        Fp[(size_t)s * 512 + near_place(c)] = b[c];
        fin = fin && isfinite((R)b[c]);
    }
    const int any = __syncthreads_or(!fin);
    if (t == 0) {
        bad[s] = any;
        if (any) bad[nsrc] = 1;
    }
}

// The neighbour sum of target block t as it stands, without the parities:
// u += scale sum_s sum_j G(x_i - y_j) f_j, in R as the products
template <typename R>
__device__ __noinline__ void near_direct(const double *__restrict__ f, const double *__restrict__ tab, int e1, int e2,
                                         int e3, const int2 *__restrict__ ent, int n, double *__restrict__ u,
                                         double scale, double *b) {
    R acc[2] = {0, 0};
    for (int e = 0; e < n; ++e) {
        const int2 en = ent[e];
        const int DX = en.y % 3 - 1, DY = (en.y / 3) % 3 - 1, DZ = en.y / 9 - 1;
        __syncthreads();
        for (int c = threadIdx.x; c < 512; c += 256) b[c] = f[(size_t)en.x * 512 + c];
        __syncthreads();
        for (int j = 0; j < 512; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = threadIdx.x + 256 * h;
                const int dx = abs((i & 7) - (j & 7) - 8 * DX);
                const int dy = abs((i >> 3 & 7) - (j >> 3 & 7) - 8 * DY);
                const int dz = abs((i >> 6) - (j >> 6) - 8 * DZ);
                const R g = dx <= e1 && dy <= e2 && dz <= e3 ? (R)tab[((size_t)dz * (e2 + 1) + dy) * (e1 + 1) + dx] : (R)0;
                acc[h] += g * (R)b[j];
            }
    }
    for (int h = 0; h < 2; ++h) u[threadIdx.x + 256 * h] += scale * (double)acc[h];
}

// u += scale T^{-1} Yp.  Sums and differences of a block's cells spread an
// infinity as NaN over the block; a target with such a source beside it takes
// the plain sum instead, where it meets each cell on its own.
template <typename R>
__global__ __launch_bounds__(256) void k_ml_unfold(const double *__restrict__ Yp, double *__restrict__ u, double scale,
                                                    const int *__restrict__ near_off, const int2 *__restrict__ near_ent,
                                                    const int *__restrict__ bad, int nsrc, const double *__restrict__ f,
                                                    const double *__restrict__ tab, int e1, int e2, int e3) {
    __shared__ double b[512];
    const int t = threadIdx.x;
    const size_t o = (size_t)blockIdx.x * 512;
    for (int c = t; c < 512; c += 256) b[c] = Yp[o + near_place(c)];
    __syncthreads();
    if (bad[nsrc]) {
        const int n0 = near_off[blockIdx.x], n = near_off[blockIdx.x + 1] - n0;   // n <= 27
        if (__syncthreads_or(t < n && bad[near_ent[n0 + t].x])) {
            near_direct<R>(f, tab, e1, e2, e3, near_ent + n0, n, u + o, scale, b);
            return;
        }
    }
    near_fold_axis(b, 1, true);
    near_fold_axis(b, 8, true);
    near_fold_axis(b, 64, true);
    for (int c = t; c < 512; c += 256) u[o + c] += scale * (0.125 * b[c]);
}

// ---- products of gathered rows on the matrix cores
//
// One tile: C[row][n] = sum_k a(row, k) b(n, k) for 128 rows (pairs) and TN
// columns by 4 TN threads, each wavefront a 32 x 64 part as
// v_mfma_f64_16x16x4f64 products, or v_mfma_f32_16x16x4f32 on request (FP32
// matrix and rounded sources, FP32 accumulation).  a(m, k) and b(n, k) load the
// operands of a thread's place in a slice, out(row, col, value) takes a result.
// Slices of 16 terms and at most 128 registers give two workgroups of eight
// wavefronts a CU; four wavefronts of 64 x 64 need 275 registers, one workgroup
// a CU (neighbour products of the sphere shell: 0.63 against 0.73 ms; four
// wavefronts with two buffers 0.64).
template <int TN, typename R, typename Rows, typename Cols, typename FA, typename FB, typename OUT>
__device__ __forceinline__ void pair_tile(Rows &As, Cols &Bs, int K, const FA &la, const FB &lb, const OUT &out) {
    constexpr bool F64 = std::is_same<R, double>::value;
    using acc_t = typename std::conditional<F64, f64x4, f32x4>::type;
    constexpr int KT = kNearKT, NT = 4 * TN, RS = NT / KT;
    constexpr int FMR = 2, FMC = 4, PA = kNearTile / RS, PB = TN / RS;
    const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int wm = (wave & 3) * 32, wn = (wave >> 2) * 64, kk = tid % KT, row = tid / KT;
    acc_t acc[FMR][FMC];
#pragma unroll
    for (int i = 0; i < FMR; ++i)
#pragma unroll
        for (int j = 0; j < FMC; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
    double ra[PA];
    R rb[PB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int q = 0; q < PA; ++q) ra[q] = la(row + q * RS, k0, kk);
#pragma unroll
        for (int q = 0; q < PB; ++q) rb[q] = lb(row + q * RS, k0, kk);
    };
    auto stage = [&]() {
#pragma unroll
        for (int q = 0; q < PA; ++q) As[row + q * RS][kk] = (R)ra[q];
#pragma unroll
        for (int q = 0; q < PB; ++q) Bs[row + q * RS][kk] = rb[q];
    };
    fetch(0);
    stage();
    __syncthreads();
    // v_mfma_f64_16x16x4f64: lane l holds A[row l%16][k l/16] and B[k l/16][col
    // l%16]; the result D[row l/16 + 4q][col l%16] lands in acc[q]
    const int r = lane % 16, kq = lane / 16;
    for (int k0 = 0; k0 < K; k0 += KT) {
        const bool more = k0 + KT < K;
        if (more) fetch(k0 + KT);
#pragma unroll
        for (int ks = 0; ks < KT; ks += 4) {
            R a[FMR], b[FMC];
#pragma unroll
            for (int i = 0; i < FMR; ++i) a[i] = As[wm + 16 * i + r][ks + kq];
#pragma unroll
            for (int j = 0; j < FMC; ++j) b[j] = Bs[wn + 16 * j + r][ks + kq];
#pragma unroll
            for (int i = 0; i < FMR; ++i)
#pragma unroll
                for (int j = 0; j < FMC; ++j) {
                    if constexpr (F64)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
                }
        }
        __syncthreads();
        if (more) {
            stage();
            __syncthreads();
        }
    }
    const int c = lane % 16, rq = lane / 16;
#pragma unroll
    for (int i = 0; i < FMR; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < FMC; ++j)   // result row of acc[q]: l/16 + 4q for the FP64 form, 4(l/16) + q for FP32
                out(wm + 16 * i + (F64 ? rq + 4 * q : 4 * rq + q), wn + 16 * j, c, (double)acc[i][j][q]);
}

// rows (target, source) of a task's pairs; rows past them read source 0 and
// are not stored
__device__ __forceinline__ void pair_rows(const int2 *__restrict__ pairs, int np, int *trow, int *srow) {
    for (int m = threadIdx.x; m < kNearTile; m += blockDim.x) {
        const int2 pr = m < np ? pairs[m] : make_int2(-1, 0);
        trow[m] = pr.x;
        srow[m] = pr.y;
    }
    __syncthreads();
}

// One product of the folded neighbour sum for up to 128 pairs of a displacement:
// C[pair][n] = sum_k Fp[src(pair)][k] K'[n][k], added atomically into Yp (a
// target receives up to 27 displacements).  tasks: int4 (matrix offset / 4096,
// first pair, pair count | column tile << 8 | z << 16, parity chunks).  Bound by
// the matrix cores: 31.7 GFLOP in 0.70 ms for the 6344 blocks of a sphere shell
// of diameter 256, where the unfolded matrices took 58.5 GFLOP and 1.33 ms (FP64
// atomics or plain stores: no difference).
template <int TN, typename R>
__global__ __launch_bounds__(4 * TN, TN == 128 ? 4 : 2) void k_ml_near(const int4 *__restrict__ tasks,
                                                                       const int2 *__restrict__ pairs,
                                                                       const double *__restrict__ X,
                                                                       const R *__restrict__ Kn,
                                                                       double *__restrict__ Y) {
    __shared__ R As[kNearTile][kNearKT + 1];   // [pair][k]
    __shared__ R Bs[TN][kNearKT + 1];          // [n][k]
    __shared__ int srow[kNearTile], trow[kNearTile];
    const int4 tk = tasks[blockIdx.x];
    const int n0 = (tk.z >> 8 & 255) * TN, N = 512 >> (tk.z >> 16);
    const unsigned ch = (unsigned)tk.w;
    const R *A = Kn + (size_t)tk.x * 4096 + (size_t)n0 * N;
    pair_rows(pairs + tk.y, tk.z & 255, trow, srow);
    // a slice, and 16 columns, lie in one parity chunk
    auto chunk = [&](int k) { return (int)(ch >> (4 * (k / 64)) & 7) * 64 + k % 64; };
    pair_tile<TN, R>(
        As, Bs, N, [&](int m, int k0, int kk) { return X[(size_t)srow[m] * 512 + (chunk(k0) + kk)]; },
        [&](int n, int k0, int kk) { return A[n * N + k0 + kk]; },
        [&](int m, int n, int c, double v) {
            const int t = trow[m];
            if (t >= 0) unsafeAtomicAdd(&Y[(size_t)t * 512 + chunk(n0 + n) + c], v);
        });
}

// M2L: C[pair][n] = sum_k M[src(pair)][k] A_d[n][k] with the node matrix A_d
// (NB x NB, NB = p^3) of a displacement, added atomically into Phi.  tasks:
// int4 (displacement, first pair, pair count, column tile); one launch for the
// pairs of every level.  Gathers, atomics and products
// about alike: the 481,568 pairs of the sphere shell of diameter 256 at p = 4
// in 0.20 ms, against 0.24 level by level (0.16 with plain stores)
template <int NB, typename R>
__global__ __launch_bounds__(NB <= 64 ? 256 : 512, NB <= 64 ? 2 : 4) void k_ml_m2l(const int4 *__restrict__ tasks,
                                                                                 const int2 *__restrict__ pairs,
                                                                                 const double *__restrict__ M,
                                                                                 const R *__restrict__ Amat,
                                                                                 double *__restrict__ Phi) {
    constexpr int TN = NB <= 64 ? 64 : 128;
    __shared__ R As[kNearTile][kNearKT + 1];   // [pair][k]
    __shared__ R Bs[TN][kNearKT + 1];          // [n][k]
    __shared__ int srow[kNearTile], trow[kNearTile];
    const int4 tk = tasks[blockIdx.x];
    const int n0 = tk.w * TN;
    const R *A = Amat + (size_t)tk.x * NB * NB;
    pair_rows(pairs + tk.y, tk.z, trow, srow);
    constexpr bool whole = NB % TN == 0;   // else the last slice and column tile are filled with zeros
    pair_tile<TN, R>(
        As, Bs, NB,
        [&](int m, int k0, int kk) {
            const int k = k0 + kk;
            const double v = M[(size_t)srow[m] * NB + (whole ? k : min(k, NB - 1))];
            return whole || k < NB ? v : 0.0;
        },
        [&](int n, int k0, int kk) {
            const int k = k0 + kk, nn = n0 + n;
            const R v = A[(whole ? nn : min(nn, NB - 1)) * NB + (whole ? k : min(k, NB - 1))];
            return whole || (nn < NB && k < NB) ? v : (R)0;
        },
        [&](int m, int n, int c, double v) {
            const int t = trow[m];
            if (t >= 0 && (whole || n0 + n + c < NB)) unsafeAtomicAdd(&Phi[(size_t)t * NB + n0 + n + c], v);
        });
}

}  // namespace
}  // namespace lgfib

using namespace lgfib;

struct lgf_ml {
    lgfib_ctx *ctx = nullptr;
    int device = 0;   // the context's device (destroy does not touch ctx)
    lgf_table_t tbl = -1;
    int B = 0, P = 0, top = 0, nsrc = 0, ntgt = 0;
    std::vector<int> ns, nt;            // clusters per level
    std::vector<size_t> m_off, t_off;   // first cluster of each level in M / Phi
    std::vector<size_t> kid_off;        // first parent row of each level's M2M map
    int nm2l = 0;                       // M2L tasks
    int64_t npairs = 0, nnear = 0, nd = 0;
    DevBuf W0, Wup, kids, par, tasks, pairs, K, near_off, near_ent, M, Phi, dinfo, nodes;
    int nntask[2] = {0, 0};             // B = 8: neighbour products on the matrix cores, 128 and 64 columns wide
    int pair_prec = LGF_F64;            // precision of the pair products (M2L, neighbour sums)
    DevBuf nbr_tasks, nbr_pairs, Kn, folded;   // folded: sources, targets, then bad
    int *bad = nullptr;                 // marks by source block, then any
};

namespace {

template <int P, int B>
int ml_run(lgf_ml *pl, int ncomp, double dx, const double *f, double *u, hipStream_t st) {
    constexpr int P3 = P * P * P, B3 = B * B * B, TB = 256 / (B * B);
    lgfib_ctx *ctx = pl->ctx;
    const Table &tb = *ctx->tables[pl->tbl];
    double *M = pl->M.as<double>(), *Phi = pl->Phi.as<double>();
    const double *Wup = pl->Wup.as<double>();
    for (int c = 0; c < ncomp; ++c) {
        const double *fc = f + (size_t)c * pl->nsrc * B3;
        double *uc = u + (size_t)c * pl->ntgt * B3;
        {
            ProfScope ps(ctx, "k_ml_p2m", st);
            hipLaunchKernelGGL((k_ml_p2m<P, B>), dim3(pl->nsrc), dim3(256), 0, st, fc, pl->W0.as<double>(), M);
            LGF_HIP(hipGetLastError());
        }
        for (int l = 0; l < pl->top; ++l) {
            ProfScope ps(ctx, "k_ml_m2m", st);
            hipLaunchKernelGGL((k_ml_m2m<P>), dim3(pl->ns[l + 1]), dim3(P3 <= 128 ? 128 : 256), 0, st, M + pl->m_off[l] * P3,
                               pl->kids.as<int>() + pl->kid_off[l] * 8, Wup + (size_t)l * 2 * P * P,
                               M + pl->m_off[l + 1] * P3);
            LGF_HIP(hipGetLastError());
        }
        const size_t nphi = (pl->t_off[pl->top] + pl->nt[pl->top]) * P3;
        hipLaunchKernelGGL(k_ml_zero, dim3((unsigned)((nphi + 255) / 256)), dim3(256), 0, st, Phi, nphi,
                           pl->bad ? pl->bad + pl->nsrc : nullptr);
        LGF_HIP(hipGetLastError());
        if (pl->nm2l > 0) {
            ProfScope ps(ctx, "k_ml_m2l", st);
            const dim3 g(pl->nm2l), b(P3 <= 64 ? 256 : 512);
            if (pl->pair_prec == LGF_F64)
                hipLaunchKernelGGL((k_ml_m2l<P3, double>), g, b, 0, st, pl->tasks.as<int4>(), pl->pairs.as<int2>(), M,
                                   pl->K.as<double>(), Phi);
            else
                hipLaunchKernelGGL((k_ml_m2l<P3, float>), g, b, 0, st, pl->tasks.as<int4>(), pl->pairs.as<int2>(), M,
                                   pl->K.as<float>(), Phi);
            LGF_HIP(hipGetLastError());
        }
        for (int l = pl->top - 1; l >= 0; --l) {
            ProfScope ps(ctx, "k_ml_l2l", st);
            hipLaunchKernelGGL((k_ml_l2l<P>), dim3(pl->nt[l]), dim3(P3 <= 128 ? 128 : 256), 0, st, Phi + pl->t_off[l + 1] * P3,
                               pl->par.as<int>() + 2 * pl->t_off[l], Wup + (size_t)l * 2 * P * P,
                               Phi + pl->t_off[l] * P3);
            LGF_HIP(hipGetLastError());
        }
        {
            ProfScope ps(ctx, "k_ml_leaf", st);
            hipLaunchKernelGGL((k_ml_leaf<P, B, B != 8>), dim3((pl->ntgt + TB - 1) / TB), dim3(256), 0, st, fc,
                               tb.g.as<double>(), tb.ext[0], tb.ext[1], tb.ext[2], pl->near_off.as<int>(),
                               pl->near_ent.as<int2>(), Phi, pl->W0.as<double>(), dx * dx, uc, pl->ntgt);
            LGF_HIP(hipGetLastError());
        }
        if (B == 8 && pl->nntask[0] + pl->nntask[1] > 0) {
            double *Fp = pl->folded.as<double>(), *Yp = Fp + (size_t)pl->nsrc * 512;
            ProfScope ps(ctx, "k_ml_near_mfma", st);
            const int4 *tk = pl->nbr_tasks.as<int4>();
            const int2 *pr = pl->nbr_pairs.as<int2>();
            auto run = [&](auto *Kn) {
                using R = std::remove_reference_t<decltype(*Kn)>;
                const dim3 g0(pl->nntask[0]), g1(pl->nntask[1]), b(256);
                hipLaunchKernelGGL(k_ml_fold<R>, dim3(std::max(pl->nsrc, pl->ntgt)), b, 0, st, fc, Fp, Yp,
                                   pl->bad, pl->nsrc, pl->ntgt);
                if (g0.x) hipLaunchKernelGGL((k_ml_near<128, R>), g0, dim3(512), 0, st, tk, pr, Fp, Kn, Yp);
                if (g1.x) hipLaunchKernelGGL((k_ml_near<64, R>), g1, b, 0, st, tk + g0.x, pr, Fp, Kn, Yp);
                hipLaunchKernelGGL(k_ml_unfold<R>, dim3(pl->ntgt), b, 0, st, Yp, uc, dx * dx, pl->near_off.as<int>(),
                                   pl->near_ent.as<int2>(), pl->bad, pl->nsrc, fc, tb.g.as<double>(), tb.ext[0],
                                   tb.ext[1], tb.ext[2]);
            };
            if (pl->pair_prec == LGF_F64) run(pl->Kn.as<double>());
            else run(pl->Kn.as<float>());
            LGF_HIP(hipGetLastError());
        }
    }
    return LGFIB_OK;
}

// Launch order of tasks (four ints each, groups of falling cost): workgroup b
// runs on XCD b % 8, and each XCD takes an eighth of every group, consecutive
// tasks of it (mostly one displacement, so its L2 keeps the matrix they share).
// Eighths of the whole list instead leave the XCDs with unequal work: the
// neighbour products of a sphere shell kept the CUs busy 79 % of the time.
std::vector<int32_t> spread_tasks(const std::vector<std::vector<int32_t>> &groups) {
    std::vector<int32_t> q[8], out;
    size_t longest = 0;
    for (const auto &g : groups) {
        const size_t n = g.size() / 4;
        for (size_t x = 0; x < 8; ++x) q[x].insert(q[x].end(), g.begin() + n * x / 8 * 4, g.begin() + n * (x + 1) / 8 * 4);
    }
    for (const auto &v : q) longest = std::max(longest, v.size());
    for (size_t i = 0; i < longest; i += 4)
        for (const auto &v : q)
            if (i < v.size()) out.insert(out.end(), v.begin() + i, v.begin() + i + 4);
    return out;
}

template <typename T> int upload(DevBuf &d, const std::vector<T> &v) {
    if (v.empty()) return LGFIB_OK;
    int rc = d.reserve(v.size() * sizeof(T));
    if (rc) return rc;
    LGF_HIP(hipMemcpy(d.p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
    return LGFIB_OK;
}

}  // namespace

extern "C" int lgf_ml_create(lgfib_ctx *ctx, lgf_table_t tbl, int B, int p, int pair_prec, const int32_t *src_blocks,
                             int nsrc, const int32_t *tgt_blocks, int ntgt, lgfib_stream_t stream, lgf_ml_t **out) {
    if (!out) return fail(LGFIB_EINVAL, "lgf_ml_create: null output");
    *out = nullptr;
    if (!ctx) return fail(LGFIB_EINVAL, "lgf_ml_create: null context");
    if (tbl < 0 || (size_t)tbl >= ctx->tables.size()) return fail(LGFIB_ENOTBUILT, "lgf_ml_create: unknown table");
    if (B != 4 && B != 8) return fail(LGFIB_EINVAL, "lgf_ml_create: B must be 4 or 8");
    if (p < 4 || p > 6 || p > B) return fail(LGFIB_EINVAL, "lgf_ml_create: p must be 4, 5 or 6 and at most B");
    if (pair_prec != LGF_F64 && (pair_prec != LGF_F32 || B != 8))
        return fail(LGFIB_EINVAL, "lgf_ml_create: pair_prec must be LGF_F64, or LGF_F32 with B = 8");
    int rc;
    if ((rc = validate_blocks(src_blocks, nsrc, "lgf_ml_create: source blocks"))) return rc;
    if ((rc = validate_blocks(tgt_blocks, ntgt, "lgf_ml_create: target blocks"))) return rc;
    LGF_HIP(hipSetDevice(ctx->device));
    auto pl = std::make_unique<lgf_ml>();
    pl->ctx = ctx;
    pl->device = ctx->device;
    pl->tbl = tbl;
    pl->B = B;
    pl->P = p;
    pl->pair_prec = pair_prec;
    pl->nsrc = nsrc;
    pl->ntgt = ntgt;
    if (nsrc == 0 || ntgt == 0) {
        *out = pl.release();
        return LGFIB_OK;
    }
    const Table &tb = *ctx->tables[tbl];
    // top level and the table reach
    int lo[3], hi[3];
    for (int a = 0; a < 3; ++a) lo[a] = hi[a] = src_blocks[a];
    for (int i = 0; i < nsrc + ntgt; ++i) {
        const int32_t *b = i < nsrc ? src_blocks + 3 * i : tgt_blocks + 3 * (i - nsrc);
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], b[a]);
            hi[a] = std::max(hi[a], b[a]);
        }
    }
    int top = 0;
    for (;;) {
        bool ok = true;
        for (int a = 0; a < 3; ++a) ok = ok && (hi[a] >> top) - (lo[a] >> top) + 1 <= kTopSpan;
        if (ok) break;
        ++top;
    }
    for (int a = 0; a < 3; ++a) {
        const long need = (long)((hi[a] >> top) - (lo[a] >> top) + 1) * ((long)B << top) - 1;
        if (need > tb.ext[a])
            return fail(LGFIB_ERANGE, "lgf_ml_create: table extent " + std::to_string(tb.ext[a]) + " on axis " +
                                          std::to_string(a) + " is short of " + std::to_string(need));
    }
    pl->top = top;
    std::vector<std::vector<int>> nodes(top + 1);
    for (int l = 0; l <= top; ++l) {
        nodes[l] = cluster_nodes(B << l, p);
        if (nodes[l].empty()) return fail(LGFIB_EINVAL, "lgf_ml_create: interpolation nodes coincide");
    }
    // clusters per level
    std::vector<std::vector<CKey>> sc(top + 1), tc(top + 1);
    std::vector<CMap> smap(top + 1), tmap(top + 1);
    for (int i = 0; i < nsrc; ++i) {
        CKey k{src_blocks[3 * i], src_blocks[3 * i + 1], src_blocks[3 * i + 2]};
        smap[0][k] = i;
        sc[0].push_back(k);
    }
    for (int i = 0; i < ntgt; ++i) {
        CKey k{tgt_blocks[3 * i], tgt_blocks[3 * i + 1], tgt_blocks[3 * i + 2]};
        tmap[0][k] = i;
        tc[0].push_back(k);
    }
    std::vector<int32_t> kids, par;
    for (int l = 0; l < top; ++l) {
        for (const CKey &c : sc[l]) {
            const CKey q = parent_of(c);
            if (smap[l + 1].emplace(q, (int)sc[l + 1].size()).second) sc[l + 1].push_back(q);
        }
        const size_t k0 = kids.size();
        kids.resize(k0 + 8 * sc[l + 1].size(), -1);
        for (size_t i = 0; i < sc[l].size(); ++i)
            kids[k0 + 8 * (size_t)smap[l + 1][parent_of(sc[l][i])] + octant_of(sc[l][i])] = (int32_t)i;
        for (const CKey &c : tc[l]) {
            const CKey q = parent_of(c);
            if (tmap[l + 1].emplace(q, (int)tc[l + 1].size()).second) tc[l + 1].push_back(q);
        }
    }
    for (int l = 0; l <= top; ++l) {   // parent map of the targets (unused at the top)
        for (const CKey &c : tc[l]) {
            par.push_back(l < top ? tmap[l + 1][parent_of(c)] : -1);
            par.push_back(octant_of(c));
        }
    }
    size_t ms = 0, ts = 0, ks = 0;
    for (int l = 0; l <= top; ++l) {
        pl->ns.push_back((int)sc[l].size());
        pl->nt.push_back((int)tc[l].size());
        pl->m_off.push_back(ms);
        pl->t_off.push_back(ts);
        pl->kid_off.push_back(ks);
        ms += sc[l].size();
        ts += tc[l].size();
        if (l < top) ks += sc[l + 1].size();
    }
    // interaction lists, grouped by displacement
    std::vector<int32_t> pairs;
    std::vector<std::vector<int32_t>> m2l_groups;        // tasks by level
    const int ytiles = (p * p * p + 127) / 128;          // k_ml_m2l's column tiles
    std::vector<int32_t> dinfo;
    for (int l = 0; l <= top; ++l) {
        // rows of all levels in one numbering, so that one launch takes them
        const int32_t t0 = (int32_t)pl->t_off[l], s0 = (int32_t)pl->m_off[l];
        std::vector<std::vector<int32_t>> byd(343);
        auto add = [&](int ti, int si, const CKey &c, const CKey &s) {
            const int Dx = c.x - s.x, Dy = c.y - s.y, Dz = c.z - s.z;
            auto &v = byd[(Dz + 3) * 49 + (Dy + 3) * 7 + Dx + 3];
            v.push_back(t0 + ti);
            v.push_back(s0 + si);
        };
        for (int ti = 0; ti < (int)tc[l].size(); ++ti) {
            const CKey c = tc[l][ti];
            if (l == top) {
                for (int si = 0; si < (int)sc[l].size(); ++si)
                    if (!adjacent(sc[l][si], c)) add(ti, si, c, sc[l][si]);
                continue;
            }
            const CKey pc = parent_of(c);
            for (int dz = -1; dz <= 1; ++dz)
                for (int dy = -1; dy <= 1; ++dy)
                    for (int dx = -1; dx <= 1; ++dx) {
                        const CKey q{pc.x + dx, pc.y + dy, pc.z + dz};
                        auto it = smap[l + 1].find(q);
                        if (it == smap[l + 1].end()) continue;
                        const int32_t *kk = kids.data() + pl->kid_off[l] * 8 + 8 * (size_t)it->second;
                        for (int o = 0; o < 8; ++o) {
                            if (kk[o] < 0) continue;
                            const CKey &s = sc[l][kk[o]];
                            if (!adjacent(s, c)) add(ti, kk[o], c, s);
                        }
                    }
        }
        std::vector<int32_t> ltasks;
        for (int di = 0; di < 343; ++di) {
            const auto &v = byd[di];
            if (v.empty()) continue;
            const int Dx = di % 7 - 3, Dy = (di / 7) % 7 - 3, Dz = di / 49 - 3;
            const int L = B << l;
            const int d = (int)(dinfo.size() / 4);
            dinfo.insert(dinfo.end(), {Dx * L, Dy * L, Dz * L, l});
            const int np = (int)(v.size() / 2);
            for (int ct = 0; ct < ytiles; ++ct)
                for (int q = 0; q < np; q += kNearTile)
                    ltasks.insert(ltasks.end(),
                                  {d, (int32_t)(pairs.size() / 2) + q, std::min(kNearTile, np - q), ct});
            pairs.insert(pairs.end(), v.begin(), v.end());
        }
        m2l_groups.push_back(std::move(ltasks));
    }
    const std::vector<int32_t> tasks = spread_tasks(m2l_groups);
    pl->nm2l = (int)(tasks.size() / 4);
    pl->npairs = (int64_t)(pairs.size() / 2);
    pl->nd = (int64_t)(dinfo.size() / 4);
    // neighbour lists of the target blocks
    std::vector<int32_t> near_off(1, 0), near_ent;
    for (int ti = 0; ti < ntgt; ++ti) {
        const CKey c = tc[0][ti];
        for (int dz = -1; dz <= 1; ++dz)
            for (int dy = -1; dy <= 1; ++dy)
                for (int dx = -1; dx <= 1; ++dx) {
                    auto it = smap[0].find(CKey{c.x + dx, c.y + dy, c.z + dz});
                    if (it == smap[0].end()) continue;
                    near_ent.push_back(it->second);
                    near_ent.push_back((dz + 1) * 9 + (dy + 1) * 3 + dx + 1);
                }
        near_off.push_back((int32_t)(near_ent.size() / 2));
    }
    pl->nnear = (int64_t)(near_ent.size() / 2);
    std::vector<int32_t> ntasks[2], npairs;
    if (B == 8) {
        std::vector<std::vector<int32_t>> byc(27);
        for (int ti = 0; ti < ntgt; ++ti)
            for (int e = near_off[ti]; e < near_off[ti + 1]; ++e) {
                byc[near_ent[2 * e + 1]].push_back(ti);
                byc[near_ent[2 * e + 1]].push_back(near_ent[2 * e]);
            }
        // products of full and half edge in tiles of 128 columns, the others
        // (edge 128 and 64) in tiles of 64
        std::vector<int32_t> first(27);
        for (int code = 0; code < 27; ++code) {
            first[code] = (int32_t)(npairs.size() / 2);
            npairs.insert(npairs.end(), byc[code].begin(), byc[code].end());
        }
        std::vector<std::vector<int32_t>> groups[2] = {std::vector<std::vector<int32_t>>(4),
                                                       std::vector<std::vector<int32_t>>(4)};   // by z
        for (int code = 0; code < 27; ++code) {
            const int zm = near_zero_axes(code), z = __builtin_popcount(zm), N = 512 >> z;
            const int TN = z < kNearNarrow ? 128 : 64, np = (int)(byc[code].size() / 2);
            auto &g = groups[TN == 64][z];
            for (int sub = 0; sub < 1 << z; ++sub)
                for (int ct = 0; ct < N / TN; ++ct)
                    for (int s0 = 0; s0 < np; s0 += kNearTile)
                        g.insert(g.end(), {code * 64 + sub * N * N / 4096, first[code] + s0,
                                           std::min(kNearTile, np - s0) | ct << 8 | z << 16,
                                           (int32_t)near_chunks(zm, sub)});
        }
        for (int w = 0; w < 2; ++w) {
            ntasks[w] = spread_tasks(groups[w]);
            pl->nntask[w] = (int)(ntasks[w].size() / 4);
        }
        ntasks[0].insert(ntasks[0].end(), ntasks[1].begin(), ntasks[1].end());
    }
    // interpolation weights
    std::vector<double> W0((size_t)p * B), Wup((size_t)std::max(top, 1) * 2 * p * p);
    for (int j = 0; j < p; ++j)
        for (int x = 0; x < B; ++x) W0[(size_t)j * B + x] = lagrange(nodes[0], j, x);
    for (int l = 0; l < top; ++l)
        for (int o = 0; o < 2; ++o)
            for (int j = 0; j < p; ++j)
                for (int k = 0; k < p; ++k)
                    Wup[(((size_t)l * 2 + o) * p + j) * p + k] =
                        lagrange(nodes[l + 1], j, (double)o * (B << l) + nodes[l][k]);
    std::vector<int32_t> nodes_flat;
    for (int l = 0; l <= top; ++l) nodes_flat.insert(nodes_flat.end(), nodes[l].begin(), nodes[l].end());
    const size_t P3 = (size_t)p * p * p;
    if ((rc = upload(pl->W0, W0)) || (rc = upload(pl->Wup, Wup)) || (rc = upload(pl->kids, kids)) ||
        (rc = upload(pl->par, par)) || (rc = upload(pl->tasks, tasks)) || (rc = upload(pl->pairs, pairs)) ||
        (rc = upload(pl->near_off, near_off)) || (rc = upload(pl->near_ent, near_ent)) ||
        (rc = upload(pl->dinfo, dinfo)) || (rc = upload(pl->nodes, nodes_flat)) ||
        (rc = upload(pl->nbr_tasks, ntasks[0])) || (rc = upload(pl->nbr_pairs, npairs)))
        return rc;
    if (pl->nntask[0] + pl->nntask[1] > 0) {
        const size_t folded = ((size_t)nsrc + ntgt) * 512 * sizeof(double);
        if ((rc = pl->folded.reserve(folded + ((size_t)nsrc + 1) * sizeof(int)))) return rc;
        pl->bad = (int *)((char *)pl->folded.p + folded);
        const bool f64 = pair_prec == LGF_F64;
        if ((rc = pl->Kn.reserve((size_t)27 * 512 * 512 * (f64 ? sizeof(double) : sizeof(float))))) return rc;
        if (f64)
            hipLaunchKernelGGL(k_ml_near_mats<double>, dim3(512, 27), dim3(256), 0, (hipStream_t)stream,
                               tb.g.as<double>(), tb.ext[0], tb.ext[1], tb.ext[2], pl->Kn.as<double>());
        else
            hipLaunchKernelGGL(k_ml_near_mats<float>, dim3(512, 27), dim3(256), 0, (hipStream_t)stream,
                               tb.g.as<double>(), tb.ext[0], tb.ext[1], tb.ext[2], pl->Kn.as<float>());
        LGF_HIP(hipGetLastError());
        LGF_HIP(hipStreamSynchronize((hipStream_t)stream));
    }
    if ((rc = pl->M.reserve(ms * P3 * sizeof(double))) || (rc = pl->Phi.reserve(ts * P3 * sizeof(double))))
        return rc;
    if (pl->nd > 0) {
        const bool f64 = pair_prec == LGF_F64;
        if ((rc = pl->K.reserve((size_t)pl->nd * P3 * P3 * (f64 ? sizeof(double) : sizeof(float))))) return rc;
        hipStream_t st = (hipStream_t)stream;
        const dim3 g((unsigned)pl->nd), b(256);
        const int4 *di = pl->dinfo.as<int4>();
        const int *nd = pl->nodes.as<int>();
        const double *tg = tb.g.as<double>();
        if (f64) {
            auto kmat = p == 4 ? k_ml_kmat<4, double> : p == 5 ? k_ml_kmat<5, double> : k_ml_kmat<6, double>;
            hipLaunchKernelGGL(kmat, g, b, 0, st, tg, tb.ext[0], tb.ext[1], di, nd, pl->K.as<double>());
        } else {
            auto kmat = p == 4 ? k_ml_kmat<4, float> : p == 5 ? k_ml_kmat<5, float> : k_ml_kmat<6, float>;
            hipLaunchKernelGGL(kmat, g, b, 0, st, tg, tb.ext[0], tb.ext[1], di, nd, pl->K.as<float>());
        }
        LGF_HIP(hipGetLastError());
        LGF_HIP(hipStreamSynchronize(st));
    }
    *out = pl.release();
    return LGFIB_OK;
}

extern "C" int lgf_ml_apply(lgfib_ctx *ctx, lgf_ml_t *pl, int ncomp, double dx, const double *f, double *u,
                            lgfib_stream_t stream) {
    if (!ctx || !pl) return fail(LGFIB_EINVAL, "lgf_ml_apply: null argument");
    if (pl->ctx != ctx) return fail(LGFIB_EINVAL, "lgf_ml_apply: the plan belongs to another context");
    if (ncomp < 1 || ncomp > 8) return fail(LGFIB_EINVAL, "lgf_ml_apply: ncomp must lie in [1, 8]");
    if (!(dx > 0.0) || !std::isfinite(dx)) return fail(LGFIB_EINVAL, "lgf_ml_apply: dx must be positive");
    const size_t B3 = (size_t)pl->B * pl->B * pl->B;
    if (pl->ntgt == 0) return LGFIB_OK;
    if (!u) return fail(LGFIB_EINVAL, "lgf_ml_apply: null output");
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const size_t ubytes = (size_t)ncomp * pl->ntgt * B3 * sizeof(double);
    if (pl->nsrc == 0) {
        LGF_HIP(hipMemsetAsync(u, 0, ubytes, st));
        return LGFIB_OK;
    }
    if (!f) return fail(LGFIB_EINVAL, "lgf_ml_apply: null input");
    const size_t fbytes = (size_t)ncomp * pl->nsrc * B3 * sizeof(double);
    const char *a = (const char *)f, *b = (const char *)u;
    if (a < b + ubytes && b < a + fbytes) return fail(LGFIB_EINVAL, "lgf_ml_apply: f and u overlap");
    if (pl->B == 4) return ml_run<4, 4>(pl, ncomp, dx, f, u, st);
    if (pl->P == 4) return ml_run<4, 8>(pl, ncomp, dx, f, u, st);
    if (pl->P == 5) return ml_run<5, 8>(pl, ncomp, dx, f, u, st);
    return ml_run<6, 8>(pl, ncomp, dx, f, u, st);
}

extern "C" int lgf_ml_info(const lgf_ml_t *pl, int64_t out[6]) {
    if (!pl || !out) return fail(LGFIB_EINVAL, "lgf_ml_info: null argument");
    int64_t ns = 0, nt = 0;
    for (int v : pl->ns) ns += v;
    for (int v : pl->nt) nt += v;
    out[0] = pl->top;
    out[1] = ns;
    out[2] = nt;
    out[3] = pl->npairs;
    out[4] = pl->nnear;
    out[5] = pl->nd;
    return LGFIB_OK;
}

extern "C" void lgf_ml_destroy(lgf_ml_t *pl) {
    if (!pl) return;
    (void)hipSetDevice(pl->device);
    delete pl;
}
