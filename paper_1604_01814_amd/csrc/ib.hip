// ib.hip -- immersed-boundary operators on a block set: discrete delta
// regularization R and interpolation I (Sec. 2.1), the staggered gradient G
// and its adjoint G^T, and the body-block set D_body (Sec. 4.1).
//
// Positions are in lattice units; cell n has centre n + (1/2,1/2,1/2) and its
// k-th face sits at x_F^(k)(n) = n + (1/2,1/2,1/2) - e_k/2.
//
// Marker positions are fixed for a plan (a rigid body in its own frame), so
// both operators are assembled once on the host as sparse matrices with the
// tensor-product delta weights: I as rows (marker, component) over face
// indices, R as rows (face) over (marker, component) entries, each row in
// ascending column order.  Applying either is then one gather per output
// (deterministic, no atomics): a thread per face for R, a thread per
// (marker, component) for I.
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <unordered_map>

#include "internal.h"

namespace lgfib {

// ------------------------------------------------------------- kernels phi

// Roma, Peskin & Berger (1999): support |r| < 3/2.
__host__ __device__ inline double phi_roma3(double r) {
    const double a = fabs(r);
    if (a <= 0.5) return (1.0 + sqrt(1.0 - 3.0 * a * a)) / 3.0;
    if (a <= 1.5) {
        const double b = 1.0 - a;
        return (5.0 - 3.0 * a - sqrt(fmax(0.0, 1.0 - 3.0 * b * b))) / 6.0;
    }
    return 0.0;
}

// Its convolution with the unit top-hat (Yang et al. 2009): support |r| < 2.
__host__ __device__ inline double phi_smooth3(double r) {
    const double a = fabs(r);
    const double s3 = 1.7320508075688772935;
    const double pi = 3.14159265358979323846;
    if (a <= 1.0) {
        return 17.0 / 48.0 + s3 * pi / 108.0 + a / 4.0 - a * a / 4.0 +
               (1.0 - 2.0 * a) / 16.0 * sqrt(fmax(0.0, -12.0 * a * a + 12.0 * a + 1.0)) -
               s3 / 12.0 * asin(fmin(1.0, fmax(-1.0, s3 / 2.0 * (2.0 * a - 1.0))));
    }
    if (a <= 2.0) {
        return 55.0 / 48.0 - s3 * pi / 108.0 - 13.0 * a / 12.0 + a * a / 4.0 +
               (2.0 * a - 3.0) / 48.0 * sqrt(fmax(0.0, -12.0 * a * a + 36.0 * a - 23.0)) +
               s3 / 36.0 * asin(fmin(1.0, fmax(-1.0, s3 / 2.0 * (2.0 * a - 3.0))));
    }
    return 0.0;
}

__host__ __device__ inline double phi_k(int kernel, double r) {
    return kernel == IB_ROMA3 ? phi_roma3(r) : phi_smooth3(r);
}

__host__ __device__ inline double half_width(int kernel) { return kernel == IB_ROMA3 ? 1.5 : 2.0; }

// ----------------------------------------------------------- host staging

static inline long long floordiv(long long a, long long b) {
    long long q = a / b;
    if ((a % b != 0) && ((a < 0) != (b < 0))) --q;
    return q;
}

// lowest lattice index n_j with phi(n_j + c - X) != 0 possible, and count
static inline void support_range(int kernel, double X, double c, long long *lo, int *cnt) {
    const double hw = half_width(kernel);
    *lo = (long long)floor(X - c - hw) + 1;
    *cnt = (int)(2 * hw) + 1;
}

// R and G^T R as one sparse operator on marker vectors: the rows are the nfr
// faces and then the cells that some marker reaches; row[q] is row q's face or
// cell.  Up to three entries for each one of I, so ptr holds 64 bits.
struct SpreadOp {
    int nfr = 0, nrows = 0;
    DevBuf row, ptr, col, val;
};
// The operators of a force system with the gradient folded in: the spread on the
// plan's own blocks, and the cell below the face of entry e of I along its
// component, -1 outside the blocks (i_low[e])
struct GradOps {
    SpreadOp spread;
    DevBuf i_low;
};
// The spread operator of a flow (the plan's faces, the flow's cells) and its
// outputs, R f and G^T R f, which nothing else writes: zeros where no marker
// reaches.  A step of a flow is done with them before it returns.
struct FlowOps {
    SpreadOp spread;
    DevBuf rf, cf;
};

struct IbPlan {
    int kernel = 0, NL = 0, B = 0, nblk = 0;
    int lo[3] = {0, 0, 0}, nb[3] = {0, 0, 0};   // block-map box
    DevBuf X;          // double [NL][3]
    DevBuf map;        // int32 [nb2][nb1][nb0] -> slot or -1
    DevBuf blocks;     // int32 [nblk][3]
    // I: rows 3 i + k -> (face index, weight);  R: rows face -> (3 i + k, weight)
    DevBuf i_ptr, i_col, i_val;
    DevBuf r_ptr, r_col, r_val;
    int64_t nnz = 0;
    // on the host: the faces that some marker reaches, and the end of each one's
    // row of R
    std::vector<int32_t> face, fend;
    // what the plan's force systems share (ib_plan_grad), and its flows
    // (ib_flow_create), as long as one of them lives
    std::weak_ptr<GradOps> grad;
    std::weak_ptr<FlowOps> flow;
};

// I of a plan on the host, as build_ib_plan leaves it
struct IbHost {
    std::vector<int32_t> iptr, icol;
    std::vector<double> ival;
};

struct IbKey {
    uint64_t h;
};

static uint64_t hash_bytes(uint64_t h, const void *p, size_t n) {
    const unsigned char *b = (const unsigned char *)p;
    for (size_t i = 0; i < n; ++i) {
        h ^= b[i];
        h *= 1099511628211ull;
    }
    return h;
}

struct IbCache {
    std::unordered_map<uint64_t, CacheEnt<IbPlan>> plans;
    std::unordered_map<uint64_t, std::vector<char>> keys;   // exact bytes of each plan's key
};

static IbCache &ib_cache(lgfib_ctx *ctx) {
    if (!ctx->ib_cache) ctx->ib_cache = std::make_shared<IbCache>();
    return *static_cast<IbCache *>(ctx->ib_cache.get());
}

// host (nullable) receives I if it is built here, and nothing if the plan is in
// the cache
static int build_ib_plan(lgfib_ctx *ctx, int kernel, const double *X, int NL, int B, const int32_t *blocks, int nblk,
                         std::shared_ptr<IbPlan> &out, IbHost *host = nullptr) {
    // cache by exact bytes of (kernel, B, X, blocks)
    std::vector<char> key;
    key.resize(sizeof(int) * 2 + sizeof(double) * 3 * (size_t)NL + sizeof(int32_t) * 3 * (size_t)nblk);
    char *kp = key.data();
    memcpy(kp, &kernel, sizeof(int));
    memcpy(kp + sizeof(int), &B, sizeof(int));
    if (NL) memcpy(kp + 2 * sizeof(int), X, sizeof(double) * 3 * (size_t)NL);
    if (nblk) memcpy(kp + 2 * sizeof(int) + sizeof(double) * 3 * (size_t)NL, blocks, sizeof(int32_t) * 3 * (size_t)nblk);
    uint64_t h = hash_bytes(1469598103934665603ull, key.data(), key.size());
    IbCache &cache = ib_cache(ctx);
    for (uint64_t salt = 0;; ++salt) {
        uint64_t hh = h ^ (salt * 0x9e3779b97f4a7c15ull);
        auto it = cache.keys.find(hh);
        if (it == cache.keys.end()) {
            h = hh;
            break;
        }
        if (it->second == key) {
            auto pl = cache.plans.find(hh);
            if (pl != cache.plans.end()) {
                pl->second.tick = ++ctx->cache_tick;
                out = pl->second.v;
                return LGFIB_OK;
            }
            cache.keys.erase(it);   // a key left by a failed build: build again
            h = hh;
            break;
        }
    }
    int rc = validate_blocks(blocks, nblk, "body blocks");
    if (rc) return rc;
    for (int i = 0; i < 3 * NL; ++i)
        if (!std::isfinite(X[i]) || fabs(X[i]) > 1e6) return fail(LGFIB_EINVAL, "marker position not finite or too large");
    auto plan = std::make_shared<IbPlan>();
    plan->kernel = kernel;
    plan->NL = NL;
    plan->B = B;
    plan->nblk = nblk;
    int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-(1 << 30), -(1 << 30), -(1 << 30)};
    for (int i = 0; i < nblk; ++i)
        for (int a = 0; a < 3; ++a) {
            lo[a] = std::min(lo[a], (int)blocks[3 * i + a]);
            hi[a] = std::max(hi[a], (int)blocks[3 * i + a]);
        }
    if (nblk == 0)
        for (int a = 0; a < 3; ++a) lo[a] = hi[a] = 0;
    size_t msize = 1;
    for (int a = 0; a < 3; ++a) {
        plan->lo[a] = lo[a];
        plan->nb[a] = hi[a] - lo[a] + 1;
        msize *= (size_t)plan->nb[a];
    }
    if (msize > (size_t)1 << 28) return fail(LGFIB_ERANGE, "body block set spans too large a box");
    std::vector<int32_t> map(msize, -1);
    for (int i = 0; i < nblk; ++i) {
        size_t idx = ((size_t)(blocks[3 * i + 2] - lo[2]) * plan->nb[1] + (blocks[3 * i + 1] - lo[1])) * plan->nb[0] +
                     (blocks[3 * i] - lo[0]);
        map[idx] = i;
    }
    auto slot_of = [&](long long bx, long long by, long long bz) -> int {
        bx -= lo[0];
        by -= lo[1];
        bz -= lo[2];
        if (bx < 0 || by < 0 || bz < 0 || bx >= plan->nb[0] || by >= plan->nb[1] || bz >= plan->nb[2]) return -1;
        return map[((size_t)bz * plan->nb[1] + by) * plan->nb[0] + bx];
    };
    // sparse I and R: the nonzero tensor-product weights of every (marker,
    // component); a support cell outside the block set is an error
    const int B3 = B * B * B;
    const int64_t nfaces = 3ll * nblk * B3;
    if (nfaces > INT32_MAX - 1 || 3ll * NL > INT32_MAX - 1) return fail(LGFIB_ERANGE, "IB operator too large");
    std::vector<int32_t> iptr(3 * (size_t)NL + 1, 0), icol;
    std::vector<double> ival;
    icol.reserve((size_t)NL * 3 * 27);
    ival.reserve((size_t)NL * 3 * 27);
    for (int i = 0; i < NL; ++i) {
        for (int k = 0; k < 3; ++k) {
            long long l[3];
            int cnt[3];
            double w[3][8];
            long long bq[3][8];   // block and place in it of the support's cells, by axis
            int at[3][8];
            for (int a = 0; a < 3; ++a) {
                const double c = (a == k) ? 0.0 : 0.5;
                support_range(kernel, X[3 * i + a], c, &l[a], &cnt[a]);
                for (int q = 0; q < cnt[a]; ++q) {
                    w[a][q] = phi_k(kernel, (double)(l[a] + q) + c - X[3 * i + a]);
                    bq[a][q] = floordiv(l[a] + q, B);
                    at[a][q] = (int)(l[a] + q - bq[a][q] * B);
                }
            }
            for (int dz = 0; dz < cnt[2]; ++dz) {
                if (w[2][dz] == 0.0) continue;
                for (int dy = 0; dy < cnt[1]; ++dy) {
                    if (w[1][dy] == 0.0) continue;
                    for (int dxx = 0; dxx < cnt[0]; ++dxx) {
                        if (w[0][dxx] == 0.0) continue;
                        const int slot = slot_of(bq[0][dxx], bq[1][dy], bq[2][dz]);
                        if (slot < 0)
                            return fail(LGFIB_ESUPPORT, "support of marker " + std::to_string(i) +
                                                            " leaves the block set");
                        const int loc = (at[2][dz] * B + at[1][dy]) * B + at[0][dxx];
                        icol.push_back((int32_t)(((long long)k * nblk + slot) * B3 + loc));
                        ival.push_back(w[2][dz] * w[1][dy] * w[0][dxx]);
                    }
                }
            }
            iptr[3 * i + k + 1] = (int32_t)icol.size();
        }
    }
    // R = transpose of I: counting sort by face; rows keep ascending (3 i + k)
    const size_t nnz = icol.size();
    std::vector<int32_t> rptr((size_t)nfaces + 1, 0), rcol(std::max<size_t>(nnz, 1));
    std::vector<double> rval(std::max<size_t>(nnz, 1));
    for (size_t e = 0; e < nnz; ++e) rptr[(size_t)icol[e] + 1]++;
    for (int64_t f = 0; f < nfaces; ++f) {
        if (rptr[f + 1] > 0) plan->face.push_back((int32_t)f);
        rptr[f + 1] += rptr[f];
    }
    plan->fend.reserve(plan->face.size());
    for (int32_t f : plan->face) plan->fend.push_back(rptr[f + 1]);
    {
        std::vector<int32_t> fill(rptr.begin(), rptr.end() - 1);
        for (int64_t row = 0; row < 3ll * NL; ++row)
            for (int32_t e = iptr[row]; e < iptr[row + 1]; ++e) {
                const int32_t pos = fill[icol[e]]++;
                rcol[pos] = (int32_t)row;
                rval[pos] = ival[e];
            }
    }
    if (nnz == 0) {
        icol.push_back(0);
        ival.push_back(0.0);
    }
    plan->nnz = (int64_t)nnz;
    if ((rc = plan->X.reserve(sizeof(double) * 3 * std::max(NL, 1)))) return rc;
    if ((rc = plan->map.reserve(sizeof(int32_t) * map.size()))) return rc;
    if ((rc = plan->blocks.reserve(sizeof(int32_t) * 3 * std::max(nblk, 1)))) return rc;
    if ((rc = plan->i_ptr.reserve(sizeof(int32_t) * iptr.size())) || (rc = plan->i_col.reserve(4 * icol.size())) ||
        (rc = plan->i_val.reserve(8 * ival.size())) || (rc = plan->r_ptr.reserve(sizeof(int32_t) * rptr.size())) ||
        (rc = plan->r_col.reserve(4 * rcol.size())) || (rc = plan->r_val.reserve(8 * rval.size())))
        return rc;
    if (NL) LGF_HIP(hipMemcpy(plan->X.p, X, sizeof(double) * 3 * NL, hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->map.p, map.data(), sizeof(int32_t) * map.size(), hipMemcpyHostToDevice));
    if (nblk) LGF_HIP(hipMemcpy(plan->blocks.p, blocks, sizeof(int32_t) * 3 * nblk, hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->i_ptr.p, iptr.data(), 4 * iptr.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->i_col.p, icol.data(), 4 * icol.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->i_val.p, ival.data(), 8 * ival.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->r_ptr.p, rptr.data(), 4 * rptr.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->r_col.p, rcol.data(), 4 * rcol.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(plan->r_val.p, rval.data(), 8 * rval.size(), hipMemcpyHostToDevice));
    if (host) *host = IbHost{std::move(iptr), std::move(icol), std::move(ival)};
    out = plan;
    cache.keys[h] = std::move(key);
    cache.plans[h] = CacheEnt<IbPlan>{std::move(plan), ++ctx->cache_tick};
    cache_trim_all(ctx, 1);
    return LGFIB_OK;
}

// a set of cell blocks on the host: block map over the box lo, nb
struct CellSet {
    const int *lo, *nb;
    const std::vector<int32_t> &map;
    int slot(int x, int y, int z) const {
        x -= lo[0], y -= lo[1], z -= lo[2];
        if (x < 0 || y < 0 || z < 0 || x >= nb[0] || y >= nb[1] || z >= nb[2]) return -1;
        return map[((size_t)z * nb[1] + y) * nb[0] + x];
    }
};

static int log2_edge(int B) { return B == 4 ? 2 : B == 8 ? 3 : 4; }   // force systems have B in {4, 8, 16}

// The spread operator of plan p with its cells numbered on the set cs (which
// holds p's blocks, in order in `blocks`).  c = G^T u has face (n, k) add to c(n)
// and subtract from c(n - e_k), so G^T R has two entries for each one of R, one
// where the cell below lies outside cs.  low (nullable) receives that cell per
// entry of I.  h: the plan's I, read back from the device if empty.
static int build_spread(const IbPlan &p, const int32_t *blocks, const CellSet &cs, int64_t ncell, IbHost &h,
                        SpreadOp &op, std::vector<int32_t> *low_out) {
    const int lb = log2_edge(p.B), B = p.B, B3 = B * B * B;
    const int64_t nc = (int64_t)p.nblk * B3, nrows = 3ll * p.NL;
    const size_t nnz = (size_t)p.nnz;
    if (ncell > INT32_MAX - 1) return fail(LGFIB_ERANGE, "IB operator too large");
    if (h.iptr.empty()) {
        h.iptr.resize(nrows + 1);
        h.icol.resize(std::max<size_t>(nnz, 1));
        h.ival.resize(h.icol.size());
        LGF_HIP(hipMemcpy(h.iptr.data(), p.i_ptr.p, 4 * h.iptr.size(), hipMemcpyDeviceToHost));
        LGF_HIP(hipMemcpy(h.icol.data(), p.i_col.p, 4 * h.icol.size(), hipMemcpyDeviceToHost));
        LGF_HIP(hipMemcpy(h.ival.data(), p.i_val.p, 8 * h.ival.size(), hipMemcpyDeviceToHost));
    }
    // slots on cs of each block and its lower neighbours
    std::vector<std::array<int32_t, 4>> slot((size_t)p.nblk);
    for (int i = 0; i < p.nblk; ++i) {
        const int32_t *q = blocks + 3 * (size_t)i;
        slot[i] = {cs.slot(q[0], q[1], q[2]), cs.slot(q[0] - 1, q[1], q[2]), cs.slot(q[0], q[1] - 1, q[2]),
                   cs.slot(q[0], q[1], q[2] - 1)};
    }
    std::vector<int32_t> own(std::max<size_t>(nnz, 1)), low(std::max<size_t>(nnz, 1), -1);
    std::vector<int64_t> dptr(ncell + 1, 0);
    for (int64_t row = 0; row < nrows; ++row) {
        const int k = (int)(row % 3), sh = k * lb, m = B - 1;
        for (int32_t e = h.iptr[row]; e < h.iptr[row + 1]; ++e) {
            const int32_t cell = (int32_t)(h.icol[e] - k * nc), loc = cell & (B3 - 1);
            const auto &sl = slot[cell >> (3 * lb)];
            own[e] = sl[0] * B3 + loc;
            if (loc >> sh & m) low[e] = own[e] - (1 << sh);
            else if (sl[1 + k] >= 0) low[e] = sl[1 + k] * B3 + loc + (m << sh);
            dptr[own[e] + 1]++;
            if (low[e] >= 0) dptr[low[e] + 1]++;
        }
    }
    std::vector<int32_t> srow(p.face);
    std::vector<int64_t> sptr;
    sptr.reserve(2 * srow.size() + 1);
    sptr.push_back(0);
    sptr.insert(sptr.end(), p.fend.begin(), p.fend.end());
    op.nfr = (int)srow.size();
    for (int64_t c = 0; c < ncell; ++c) {
        const bool any = dptr[c + 1] > 0;
        dptr[c + 1] += dptr[c];
        if (any) {
            srow.push_back((int32_t)c);
            sptr.push_back((int64_t)nnz + dptr[c + 1]);
        }
    }
    op.nrows = (int)srow.size();
    std::vector<int32_t> col(std::max<size_t>(dptr[ncell], 1));   // the cells' rows; the faces' are R's
    std::vector<double> val(col.size());
    auto put = [&](int32_t cell, int64_t row, double w) {   // dptr[cell]: the next place of the cell
        const size_t q = dptr[cell]++;
        col[q] = (int32_t)row;
        val[q] = w;
    };
    for (int64_t row = 0; row < nrows; ++row)
        for (int32_t e = h.iptr[row]; e < h.iptr[row + 1]; ++e) {
            put(own[e], row, h.ival[e]);
            if (low[e] >= 0) put(low[e], row, -h.ival[e]);
        }
    srow.resize(std::max<size_t>(srow.size(), 1));
    int rc;
    if ((rc = op.row.reserve(4 * srow.size())) || (rc = op.ptr.reserve(8 * sptr.size())) ||
        (rc = op.col.reserve(4 * (nnz + col.size()))) || (rc = op.val.reserve(8 * (nnz + val.size()))))
        return rc;
    LGF_HIP(hipMemcpy(op.row.p, srow.data(), 4 * srow.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(op.ptr.p, sptr.data(), 8 * sptr.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(op.col.p, p.r_col.p, 4 * nnz, hipMemcpyDeviceToDevice));
    LGF_HIP(hipMemcpy(op.val.p, p.r_val.p, 8 * nnz, hipMemcpyDeviceToDevice));
    LGF_HIP(hipMemcpy(op.col.as<int>() + nnz, col.data(), 4 * col.size(), hipMemcpyHostToDevice));
    LGF_HIP(hipMemcpy(op.val.as<double>() + nnz, val.data(), 8 * val.size(), hipMemcpyHostToDevice));
    if (low_out) *low_out = std::move(low);
    return LGFIB_OK;
}

// The operators of the force Schur complement with the staggered gradient
// folded in: the spread operator on the plan's own blocks, and for (G d)^(k)(n)
// = d(n) - d(n - e_k) the cell below each entry of I.
static int ib_plan_grad(IbPlan &p, const int32_t *blocks, IbHost &h, std::shared_ptr<GradOps> &out) {
    if ((out = p.grad.lock())) return LGFIB_OK;
    std::vector<int32_t> map((size_t)p.nb[0] * p.nb[1] * p.nb[2], -1), low;
    for (int i = 0; i < p.nblk; ++i)
        map[((size_t)(blocks[3 * i + 2] - p.lo[2]) * p.nb[1] + (blocks[3 * i + 1] - p.lo[1])) * p.nb[0] +
            (blocks[3 * i] - p.lo[0])] = i;
    auto g = std::make_shared<GradOps>();
    int rc;
    if ((rc = build_spread(p, blocks, CellSet{p.lo, p.nb, map}, (int64_t)p.nblk * p.B * p.B * p.B, h, g->spread, &low)) ||
        (rc = g->i_low.reserve(4 * low.size())))
        return rc;
    LGF_HIP(hipMemcpy(g->i_low.p, low.data(), 4 * low.size(), hipMemcpyHostToDevice));
    p.grad = out = std::move(g);
    return LGFIB_OK;
}

size_t ib_cache_trim(lgfib_ctx *ctx, size_t cap, int64_t *left) {
    if (!ctx->ib_cache) {
        if (left) *left = 0;
        return 0;
    }
    IbCache &cache = ib_cache(ctx);
    const size_t n = cache_trim(cache.plans, cap, kNoByteCap, [&](uint64_t h, const IbPlan &) { cache.keys.erase(h); });
    if (left) *left = (int64_t)cache.plans.size();
    return n;
}

// --------------------------------------------------------------- kernels

struct BlockMapDev {
    int lo0, lo1, lo2, nb0, nb1, nb2, B;
    const int *map;
    const int *blocks;
    __device__ int slot(int bx, int by, int bz) const {
        bx -= lo0;
        by -= lo1;
        bz -= lo2;
        if (bx < 0 || by < 0 || bz < 0 || bx >= nb0 || by >= nb1 || bz >= nb2) return -1;
        return map[((size_t)bz * nb1 + by) * nb0 + bx];
    }
};


// Block sums of a grid-wide reduction go to part[block]; the last block to
// finish (a device-scope counter) adds them in block order, so the result
// does not depend on which block finishes last.  One launch per reduction.
__device__ inline void grid_sum_to(double s, double *part, unsigned *counter, double *out) {
    __shared__ double sh[256];
    __shared__ bool last;
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x] = sh[0];
        __threadfence();
        last = atomicAdd(counter, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    double v = 0.0;
    for (unsigned i = threadIdx.x; i < gridDim.x; i += 256) v += part[i];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *out = sh[0];
        *counter = 0u;
    }
}

// y[row] = scale * sum_e val[e] x[col[e]] over the row's entries in FP64, less
// sub[row] where given.
// R: rows are faces, columns 3 i + k, scale dx^-3
// (g^(k)(n) = dx^-3 sum_i x_i^(k) prod_j phi(x_F^(k)(n)_j - X_ij)).
// I: rows 3 i + k, columns face indices, scale 1.
// L lanes share a row (entries strided by L, then a butterfly sum), which
// keeps the dependent col -> x loads of a row short; the summation order is
// fixed, so results are reproducible.
template <typename In, typename Out, int L>
__global__ __launch_bounds__(256) void k_csr_gather(const int *__restrict__ ptr, const int *__restrict__ col,
                                                    const double *__restrict__ val, const In *__restrict__ x,
                                                    const Out *__restrict__ sub, Out *__restrict__ y, int nrows,
                                                    double scale) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int row = (int)(t / L), lane = (int)(t % L);
    const bool live = row < nrows;
    double acc = 0.0;
    if (live) {
        const int e1 = ptr[row + 1];
        for (int e = ptr[row] + lane; e < e1; e += L) acc += val[e] * (double)x[col[e]];
    }
#pragma unroll
    for (int m = L / 2; m > 0; m >>= 1) acc += __shfl_xor(acc, m, L);
    if (live && lane == 0) y[row] = sub ? (Out)(acc * scale) - sub[row] : (Out)(acc * scale);
}

// Sum of n partial sums, the same value in every lane of every wavefront: each
// lane's share first, so that its loads can be issued ahead of other work
__device__ __forceinline__ double part_lane(const double *__restrict__ part, int n) {
    const int i0 = threadIdx.x % 64;
    double v = part[min(i0, n - 1)];
    v = i0 < n ? v : 0.0;
    for (int i = i0 + 64; i < n; i += 64) v += part[i];
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// The CG's search direction of the iteration about to start, p = r + beta
// p_old with beta = rs / rs_old (zero at the start of a sweep, when p_old is
// not used); rs and rs_old come as nred partial sums each.
struct CgDir {
    const double *r, *p_old, *rs, *rs_old;
    double *p;
    int nred, n;
};

// faces = R x and c = G^T R x in one launch, eight lanes a row, on the rows
// that some marker reaches (the others hold zeros from the start).  Short
// gathers bound by latency: at 2200 markers R took 4.2 us and G^T of its faces
// another 3.8; with the cells' rows folded on the host both run side by side in
// 5.5 us, 7.4 with DIR.  Over all faces and cells instead of the reached rows (of
// 290,000) it took 10.5 us.  DIR: x is the CG's new search direction, formed
// as R r + beta R p_old so that beta's sums are off the gathers' path, and
// stored for the update.
template <bool DIR, typename In, typename Out>
__global__ __launch_bounds__(256) void k_spread(const long *__restrict__ ptr, const int *__restrict__ col,
                                                const double *__restrict__ val, const int *__restrict__ out,
                                                const In *__restrict__ x, CgDir dir, Out *__restrict__ faces,
                                                Out *__restrict__ c, int nrows, int nfr) {
    constexpr int L = 8;
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    const int row = (int)(t / L), lane = threadIdx.x % L;
    const bool live = row < nrows;
    double acc = 0.0, old = 0.0, rs = 0.0, ro = 0.0, r0 = 0.0, p0 = 0.0;
    if constexpr (DIR) {   // these loads run ahead of the gathers
        rs = part_lane(dir.rs, dir.nred);
        ro = part_lane(dir.rs_old, dir.nred);
        r0 = dir.r[min(t, (long)dir.n - 1)];
        p0 = dir.p_old[min(t, (long)dir.n - 1)];
    }
    if (live) {
        const long e1 = ptr[row + 1];
        for (long e = ptr[row] + lane; e < e1; e += L) {
            const int j = col[e];
            const double w = val[e];
            if constexpr (DIR) {
                acc += w * dir.r[j];
                old += w * dir.p_old[j];
            } else {
                acc += w * (double)x[j];
            }
        }
    }
    if constexpr (DIR) {
        rs = wave_sum(rs);
        ro = wave_sum(ro);
        const double beta = ro > 0.0 ? rs / ro : 0.0;
        if (t < dir.n) dir.p[t] = beta == 0.0 ? r0 : r0 + beta * p0;
        for (long i = t + gridDim.x * 256l; i < dir.n; i += gridDim.x * 256l)
            dir.p[i] = beta == 0.0 ? dir.r[i] : dir.r[i] + beta * dir.p_old[i];
        if (beta != 0.0) acc += beta * old;
    }
#pragma unroll
    for (int m = L / 2; m > 0; m >>= 1) acc += __shfl_xor(acc, m, L);
    if (live && lane == 0) {
        const int o = out[row];
        if (row < nfr) faces[o] = (Out)acc;
        else c[o] = (Out)acc;
    }
}

// y = I (a + G d), sixteen lanes a row: the gradient is formed where I reads
// it, so that a + G d is never stored (a launch of 3.2 us at 2200 markers).
// dot_p: part[block] receives the block's share of dot_p . y, in row order.
template <typename In, typename Out>
__global__ __launch_bounds__(256) void k_gather(const int *__restrict__ ptr, const int *__restrict__ col,
                                                const int *__restrict__ low, const double *__restrict__ val,
                                                const In *__restrict__ a, const In *__restrict__ d,
                                                Out *__restrict__ y, int nrows, int nc,
                                                const double *__restrict__ dot_p, double *__restrict__ part) {
    __shared__ double sh[16];
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    const int row = (int)(t / 16), lane = (int)(t % 16);
    const bool live = row < nrows;
    double acc = 0.0;
    if (live) {
        const int e1 = ptr[row + 1], shift = (row % 3) * nc;
        for (int e = ptr[row] + lane; e < e1; e += 16) {
            const int f = col[e], m = low[e];
            const In dm = d[max(m, 0)];
            acc += val[e] * (double)(a[f] + (d[f - shift] - (m >= 0 ? dm : (In)0)));
        }
    }
#pragma unroll
    for (int m = 8; m > 0; m >>= 1) acc += __shfl_xor(acc, m, 16);
    if (live && lane == 0) y[row] = (Out)acc;
    if (!dot_p) return;
    if (lane == 0) sh[threadIdx.x / 16] = live ? acc * dot_p[row] : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) v += sh[q];
        part[blockIdx.x] = v;
    }
}

static BlockMapDev devmap(const IbPlan &p) {
    BlockMapDev m;
    m.lo0 = p.lo[0];
    m.lo1 = p.lo[1];
    m.lo2 = p.lo[2];
    m.nb0 = p.nb[0];
    m.nb1 = p.nb[1];
    m.nb2 = p.nb[2];
    m.B = p.B;
    m.map = p.map.as<int>();
    m.blocks = p.blocks.as<int>();
    return m;
}

static unsigned nblocks(size_t n, int t) { return (unsigned)((n + t - 1) / t); }

template <typename In, typename Out>
static int launch_regularize(lgfib_ctx *ctx, const IbPlan &p, double dx, const In *x, Out *faces, hipStream_t st) {
    if (p.nblk == 0) return LGFIB_OK;
    ProfScope ps(ctx, "k_regularize", st);
    const int nrows = 3 * p.nblk * p.B * p.B * p.B;
    hipLaunchKernelGGL((k_csr_gather<In, Out, 4>), dim3(nblocks(4 * (size_t)nrows, 256)), dim3(256), 0, st,
                       p.r_ptr.as<int>(),
                       p.r_col.as<int>(), p.r_val.as<double>(), x, (const Out *)nullptr, faces, nrows,
                       1.0 / (dx * dx * dx));
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

template <typename In, typename Out>
static int launch_interpolate(lgfib_ctx *ctx, const IbPlan &p, const In *faces, Out *v, hipStream_t st,
                              const Out *sub = nullptr) {
    if (p.NL == 0) return LGFIB_OK;
    ProfScope ps(ctx, "k_interpolate", st);
    const int nrows = 3 * p.NL;
    hipLaunchKernelGGL((k_csr_gather<In, Out, 16>), dim3(nblocks(16 * (size_t)nrows, 256)), dim3(256), 0, st,
                       p.i_ptr.as<int>(),
                       p.i_col.as<int>(), p.i_val.as<double>(), faces, sub, v, nrows, 1.0);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

// faces = R x, c = G^T R x (faces and c hold zeros where no marker reaches);
// dir: the CG's direction
template <typename In, typename Out>
static int launch_spread(lgfib_ctx *ctx, const SpreadOp &op, const In *x, const CgDir *dir, Out *faces, Out *c,
                         hipStream_t st) {
    ProfScope ps(ctx, "k_spread", st);
    const dim3 grid(std::max(1u, nblocks(8 * (size_t)op.nrows, 256)));
    if (dir)
        hipLaunchKernelGGL((k_spread<true, In, Out>), grid, dim3(256), 0, st, op.ptr.as<long>(), op.col.as<int>(),
                           op.val.as<double>(), op.row.as<int>(), x, *dir, faces, c, op.nrows, op.nfr);
    else
        hipLaunchKernelGGL((k_spread<false, In, Out>), grid, dim3(256), 0, st, op.ptr.as<long>(), op.col.as<int>(),
                           op.val.as<double>(), op.row.as<int>(), x, CgDir{}, faces, c, op.nrows, op.nfr);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

static unsigned gather_blocks(int NL) { return nblocks(16 * 3 * (size_t)NL, 256); }

// y = I (a + G d); with dot_p the blocks' shares of dot_p . y go to part
template <typename In, typename Out>
static int launch_gather(lgfib_ctx *ctx, const IbPlan &p, const GradOps &g, const In *a, const In *d, Out *y,
                         const double *dot_p, double *part, hipStream_t st) {
    ProfScope ps(ctx, "k_gather", st);
    hipLaunchKernelGGL((k_gather<In, Out>), dim3(gather_blocks(p.NL)), dim3(256), 0, st, p.i_ptr.as<int>(),
                       p.i_col.as<int>(), g.i_low.as<int>(), p.i_val.as<double>(), a, d, y, 3 * p.NL,
                       p.nblk * p.B * p.B * p.B, dot_p, part);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

static int body_blocks(int kernel, const double *X, int NL, int B, std::vector<int32_t> &out) {
    struct H {
        size_t operator()(const std::array<long long, 3> &a) const {
            return std::hash<long long>()(a[0] * 73856093ll ^ a[1] * 19349663ll ^ a[2] * 83492791ll);
        }
    };
    std::unordered_map<std::array<long long, 3>, char, H> set;
    for (int i = 0; i < NL; ++i) {
        for (int k = 0; k < 3; ++k) {
            long long l[3];
            int cnt[3];
            for (int a = 0; a < 3; ++a) support_range(kernel, X[3 * i + a], (a == k) ? 0.0 : 0.5, &l[a], &cnt[a]);
            for (int dz = 0; dz < cnt[2]; ++dz)
                for (int dy = 0; dy < cnt[1]; ++dy)
                    for (int dxx = 0; dxx < cnt[0]; ++dxx) {
                        const long long n[3] = {l[0] + dxx, l[1] + dy, l[2] + dz};
                        double w = 1.0;
                        for (int a = 0; a < 3; ++a)
                            w *= phi_k(kernel, (double)n[a] + ((a == k) ? 0.0 : 0.5) - X[3 * i + a]);
                        if (w == 0.0) continue;
                        // the support cell and its 26 neighbours
                        for (int ez = -1; ez <= 1; ++ez)
                            for (int ey = -1; ey <= 1; ++ey)
                                for (int ex = -1; ex <= 1; ++ex)
                                    set[{floordiv(n[0] + ex, B), floordiv(n[1] + ey, B), floordiv(n[2] + ez, B)}] = 1;
                    }
        }
    }
    std::vector<std::array<long long, 3>> v;
    v.reserve(set.size());
    for (auto &kv : set) v.push_back(kv.first);
    std::sort(v.begin(), v.end(), [](const std::array<long long, 3> &a, const std::array<long long, 3> &b) {
        if (a[2] != b[2]) return a[2] < b[2];
        if (a[1] != b[1]) return a[1] < b[1];
        return a[0] < b[0];
    });
    out.clear();
    for (auto &b : v) {
        for (int a = 0; a < 3; ++a) {
            if (b[a] < -(1 << 20) || b[a] >= (1 << 20)) return fail(LGFIB_ERANGE, "body block coordinate out of range");
            out.push_back((int32_t)b[a]);
        }
    }
    return LGFIB_OK;
}

}  // namespace lgfib

using namespace lgfib;

static int ib_check(lgfib_ctx *ctx, int kernel, const double *X, int NL, int B, const int32_t *blocks, int nblk,
                    int prec, double dx, const char *who) {
    if (!ctx) return fail(LGFIB_EINVAL, std::string(who) + ": null context");
    if (kernel != IB_ROMA3 && kernel != IB_SMOOTH3) return fail(LGFIB_EINVAL, std::string(who) + ": unknown kernel");
    if (B != 4 && B != 8 && B != 16 && B != 32) return fail(LGFIB_EINVAL, std::string(who) + ": B must be 4, 8, 16 or 32");
    if (NL < 0 || nblk < 0) return fail(LGFIB_EINVAL, std::string(who) + ": negative count");
    if (NL > 0 && !X) return fail(LGFIB_EINVAL, std::string(who) + ": null marker positions");
    if (prec != LGF_F32 && prec != LGF_F64) return fail(LGFIB_EINVAL, std::string(who) + ": bad prec");
    if (!(dx > 0.0) || !std::isfinite(dx)) return fail(LGFIB_EINVAL, std::string(who) + ": dx must be positive");
    return LGFIB_OK;
}

extern "C" int ib_body_blocks(int kernel, const double *X, int NL, int B, int32_t *out, int max, int *n) {
    if (kernel != IB_ROMA3 && kernel != IB_SMOOTH3) return fail(LGFIB_EINVAL, "ib_body_blocks: unknown kernel");
    if (B < 1 || NL < 0 || (NL > 0 && !X) || !n) return fail(LGFIB_EINVAL, "ib_body_blocks: bad argument");
    for (int i = 0; i < 3 * NL; ++i)
        if (!std::isfinite(X[i]) || fabs(X[i]) > 1e6) return fail(LGFIB_EINVAL, "ib_body_blocks: bad marker position");
    std::vector<int32_t> v;
    int rc = body_blocks(kernel, X, NL, B, v);
    if (rc) return rc;
    *n = (int)(v.size() / 3);
    if (*n > max || (*n > 0 && !out)) return fail(LGFIB_ERANGE, "ib_body_blocks: output holds fewer blocks than needed");
    std::copy(v.begin(), v.end(), out);
    return LGFIB_OK;
}

extern "C" int ib_regularize(lgfib_ctx *ctx, int kernel, const double *X, int NL, int B, const int32_t *blocks,
                             int nblk, int prec, double dx, const void *x, void *faces, lgfib_stream_t stream) {
    int rc = ib_check(ctx, kernel, X, NL, B, blocks, nblk, prec, dx, "ib_regularize");
    if (rc) return rc;
    if ((NL > 0 && !x) || (nblk > 0 && !faces)) return fail(LGFIB_EINVAL, "ib_regularize: null field pointer");
    LGF_HIP(hipSetDevice(ctx->device));
    std::shared_ptr<IbPlan> p;
    if ((rc = build_ib_plan(ctx, kernel, X, NL, B, blocks, nblk, p))) return rc;
    if (prec == LGF_F64)
        return launch_regularize<double, double>(ctx, *p, dx, (const double *)x, (double *)faces, (hipStream_t)stream);
    return launch_regularize<float, float>(ctx, *p, dx, (const float *)x, (float *)faces, (hipStream_t)stream);
}

extern "C" int ib_interpolate(lgfib_ctx *ctx, int kernel, const double *X, int NL, int B, const int32_t *blocks,
                              int nblk, int prec, double dx, const void *faces, void *v, lgfib_stream_t stream) {
    int rc = ib_check(ctx, kernel, X, NL, B, blocks, nblk, prec, dx, "ib_interpolate");
    if (rc) return rc;
    if ((NL > 0 && !v) || (nblk > 0 && !faces)) return fail(LGFIB_EINVAL, "ib_interpolate: null field pointer");
    LGF_HIP(hipSetDevice(ctx->device));
    std::shared_ptr<IbPlan> p;
    if ((rc = build_ib_plan(ctx, kernel, X, NL, B, blocks, nblk, p))) return rc;
    if (prec == LGF_F64)
        return launch_interpolate<double, double>(ctx, *p, (const double *)faces, (double *)v, (hipStream_t)stream);
    return launch_interpolate<float, float>(ctx, *p, (const float *)faces, (float *)v, (hipStream_t)stream);
}

// ---------------------------------------------------------- Schur system

namespace lgfib {
constexpr int kRedBlocks = 256;   // blocks of a grid-wide reduction
// partial-sum slots: r.r of even and odd CG iterations, then one per block of
// k_gather (or of k_dot)
inline size_t red_parts(int NL) { return 2 * kRedBlocks + std::max<size_t>(kRedBlocks, (16 * 3 * (size_t)NL + 255) / 256); }
}

struct ib_system {
    lgfib_ctx *ctx = nullptr;
    int kernel = 0, NL = 0, B = 0, nblk = 0;
    double a = 0.0;
    std::vector<double> X;
    std::vector<int32_t> blocks;
    lgf_table_t tbl = -1;
    std::shared_ptr<IbPlan> plan;   // held: pinned in the context's cache
    std::shared_ptr<GradOps> grad;
    // work fields per precision: faces g, faces a, cells c, cells d; g and c are
    // written by k_spread alone
    DevBuf g[2], af[2], c[2], d[2];
    // CG vectors (FP64)
    DevBuf r, p, p2, ap, x, tmp, red, scal, cnt;   // p, p2: the search direction of even / odd iterations
    double *host_scal = nullptr;       // pinned; [64 ..]: the CG's r.r as 2 x kRedBlocks partial sums
    double *host_scal_dev = nullptr;   // its device address
    hipEvent_t ev[2] = {nullptr, nullptr};
    // captured CG iterations per matvec precision (index 0 FP32, 1 FP64) and
    // parity of the iteration; valid while the shared FFT workspaces stay put
    hipGraphExec_t cg_exec[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};
    const void *cg_work[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};
    uint64_t cg_epoch[2] = {0, 0};   // the context's cache epoch when captured
    bool cg_nograph[2] = {false, false};   // capture failed once: run eagerly
    hipStream_t cap = nullptr;
    // inverse Cholesky factor W = L^{-1} of the dense C (ib_system_factor)
    DevBuf wfac;
    bool factored = false;
    DevBuf gamma;   // R 1 on the body faces (force smoothing), built on first use
    DevBuf dense_cols;   // workspace of the column-batched dense build of C
};

namespace lgfib {

// y = C x = I [E(a) + G K^{-1} G^T] R x with the field work in Real; x and y
// may be held in another type (the FP32 matvec of the CG reads and writes its
// FP64 vectors directly).
// dir: x is the CG's new direction, and its dot product with y goes to part.
template <typename Real, typename VIn, typename VOut>
static int schur_apply_t(ib_system *s, const VIn *x, VOut *y, hipStream_t st, const CgDir *dir = nullptr) {
    lgfib_ctx *ctx = s->ctx;
    const int pi = sizeof(Real) == 8 ? 1 : 0;
    const int prec = pi ? LGF_F64 : LGF_F32;
    Real *g = s->g[pi].as<Real>(), *af = s->af[pi].as<Real>(), *c = s->c[pi].as<Real>(), *d = s->d[pi].as<Real>();
    int rc;
    if ((rc = launch_spread<VIn, Real>(ctx, s->grad->spread, x, dir, g, c, st))) return rc;
    if ((rc = lgf_if_apply(ctx, s->a, s->B, s->blocks.data(), s->nblk, s->blocks.data(), s->nblk, 3, prec, g, af,
                           (lgfib_stream_t)st)))
        return rc;
    if ((rc = lgf_poisson_apply(ctx, s->tbl, s->B, s->blocks.data(), s->nblk, s->blocks.data(), s->nblk, 1, prec, 1.0,
                                c, d, 0, (lgfib_stream_t)st)))
        return rc;
    return launch_gather<Real, VOut>(ctx, *s->plan, *s->grad, af, d, y, dir ? dir->p : nullptr,
                                     s->red.as<double>() + 2 * kRedBlocks, st);
}

}  // namespace lgfib

extern "C" int ib_system_create(lgfib_ctx *ctx, int kernel, const double *X, int NL, int B, const int32_t *blocks,
                                int nblk, double a, ib_system **out) {
    if (!out) return fail(LGFIB_EINVAL, "ib_system_create: null output");
    *out = nullptr;
    int rc = ib_check(ctx, kernel, X, NL, B, blocks, nblk, LGF_F64, 1.0, "ib_system_create");
    if (rc) return rc;
    if (B > 16) return fail(LGFIB_EINVAL, "ib_system_create: B must be 4, 8 or 16");
    if (NL < 1 || nblk < 1) return fail(LGFIB_EINVAL, "ib_system_create: need markers and blocks");
    if (!(a >= 0.0) || a > 4.0) return fail(LGFIB_EINVAL, "ib_system_create: a must lie in [0, 4]");
    LGF_HIP(hipSetDevice(ctx->device));
    auto s = std::make_unique<ib_system>();
    s->ctx = ctx;
    s->kernel = kernel;
    s->NL = NL;
    s->B = B;
    s->nblk = nblk;
    s->a = a;
    s->X.assign(X, X + 3 * (size_t)NL);
    s->blocks.assign(blocks, blocks + 3 * (size_t)nblk);
    IbHost host;
    if ((rc = build_ib_plan(ctx, kernel, X, NL, B, blocks, nblk, s->plan, &host))) return rc;
    if ((rc = ib_plan_grad(*s->plan, blocks, host, s->grad))) return rc;
    int ext[3];
    for (int q = 0; q < 3; ++q) ext[q] = s->plan->nb[q] * B - 1;
    if ((rc = lgf_table_build(ctx, LGF_KIND_K, a, ext, nullptr, &s->tbl))) return rc;
    const size_t B3 = (size_t)B * B * B;
    for (int pi = 0; pi < 2; ++pi) {
        const size_t es = pi ? 8 : 4;
        if ((rc = s->g[pi].reserve(3 * nblk * B3 * es))) return rc;
        if ((rc = s->af[pi].reserve(3 * nblk * B3 * es))) return rc;
        if ((rc = s->c[pi].reserve(nblk * B3 * es))) return rc;
        if ((rc = s->d[pi].reserve(nblk * B3 * es))) return rc;
    }
    const size_t nv = 3 * (size_t)NL * 8;
    if ((rc = s->r.reserve(nv)) || (rc = s->p.reserve(nv)) || (rc = s->p2.reserve(nv)) || (rc = s->ap.reserve(nv)) || (rc = s->x.reserve(nv)) ||
        (rc = s->tmp.reserve(nv)) || (rc = s->red.reserve(red_parts(NL) * 8)) || (rc = s->scal.reserve(64 * 8)) ||
        (rc = s->cnt.reserve(64)))
        return rc;
    LGF_HIP(hipMemset(s->cnt.p, 0, 64));
    for (int pi = 0; pi < 2; ++pi) {   // k_spread writes only the rows that markers reach
        LGF_HIP(hipMemset(s->g[pi].p, 0, s->g[pi].bytes));
        LGF_HIP(hipMemset(s->c[pi].p, 0, s->c[pi].bytes));
    }
    LGF_HIP(hipStreamSynchronize(nullptr));
    LGF_HIP(hipHostMalloc((void **)&s->host_scal, (64 + 2 * kRedBlocks) * sizeof(double), hipHostMallocDefault));
    LGF_HIP(hipHostGetDevicePointer((void **)&s->host_scal_dev, s->host_scal, 0));
    for (auto &e : s->ev) LGF_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    *out = s.release();
    return LGFIB_OK;
}

extern "C" void ib_system_destroy(ib_system *sys) {
    if (!sys) return;
    (void)hipSetDevice(sys->ctx->device);
    (void)hipDeviceSynchronize();
    if (sys->host_scal) (void)hipHostFree(sys->host_scal);
    for (auto &e : sys->ev)
        if (e) (void)hipEventDestroy(e);
    for (auto &row : sys->cg_exec)
        for (auto &g : row)
            if (g) (void)hipGraphExecDestroy(g);
    if (sys->cap) (void)hipStreamDestroy(sys->cap);
    delete sys;
}

extern "C" int ib_schur_apply(lgfib_ctx *ctx, ib_system *sys, int prec, const void *x, void *y,
                              lgfib_stream_t stream) {
    if (!ctx || !sys || sys->ctx != ctx) return fail(LGFIB_EINVAL, "ib_schur_apply: bad context or system");
    if (prec != LGF_F32 && prec != LGF_F64) return fail(LGFIB_EINVAL, "ib_schur_apply: bad prec");
    if (!x || !y) return fail(LGFIB_EINVAL, "ib_schur_apply: null vector");
    const size_t nb = 3 * (size_t)sys->NL * (prec == LGF_F64 ? 8 : 4);
    if ((const char *)x < (const char *)y + nb && (const char *)y < (const char *)x + nb)
        return fail(LGFIB_EINVAL, "ib_schur_apply: x and y overlap");
    LGF_HIP(hipSetDevice(ctx->device));
    if (prec == LGF_F64)
        return schur_apply_t<double, double, double>(sys, (const double *)x, (double *)y, (hipStream_t)stream);
    return schur_apply_t<float, float, float>(sys, (const float *)x, (float *)y, (hipStream_t)stream);
}

// ------------------------------------------------------ conjugate gradients

namespace lgfib {

__global__ __launch_bounds__(256) void k_dot(const double *__restrict__ a, const double *__restrict__ b, size_t n,
                                             double *part, unsigned *counter, double *out) {
    double s = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) s += a[i] * b[i];
    grid_sum_to(s, part, counter, out);
}

// x += alpha p ; r -= alpha Ap, alpha = rs / pAp (0 once the search direction
// vanishes: the host tests convergence one iteration late, so a converged
// solve may run one more, harmless, iteration); then each workgroup's share of
// r.r to part and to pinned host memory.  pAp and rs arrive as partial sums
// that every wavefront adds itself, in the same order: no atomics and no
// fences.  At 6600 unknowns a whole update in one workgroup (both reductions
// and the direction) took 9.2 us, this kernel with a last-workgroup sum 6.4,
// and as it is 4.5.
__global__ __launch_bounds__(256) void k_cg_xr(double *__restrict__ x, double *__restrict__ r,
                                               const double *__restrict__ p, const double *__restrict__ ap,
                                               const double *__restrict__ pap_part, int npart,
                                               const double *__restrict__ rs_part, int nred, size_t n,
                                               double *__restrict__ part, double *__restrict__ host_part) {
    __shared__ double sh[4];
    const size_t i0 = (size_t)blockIdx.x * 256 + threadIdx.x;
    const bool in = i0 < n;   // the first elements' loads are in flight beside the partial sums'
    const double x0 = in ? x[i0] : 0.0, p0 = in ? p[i0] : 0.0, r0 = in ? r[i0] : 0.0, a0 = in ? ap[i0] : 0.0;
    double pap = part_lane(pap_part, npart), rs = part_lane(rs_part, nred);
    pap = wave_sum(pap);
    rs = wave_sum(rs);
    const double alpha = pap > 0.0 ? rs / pap : 0.0;
    double s = 0.0;
    if (in) {
        x[i0] = x0 + alpha * p0;
        const double ri = r0 - alpha * a0;
        r[i0] = ri;
        s = ri * ri;
    }
    for (size_t i = i0 + (size_t)gridDim.x * 256; i < n; i += (size_t)gridDim.x * 256) {
        x[i] += alpha * p[i];
        const double ri = r[i] - alpha * ap[i];
        r[i] = ri;
        s += ri * ri;
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
    if (threadIdx.x % 64 == 0) sh[threadIdx.x / 64] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double v = (sh[0] + sh[1]) + (sh[2] + sh[3]);
        part[blockIdx.x] = v;
        host_part[blockIdx.x] = v;
    }
}

// dot products of vectors small enough for one workgroup (the marker systems)
constexpr int kStepThreads = 1024;
constexpr size_t kStepMaxN = 65536;

// workgroup sum: butterfly within each wavefront, then across the wavefronts'
// partials (fixed order, so the result is reproducible)
__device__ inline double wg_sum(double v, double *sh) {
    constexpr int kWaves = kStepThreads / 64;
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    if (lane == 0) sh[wave] = v;
    __syncthreads();
    double t = lane < kWaves ? sh[lane] : 0.0;
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) t += __shfl_xor(t, m, 64);
    __syncthreads();   // sh is reused by the next call
    return t;
}

// a.b in one workgroup (small vectors)
__global__ __launch_bounds__(kStepThreads) void k_dot_small(const double *__restrict__ a,
                                                            const double *__restrict__ b, int n, double *out) {
    __shared__ double sh[kStepThreads];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += kStepThreads) s += a[i] * b[i];
    const double t = wg_sum(s, sh);
    if (threadIdx.x == 0) *out = t;
}

// out = (b.b, |b - y|^2) in one workgroup; out is pinned host memory
__global__ __launch_bounds__(kStepThreads) void k_resid_norms(const double *__restrict__ b,
                                                              const double *__restrict__ y, int n, double *out) {
    __shared__ double sh[kStepThreads];
    double s = 0.0, q = 0.0;
    for (int i = threadIdx.x; i < n; i += kStepThreads) {
        const double d = b[i] - y[i];
        s += b[i] * b[i];
        q += d * d;
    }
    const double bb = wg_sum(s, sh), rr = wg_sum(q, sh);
    if (threadIdx.x == 0) {
        out[0] = bb;
        out[1] = rr;
    }
}

// r = b - y
__global__ void k_sub(double *__restrict__ r, const double *__restrict__ b, const double *__restrict__ y, size_t n) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) r[t] = b[t] - y[t];
}

__global__ void k_scale(double *__restrict__ y, const double *__restrict__ x, double a, size_t n) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] = a * x[t];
}

__global__ void k_axpy(double *__restrict__ y, const double *__restrict__ x, double a, size_t n) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] += a * x[t];
}

static unsigned red_blocks(size_t n) { return (unsigned)std::min<size_t>(kRedBlocks, std::max<size_t>(1, (n + 255) / 256)); }

static int dot(ib_system *s, const double *a, const double *b, double *out, hipStream_t st) {
    const size_t n = 3 * (size_t)s->NL;
    if (n <= kStepMaxN) {
        hipLaunchKernelGGL(k_dot_small, dim3(1), dim3(kStepThreads), 0, st, a, b, (int)n, out);
        LGF_HIP(hipGetLastError());
        return LGFIB_OK;
    }
    hipLaunchKernelGGL(k_dot, dim3(red_blocks(n)), dim3(256), 0, st, a, b, n, s->red.as<double>() + 2 * kRedBlocks,
                       s->cnt.as<unsigned>(), out);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

static int read_scal(ib_system *s, int slot, double *v, hipStream_t st) {
    LGF_HIP(hipMemcpyAsync(s->host_scal + slot, s->scal.as<double>() + slot, sizeof(double), hipMemcpyDeviceToHost, st));
    LGF_HIP(hipStreamSynchronize(st));
    *v = s->host_scal[slot];
    return LGFIB_OK;
}

// y = C x with an FP64 interface, field work in prec
static int matvec(ib_system *s, int prec, const double *x, double *y, hipStream_t st, const CgDir *dir = nullptr) {
    if (prec == LGF_F64) return schur_apply_t<double, double, double>(s, x, y, st, dir);
    return schur_apply_t<float, double, double>(s, x, y, st, dir);
}

// One CG iteration (new direction, matvec, p.Ap, x/r update with r.r, the copy
// of r.r to pinned memory) for iterations of parity `par`.
static int cg_iteration(ib_system *s, int prec, int par, hipStream_t st) {
    const size_t n = 3 * (size_t)s->NL;
    double *x = s->x.as<double>(), *r = s->r.as<double>(), *ap = s->ap.as<double>(), *red = s->red.as<double>();
    double *p[2] = {s->p.as<double>(), s->p2.as<double>()};
    double *rs = red + par * kRedBlocks, *rs_next = red + (1 - par) * kRedBlocks;   // rs_next holds the previous one
    const int nred = (int)red_blocks(n);
    const CgDir dir{r, p[1 - par], rs, rs_next, p[par], nred, (int)n};
    int rc;
    if ((rc = matvec(s, prec, p[par], ap, st, &dir))) return rc;
    hipLaunchKernelGGL(k_cg_xr, dim3(nred), dim3(256), 0, st, x, r, p[par], ap, red + 2 * kRedBlocks,
                       (int)gather_blocks(s->NL), rs, nred, n, rs_next, s->host_scal_dev + 64 + par * kRedBlocks);
    LGF_HIP(hipGetLastError());
    return LGFIB_OK;
}

// r.r after an iteration of parity par, once its event has passed
static double cg_rr(const ib_system *s, int par) {
    const double *p = s->host_scal + 64 + par * kRedBlocks;
    double v = 0.0;
    for (unsigned i = 0; i < red_blocks(3 * (size_t)s->NL); ++i) v += p[i];
    return v;
}

// r = b - C x, *rr = r.r, with C x the mean of nev FP64 matvecs C(s x) / s at
// scales s in [1, 2).  The operator is the same at every scale but not its
// roundings, so the mean carries 1 / sqrt(nev) of one matvec's rounding error
// (2200 markers, |x| = 2870 |b|: 1.3e-13 |b| of one matvec; that of x itself
// 1.7e-14).  Overwrites tmp and, for nev > 1, p and ap.
static int true_residual(ib_system *s, const double *b, const double *x, double *r, int nev, double *rr,
                         hipStream_t st) {
    const size_t n = 3 * (size_t)s->NL;
    const unsigned gb = nblocks(n, 256);
    double *y = s->tmp.as<double>(), *xs = s->p.as<double>();
    int rc;
    if (nev == 1) {
        if ((rc = matvec(s, LGF_F64, x, y, st))) return rc;
        hipLaunchKernelGGL(k_sub, dim3(gb), dim3(256), 0, st, r, b, y, n);
        LGF_HIP(hipGetLastError());
    } else {
        LGF_HIP(hipMemcpyAsync(r, b, n * 8, hipMemcpyDeviceToDevice, st));
        for (int e = 0; e < nev; ++e) {
            const double sc = 1.0 + (double)e / nev;
            hipLaunchKernelGGL(k_scale, dim3(gb), dim3(256), 0, st, xs, x, sc, n);
            LGF_HIP(hipGetLastError());
            if ((rc = matvec(s, LGF_F64, xs, y, st))) return rc;
            hipLaunchKernelGGL(k_axpy, dim3(gb), dim3(256), 0, st, r, (const double *)y, -1.0 / (sc * nev), n);
            LGF_HIP(hipGetLastError());
        }
    }
    if ((rc = dot(s, r, r, s->scal.as<double>() + 2, st))) return rc;
    return read_scal(s, 2, rr, st);
}

constexpr int kMaxMean = 64;         // matvecs of a true residual, at most
constexpr double kMeanReach = 16.0;  // and how far from the target they may help: sqrt(64), and an FP64 sweep's drift

static bool cg_graphs_wanted() {
    const char *e = getenv("LGFIB_CG_GRAPH");
    return !(e && e[0] == '0');
}

// Capture both parities of the CG iteration into graphs (on a private
// stream, after an eager matvec has created every plan, table spectrum and
// workspace the matvec touches).  Recaptured when the context's FFT
// workspaces have been reallocated by other work.
static int cg_graphs(ib_system *s, int prec, hipStream_t st, bool *ok) {
    const int pi = prec == LGF_F64 ? 1 : 0;
    *ok = false;
    if (!cg_graphs_wanted() || s->cg_nograph[pi]) return LGFIB_OK;
    lgfib_ctx *ctx = s->ctx;
    if (s->cg_exec[pi][0] && s->cg_work[pi][0] == ctx->work1.p && s->cg_work[pi][1] == ctx->work2.p &&
        s->cg_epoch[pi] == ctx->cache_epoch) {
        *ok = true;
        return LGFIB_OK;
    }
    if (ctx->profiling) return LGFIB_OK;   // profiling events stay out of graphs
    int rc;
    if ((rc = matvec(s, prec, s->p.as<double>(), s->tmp.as<double>(), st))) return rc;
    LGF_HIP(hipStreamSynchronize(st));
    if (!s->cap) LGF_HIP(hipStreamCreateWithFlags(&s->cap, hipStreamNonBlocking));
    for (int par = 0; par < 2; ++par) {
        if (s->cg_exec[pi][par]) {
            LGF_HIP(hipGraphExecDestroy(s->cg_exec[pi][par]));
            s->cg_exec[pi][par] = nullptr;
        }
        hipGraph_t g = nullptr;
        LGF_HIP(hipStreamBeginCapture(s->cap, hipStreamCaptureModeThreadLocal));
        rc = cg_iteration(s, prec, par, s->cap);
        const hipError_t e = hipStreamEndCapture(s->cap, &g);
        hipError_t ei = hipErrorUnknown;
        if (!rc && e == hipSuccess && g) ei = hipGraphInstantiate(&s->cg_exec[pi][par], g, nullptr, nullptr, 0);
        if (g) (void)hipGraphDestroy(g);
        if (ei != hipSuccess) {   // the eager loop runs the same kernels
            (void)hipGetLastError();
            for (auto &x : s->cg_exec[pi])
                if (x) {
                    (void)hipGraphExecDestroy(x);
                    x = nullptr;
                }
            s->cg_nograph[pi] = true;
            return LGFIB_OK;
        }
    }
    s->cg_work[pi][0] = ctx->work1.p;
    s->cg_work[pi][1] = ctx->work2.p;
    s->cg_epoch[pi] = ctx->cache_epoch;
    *ok = true;
    return LGFIB_OK;
}

}  // namespace lgfib

// column j of a row-major matrix: C[i][j] = y[i]
__global__ void k_put_column(double *__restrict__ C, long ld, int j, const double *__restrict__ y, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) C[(long)i * ld + j] = y[i];
}

__global__ void k_unit(double *__restrict__ e, int n, int j) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) e[i] = i == j ? 1.0 : 0.0;
}

static int direct_solve(ib_system *s, const double *b, double *f, ib_solve_stats_t *S, hipStream_t st) {
    const int n = 3 * s->NL;
    int rc;
    hipEvent_t e0, e1;
    LGF_HIP(hipEventCreate(&e0));
    LGF_HIP(hipEventCreate(&e1));
    LGF_HIP(hipEventRecord(e0, st));
    if ((rc = chol_solve_f64(s->ctx, n, s->wfac.as<double>(), n, b, f, st))) return rc;
    LGF_HIP(hipEventRecord(e1, st));
    if (S) {
        double *ap = s->ap.as<double>();
        if ((rc = matvec(s, LGF_F64, f, ap, st))) return rc;
        hipLaunchKernelGGL(k_resid_norms, dim3(1), dim3(kStepThreads), 0, st, b, ap, n, s->host_scal_dev);
        LGF_HIP(hipGetLastError());
    }
    LGF_HIP(hipStreamSynchronize(st));
    float ms = 0.f;
    LGF_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (S) {
        *S = ib_solve_stats_t{};
        S->ms = ms;
        const double bb = s->host_scal[0], rr = s->host_scal[1];
        S->rel_residual = bb > 0.0 ? sqrt(rr / bb) : 0.0;
    }
    return LGFIB_OK;
}

extern "C" int ib_force_solve(lgfib_ctx *ctx, ib_system *sys, int prec, const double *b, double *f, const double *x0,
                              double rtol, int maxit, ib_solve_stats_t *stats, lgfib_stream_t stream) {
    if (!ctx || !sys || sys->ctx != ctx) return fail(LGFIB_EINVAL, "ib_force_solve: bad context or system");
    if (prec == IB_SOLVE_DIRECT) {
        if (!b || !f) return fail(LGFIB_EINVAL, "ib_force_solve: null vector");
        if (!sys->factored) return fail(LGFIB_ENOTBUILT, "ib_force_solve: the system has no factor (ib_system_factor)");
        LGF_HIP(hipSetDevice(ctx->device));
        return direct_solve(sys, b, f, stats, (hipStream_t)stream);
    }
    if (prec != LGF_F32 && prec != LGF_F64) return fail(LGFIB_EINVAL, "ib_force_solve: bad prec");
    if (!b || !f) return fail(LGFIB_EINVAL, "ib_force_solve: null vector");
    if (!(rtol > 0.0) || maxit < 1) return fail(LGFIB_EINVAL, "ib_force_solve: rtol > 0 and maxit >= 1 required");
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    ib_solve_stats_t loc{};
    ib_solve_stats_t *S = stats ? stats : &loc;
    *S = ib_solve_stats_t{};
    hipEvent_t e0, e1;
    LGF_HIP(hipEventCreate(&e0));
    LGF_HIP(hipEventCreate(&e1));
    LGF_HIP(hipEventRecord(e0, st));
    const size_t n = 3 * (size_t)sys->NL;
    const unsigned gb = nblocks(n, 256);
    double *x = sys->x.as<double>(), *r = sys->r.as<double>(),
           *scal = sys->scal.as<double>();
    int rc;
    double bb;
    if ((rc = dot(sys, b, b, scal + 3, st)) || (rc = read_scal(sys, 3, &bb, st))) return rc;
    const double bnorm = sqrt(bb);
    if (bnorm == 0.0) {
        LGF_HIP(hipMemsetAsync(f, 0, n * 8, st));
        LGF_HIP(hipStreamSynchronize(st));
        S->rel_residual = 0.0;
        return LGFIB_OK;
    }
    // initial guess
    bool use_x0 = false;
    if (x0) {
        std::vector<double> h(n);
        LGF_HIP(hipMemcpyAsync(h.data(), x0, n * 8, hipMemcpyDeviceToHost, st));
        LGF_HIP(hipStreamSynchronize(st));
        use_x0 = true;
        for (double v : h)
            if (!std::isfinite(v)) {
                use_x0 = false;
                break;
            }
    }
    double rr;
    if (use_x0) {
        LGF_HIP(hipMemcpyAsync(x, x0, n * 8, hipMemcpyDeviceToDevice, st));
        if ((rc = true_residual(sys, b, x, r, 1, &rr, st))) return rc;
        S->restarts++;
        if (!(sqrt(rr) <= bnorm)) use_x0 = false;
    }
    if (!use_x0) {
        S->fallback = x0 ? 1 : 0;
        LGF_HIP(hipMemsetAsync(x, 0, n * 8, st));
        LGF_HIP(hipMemcpyAsync(r, b, n * 8, hipMemcpyDeviceToDevice, st));
        rr = bb;
    }
    // CG; with an FP32 matvec the recursive residual drifts from the true one,
    // so each sweep stops after reducing it by 1e-4 (or reaching the target),
    // and the next sweep restarts from the FP64 true residual.  The recursive
    // residual of iteration j is copied to pinned memory and read by the host
    // while iteration j+1 is already queued, so the device never waits for
    // the convergence test.
    // A true residual that a sweep has not halved may be the rounding of the
    // matvecs it is formed with (2200 markers on a sphere: 1e-15 to 1.3e-13 of |b|
    // by the velocities).  It is then formed, and the next sweeps start, from the
    // mean of 4, of 16 and at last of 64 of them; where that does not help
    // either, or the target is out of its reach, sweeps go on from single ones
    // up to maxit.  An FP64 solve, which one sweep takes to its floor, ends
    // there instead.
    const double target = rtol * bnorm;
    double true_r = sqrt(rr);
    int it = 0, nev = 1;
    bool mean = true;   // more matvecs may still help
    while (true_r > target && it < maxit) {
        const double sweep_stop = prec == LGF_F64 ? target : std::max(target * 0.5, true_r * 1e-4);
        // r.r as the only partial sum, and no previous one: beta = 0
        LGF_HIP(hipMemsetAsync(sys->red.p, 0, 2 * kRedBlocks * sizeof(double), st));
        if ((rc = dot(sys, r, r, sys->red.as<double>(), st))) return rc;
        bool graphs = false;
        if ((rc = cg_graphs(sys, prec, st, &graphs))) return rc;
        if (graphs) S->graphs = 1;
        int j = 0;
        bool stop = false;
        while (!stop && it < maxit) {
            if (graphs) {
                LGF_HIP(hipGraphLaunch(sys->cg_exec[prec == LGF_F64 ? 1 : 0][j & 1], st));
            } else if ((rc = cg_iteration(sys, prec, j & 1, st))) {
                return rc;
            }
            LGF_HIP(hipEventRecord(sys->ev[j & 1], st));
            ++it;
            ++j;
            if (j >= 2) {   // test iteration j-2 (0-based) while j-1 runs
                LGF_HIP(hipEventSynchronize(sys->ev[j & 1]));
                const double rsn = cg_rr(sys, j & 1);
                if (sqrt(rsn) <= sweep_stop || !std::isfinite(rsn)) stop = true;
            }
        }
        const double last = true_r;
        if ((rc = true_residual(sys, b, x, r, nev, &rr, st))) return rc;
        if (mean && it < maxit && sqrt(rr) > target && !(sqrt(rr) <= 0.5 * last) && sqrt(rr) <= kMeanReach * target) {
            mean = nev < kMaxMean;
            nev = mean ? 4 * nev : 1;
            if (mean && (rc = true_residual(sys, b, x, r, nev, &rr, st))) return rc;
        }
        true_r = sqrt(rr);
        const bool ends = !std::isfinite(true_r) || (prec == LGF_F64 && !(mean && true_r <= kMeanReach * target));
        if (prec != LGF_F64 || (true_r > target && it < maxit && !ends)) S->restarts++;
        if (ends) break;
    }
    LGF_HIP(hipMemcpyAsync(f, x, n * 8, hipMemcpyDeviceToDevice, st));
    LGF_HIP(hipEventRecord(e1, st));
    LGF_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    LGF_HIP(hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    S->iterations = it;
    S->rel_residual = true_r / bnorm;
    S->ms = ms;
    if (!(true_r <= target)) {
        char msg[128];
        snprintf(msg, sizeof msg, "ib_force_solve: relative residual %.3e after %d iterations", true_r / bnorm, it);
        return fail(LGFIB_ENOCONV, msg);
    }
    return LGFIB_OK;
}

// ------------------------------------------------------------ Stokes driver
//
// One integrating-factor Euler step (one-stage IF-HERK with a11 = c1 = 1,
// H = E(a), nonlinear term omitted) of the discrete Stokes equations with a
// rigid immersed surface, by the nested projection of Sec. 3.1:
//   (ip)  d* = L^{-1}(-G^T u_k)
//   (f)   C f = I H [u_k - G d*] - u_B(t_{k+1})
//   (pc)  d  = d* + L^{-1} G^T R f
//   (vc)  u_{k+1} = H [u_k - G d - R f]
// (in (f) the faces u_k - G d* are read as the face field that H acts on).
// Velocities live on the flow blocks D_flow (which hold D_body).  The cell
// variables live on D_flow and its lower neighbours (every block b - (i,j,k),
// i,j,k in {0,1}): the divergence of a face field on D_flow reaches the layer
// of cells below its lower faces, and the gradient at those faces reads it,
// so u - G d is the unbounded lattice's projection restricted to D_flow (a
// non-expansive step).  The force solve uses the body system.  Lattice
// units, FP64 state.

struct ib_flow {
    lgfib_ctx *ctx = nullptr;
    ib_system *sys = nullptr;
    int B = 0, nflow = 0, ncell = 0;
    std::vector<int32_t> blocks;    // D_flow (faces)
    std::vector<int32_t> cblocks;   // cell blocks
    std::shared_ptr<IbPlan> plan;   // markers binned on the flow blocks (held: pinned in the cache)
    int clo[3] = {0, 0, 0}, cnb[3] = {0, 0, 0};
    DevBuf cmap, cblk;              // block map of the cell blocks
    lgf_table_t tbl = -1;           // G_L over the cell span
    DevBuf c, dstar, w, h, rhs;
    std::shared_ptr<FlowOps> ops;   // shared by the plan's flows
};

namespace lgfib {
// The drivers' stencils.  FP64 streams of 3 B^3 faces a block, bound by HBM once
// the index arithmetic is out of the way: one block per B^3 threads, shifts for
// the power-of-two block edge, and a block lookup only where the neighbour lies
// in another block.  With 64-bit divisions and a lookup for every face the two
// took 24.6 and 14.9 us on 1728 blocks of 8^3 at 99% and 81% VALU activity; now
// 10.7 and 14.1, and 24.6 for the second gradient with its five streams.
struct CellAt {
    int b, cell, l[3];
};
__device__ __forceinline__ CellAt cell_at(unsigned t, int lb) {
    const int m = (1 << lb) - 1;
    CellAt a;
    a.b = (int)(t >> (3 * lb));
    a.cell = (int)(t & ((1u << (3 * lb)) - 1));
    a.l[0] = a.cell & m;
    a.l[1] = (a.cell >> lb) & m;
    a.l[2] = a.cell >> (2 * lb);
    return a;
}

// c(n) = sc sum_k u^(k)(n) - u^(k)(n + e_k) on the cell blocks A; faces u on
// the flow blocks F (zero elsewhere)
__global__ __launch_bounds__(256) void k_div_cross(BlockMapDev F, BlockMapDev A, int lb, const double *__restrict__ u,
                                                   double *__restrict__ c, int nF, unsigned ncell, double sc) {
    const unsigned t = blockIdx.x * 256 + threadIdx.x;
    if (t >= ncell) return;
    const CellAt a = cell_at(t, lb);
    const int top = (1 << lb) - 1;
    const int bx = A.blocks[3 * a.b], by = A.blocks[3 * a.b + 1], bz = A.blocks[3 * a.b + 2];
    const int own = F.slot(bx, by, bz);
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double *uk = u + ((size_t)k * nF << (3 * lb));
        const bool up = a.l[k] == top;
        const int nb = up ? F.slot(bx + (k == 0), by + (k == 1), bz + (k == 2)) : own;
        const int ncl = a.cell + ((up ? -top : 1) << (k * lb));
        if (own >= 0) s += uk[((size_t)own << (3 * lb)) + a.cell];
        if (nb >= 0) s -= uk[((size_t)nb << (3 * lb)) + ncl];
    }
    c[t] = sc * s;
}

// On the faces of F, with d on the cell blocks A (which hold F and its lower
// neighbours): w = u - G d, and in its second form w = u - q, q = G d + rf, of
// which qlam (nullable) receives q - g (g nullable).
template <bool SECOND>
__global__ __launch_bounds__(256) void k_grad_cross(BlockMapDev F, BlockMapDev A, int lb, const double *__restrict__ u,
                                                    const double *__restrict__ d, const double *__restrict__ rf,
                                                    const double *__restrict__ g, double *__restrict__ w,
                                                    double *__restrict__ qlam, int nF, unsigned nface) {
    const unsigned t = blockIdx.x * 256 + threadIdx.x;
    if (t >= nface) return;
    const CellAt a = cell_at(t, lb);
    const int top = (1 << lb) - 1;
    const int bx = F.blocks[3 * a.b], by = F.blocks[3 * a.b + 1], bz = F.blocks[3 * a.b + 2];
    const int own = A.slot(bx, by, bz);
    const double dc = d[((size_t)own << (3 * lb)) + a.cell];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const bool low = a.l[k] == 0;
        const int nb = low ? A.slot(bx - (k == 0), by - (k == 1), bz - (k == 2)) : own;
        const int ncl = a.cell + ((low ? top : -1) * (1 << (k * lb)));
        const double dm = nb >= 0 ? d[((size_t)nb << (3 * lb)) + ncl] : 0.0;
        const size_t i = ((size_t)k * nF << (3 * lb)) + t;
        if constexpr (SECOND) {
            const double q = (dc - dm) + rf[i];
            w[i] = u[i] - q;
            if (qlam) qlam[i] = g ? q - g[i] : q;
        } else {
            w[i] = u[i] - (dc - dm);
        }
    }
}

// r = h + sum_j c[j] q[j] + g (terms in this order; null q and g are left out)
struct HerkTerms {
    const double *q[7];
    double c[7];
};
__global__ __launch_bounds__(256) void k_combine(double *__restrict__ r, const double *__restrict__ h, HerkTerms m,
                                                 const double *__restrict__ g, size_t n) {
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    double v = h[t];
#pragma unroll
    for (int j = 0; j < 7; ++j)
        if (m.q[j]) v += m.c[j] * m.q[j][t];
    if (g) v += g[t];
    r[t] = v;
}
}  // namespace lgfib

extern "C" int ib_flow_create(lgfib_ctx *ctx, ib_system *sys, const int32_t *flow_blocks, int nflow,
                              ib_flow **out) {
    if (!out) return fail(LGFIB_EINVAL, "ib_flow_create: null output");
    *out = nullptr;
    if (!ctx || !sys || sys->ctx != ctx) return fail(LGFIB_EINVAL, "ib_flow_create: bad context or system");
    if (nflow < 1 || !flow_blocks) return fail(LGFIB_EINVAL, "ib_flow_create: need flow blocks");
    LGF_HIP(hipSetDevice(ctx->device));
    int rc = validate_blocks(flow_blocks, nflow, "flow blocks");
    if (rc) return rc;
    // D_body must be contained in D_flow
    {
        std::unordered_map<uint64_t, int> in;
        auto key = [](const int32_t *b) {
            return ((uint64_t)(uint32_t)(b[0] + (1 << 20))) | ((uint64_t)(uint32_t)(b[1] + (1 << 20)) << 21) |
                   ((uint64_t)(uint32_t)(b[2] + (1 << 20)) << 42);
        };
        for (int i = 0; i < nflow; ++i) in[key(flow_blocks + 3 * i)] = i;
        for (int i = 0; i < sys->nblk; ++i)
            if (!in.count(key(sys->blocks.data() + 3 * i)))
                return fail(LGFIB_EINVAL, "ib_flow_create: a body block is not among the flow blocks");
    }
    auto f = std::make_unique<ib_flow>();
    f->ctx = ctx;
    f->sys = sys;
    f->B = sys->B;
    f->nflow = nflow;
    f->blocks.assign(flow_blocks, flow_blocks + 3 * (size_t)nflow);
    IbHost host;
    if ((rc = build_ib_plan(ctx, sys->kernel, sys->X.data(), sys->NL, sys->B, flow_blocks, nflow, f->plan, &host)))
        return rc;
    // cell blocks: the flow blocks and their lower neighbours, sorted (z, y, x)
    {
        std::vector<std::array<int32_t, 3>> v;
        v.reserve(8 * (size_t)nflow);
        for (int i = 0; i < nflow; ++i)
            for (int dz = 0; dz < 2; ++dz)
                for (int dy = 0; dy < 2; ++dy)
                    for (int dx = 0; dx < 2; ++dx)
                        v.push_back({flow_blocks[3 * i] - dx, flow_blocks[3 * i + 1] - dy, flow_blocks[3 * i + 2] - dz});
        std::sort(v.begin(), v.end(), [](const std::array<int32_t, 3> &a, const std::array<int32_t, 3> &b) {
            if (a[2] != b[2]) return a[2] < b[2];
            if (a[1] != b[1]) return a[1] < b[1];
            return a[0] < b[0];
        });
        v.erase(std::unique(v.begin(), v.end()), v.end());
        for (auto &b : v) f->cblocks.insert(f->cblocks.end(), b.begin(), b.end());
        f->ncell = (int)v.size();
    }
    if ((rc = validate_blocks(f->cblocks.data(), f->ncell, "cell blocks"))) return rc;
    {
        int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-(1 << 30), -(1 << 30), -(1 << 30)};
        for (int i = 0; i < f->ncell; ++i)
            for (int a = 0; a < 3; ++a) {
                lo[a] = std::min(lo[a], f->cblocks[3 * i + a]);
                hi[a] = std::max(hi[a], f->cblocks[3 * i + a]);
            }
        size_t msize = 1;
        for (int a = 0; a < 3; ++a) {
            f->clo[a] = lo[a];
            f->cnb[a] = hi[a] - lo[a] + 1;
            msize *= (size_t)f->cnb[a];
        }
        if (msize > (size_t)1 << 28) return fail(LGFIB_ERANGE, "ib_flow_create: flow blocks span too large a box");
        std::vector<int32_t> map(msize, -1);
        for (int i = 0; i < f->ncell; ++i)
            map[((size_t)(f->cblocks[3 * i + 2] - lo[2]) * f->cnb[1] + (f->cblocks[3 * i + 1] - lo[1])) * f->cnb[0] +
                (f->cblocks[3 * i] - lo[0])] = i;
        if ((rc = f->cmap.reserve(map.size() * 4)) || (rc = f->cblk.reserve(f->cblocks.size() * 4))) return rc;
        LGF_HIP(hipMemcpy(f->cmap.p, map.data(), map.size() * 4, hipMemcpyHostToDevice));
        LGF_HIP(hipMemcpy(f->cblk.p, f->cblocks.data(), f->cblocks.size() * 4, hipMemcpyHostToDevice));
        if (!(f->ops = f->plan->flow.lock())) {   // the plan's blocks determine the cells
            auto o = std::make_shared<FlowOps>();
            const size_t ncc = (size_t)f->ncell * f->B * f->B * f->B, nf = 3 * (size_t)nflow * f->B * f->B * f->B;
            if ((rc = build_spread(*f->plan, flow_blocks, CellSet{f->clo, f->cnb, map}, (int64_t)ncc, host, o->spread,
                                   nullptr)) ||
                (rc = o->cf.reserve(ncc * 8)) || (rc = o->rf.reserve(nf * 8)))
                return rc;
            LGF_HIP(hipMemset(o->cf.p, 0, ncc * 8));
            LGF_HIP(hipMemset(o->rf.p, 0, nf * 8));
            LGF_HIP(hipStreamSynchronize(nullptr));
            f->plan->flow = f->ops = std::move(o);
        }
    }
    int ext[3];
    for (int q = 0; q < 3; ++q) ext[q] = f->cnb[q] * sys->B - 1;
    if ((rc = lgf_table_build(ctx, LGF_KIND_L, 0.0, ext, nullptr, &f->tbl))) return rc;
    const size_t B3 = (size_t)sys->B * sys->B * sys->B;
    const size_t nfc = (size_t)nflow * B3, ncc = (size_t)f->ncell * B3;
    if ((rc = f->c.reserve(ncc * 8)) || (rc = f->dstar.reserve(ncc * 8)) || (rc = f->w.reserve(3 * nfc * 8)) ||
        (rc = f->h.reserve(3 * nfc * 8)) || (rc = f->rhs.reserve(3 * (size_t)sys->NL * 8)))
        return rc;
    *out = f.release();
    return LGFIB_OK;
}

extern "C" void ib_flow_destroy(ib_flow *flow) {
    if (!flow) return;
    (void)hipSetDevice(flow->ctx->device);
    (void)hipDeviceSynchronize();
    delete flow;
}

// One stage system H^{-1} u' + Q lam = u, Q^T u' = (0, u_B) by the nested
// projection; u is the right-hand side, u_out (may be u) receives u'; qlam
// (nullable, faces) receives Q lam - g = G d + R f - g (g nullable).
static int flow_stage(lgfib_ctx *ctx, ib_flow *fl, const double *u, double *u_out, const double *ub, double *f,
                      const double *x0, double rtol, int maxit, int prec, ib_solve_stats_t *stats, double *b_out,
                      const double *g, double *qlam, hipStream_t st) {
    ib_system *sys = fl->sys;
    const IbPlan &P = *fl->plan;
    const int B = fl->B, lb = log2_edge(B);
    const size_t B3 = (size_t)B * B * B;
    const size_t nfc = (size_t)fl->nflow * B3, nf = 3 * nfc, ncc = (size_t)fl->ncell * B3, nl = 3 * (size_t)sys->NL;
    double *c = fl->c.as<double>(), *d = fl->dstar.as<double>(), *rf = fl->ops->rf.as<double>();
    double *w = fl->w.as<double>(), *h = fl->h.as<double>(), *rhs = fl->rhs.as<double>();
    const int32_t *bl = fl->blocks.data(), *cb = fl->cblocks.data();
    const int nb = fl->nflow, nc = fl->ncell;
    const BlockMapDev Fm = devmap(P);
    BlockMapDev Am;
    Am.lo0 = fl->clo[0];
    Am.lo1 = fl->clo[1];
    Am.lo2 = fl->clo[2];
    Am.nb0 = fl->cnb[0];
    Am.nb1 = fl->cnb[1];
    Am.nb2 = fl->cnb[2];
    Am.B = B;
    Am.map = fl->cmap.as<int>();
    Am.blocks = fl->cblk.as<int>();
    int rc;
    // (ip) d* = L^{-1}(-G^T u)
    hipLaunchKernelGGL(k_div_cross, dim3(nblocks(ncc, 256)), dim3(256), 0, st, Fm, Am, lb, u, c, nb, (unsigned)ncc,
                       -1.0);
    LGF_HIP(hipGetLastError());
    if ((rc = lgf_poisson_apply(ctx, fl->tbl, B, cb, nc, cb, nc, 1, LGF_F64, 1.0, c, d, 0, (lgfib_stream_t)st))) return rc;
    // (f) b = I E(a)[u - G d*] - u_B ;  C f = b
    hipLaunchKernelGGL(k_grad_cross<false>, dim3(nblocks(nfc, 256)), dim3(256), 0, st, Fm, Am, lb, u, (const double *)d,
                       (const double *)nullptr, (const double *)nullptr, w, (double *)nullptr, nb, (unsigned)nfc);
    LGF_HIP(hipGetLastError());
    if ((rc = lgf_if_apply(ctx, sys->a, B, bl, nb, bl, nb, 3, LGF_F64, w, h, (lgfib_stream_t)st))) return rc;
    if ((rc = launch_interpolate<double, double>(ctx, P, h, rhs, st, ub))) return rc;
    if (b_out) LGF_HIP(hipMemcpyAsync(b_out, rhs, nl * 8, hipMemcpyDeviceToDevice, st));
    rc = ib_force_solve(ctx, sys, prec, rhs, f, x0, rtol, maxit, stats, (lgfib_stream_t)st);
    if (rc && rc != LGFIB_ENOCONV) return rc;
    const int solve_rc = rc;
    // (pc) d = d* + L^{-1} G^T R f
    if ((rc = launch_spread<double, double>(ctx, fl->ops->spread, f, nullptr, rf, fl->ops->cf.as<double>(), st))) return rc;
    if ((rc = lgf_poisson_apply(ctx, fl->tbl, B, cb, nc, cb, nc, 1, LGF_F64, 1.0, fl->ops->cf.p, d, 1, (lgfib_stream_t)st)))
        return rc;
    // (vc) u' = E(a)[u - G d - R f]
    hipLaunchKernelGGL(k_grad_cross<true>, dim3(nblocks(nfc, 256)), dim3(256), 0, st, Fm, Am, lb, u, (const double *)d,
                       (const double *)rf, g, w, qlam, nb, (unsigned)nfc);
    LGF_HIP(hipGetLastError());
    if ((rc = lgf_if_apply(ctx, sys->a, B, bl, nb, bl, nb, 3, LGF_F64, w, u_out, (lgfib_stream_t)st))) return rc;
    return solve_rc;
}

extern "C" int ib_flow_step(lgfib_ctx *ctx, ib_flow *fl, double *u, const double *ub, double *f, const double *x0,
                            double rtol, int maxit, int prec, ib_solve_stats_t *stats, double *b_out,
                            lgfib_stream_t stream) {
    if (!ctx || !fl || fl->ctx != ctx) return fail(LGFIB_EINVAL, "ib_flow_step: bad context or flow");
    if (!u || !ub || !f) return fail(LGFIB_EINVAL, "ib_flow_step: null vector");
    LGF_HIP(hipSetDevice(ctx->device));
    const int rc = flow_stage(ctx, fl, u, u, ub, f, x0, rtol, maxit, prec, stats, b_out, nullptr, nullptr,
                              (hipStream_t)stream);
    if (rc && rc != LGFIB_ENOCONV) return rc;
    LGF_HIP(hipStreamSynchronize((hipStream_t)stream));
    return rc;
}

// Columns j0 .. j0+K-1 of C in one pass (FP64): the operator of
// schur_apply_t on K unit vectors, with the integrating factor applied to
// the 3K face components and the K^{-1} convolution to the K cell fields in
// shared launches (each component is transformed on its own, so the columns
// are those of K separate applications).
static constexpr int kDenseCols = 8;
static int schur_dense_cols(ib_system *s, int j0, int K, double *C, long ld, hipStream_t st) {
    lgfib_ctx *ctx = s->ctx;
    const IbPlan &P = *s->plan;
    const int n = 3 * s->NL;
    const size_t nc = (size_t)s->nblk * s->B * s->B * s->B, nf = 3 * nc;
    double *base = s->dense_cols.as<double>();
    double *g = base, *af = g + kDenseCols * nf, *c = af + kDenseCols * nf, *d = c + kDenseCols * nc;
    double *e = d + kDenseCols * nc, *y = e + (size_t)kDenseCols * n;
    int rc;
    for (int k = 0; k < K; ++k) {
        hipLaunchKernelGGL(k_unit, dim3(nblocks(n, 256)), dim3(256), 0, st, e + (size_t)k * n, n, j0 + k);
        LGF_HIP(hipGetLastError());
        if ((rc = launch_spread<double, double>(ctx, s->grad->spread, e + (size_t)k * n, nullptr, g + k * nf, c + k * nc, st)))
            return rc;
    }
    for (int c0 = 0; c0 < 3 * K; c0 += 8) {
        const int m = std::min(8, 3 * K - c0);
        if ((rc = lgf_if_apply(ctx, s->a, s->B, s->blocks.data(), s->nblk, s->blocks.data(), s->nblk, m, LGF_F64,
                               g + c0 * nc, af + c0 * nc, (lgfib_stream_t)st)))
            return rc;
    }
    if ((rc = lgf_poisson_apply(ctx, s->tbl, s->B, s->blocks.data(), s->nblk, s->blocks.data(), s->nblk, K, LGF_F64,
                                1.0, c, d, 0, (lgfib_stream_t)st)))
        return rc;
    for (int k = 0; k < K; ++k) {
        if ((rc = launch_gather<double, double>(ctx, P, *s->grad, af + k * nf, d + k * nc, y + (size_t)k * n, nullptr, nullptr,
                                                st)))
            return rc;
        hipLaunchKernelGGL(k_put_column, dim3(nblocks(n, 256)), dim3(256), 0, st, C, ld, j0 + k,
                           (const double *)(y + (size_t)k * n), n);
        LGF_HIP(hipGetLastError());
    }
    return LGFIB_OK;
}

extern "C" int ib_schur_dense(lgfib_ctx *ctx, ib_system *sys, double *C, int ld, lgfib_stream_t stream) {
    if (!ctx || !sys || sys->ctx != ctx) return fail(LGFIB_EINVAL, "ib_schur_dense: bad context or system");
    const int n = 3 * sys->NL;
    if (!C || ld < n) return fail(LGFIB_EINVAL, "ib_schur_dense: null matrix or ld < 3 NL");
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const size_t nc = (size_t)sys->nblk * sys->B * sys->B * sys->B;
    int rc;
    if ((rc = sys->dense_cols.reserve(((size_t)kDenseCols * (8 * nc + 2 * (size_t)n)) * sizeof(double)))) return rc;
    // g and c of the columns (schur_dense_cols' layout): zeros where no marker reaches
    LGF_HIP(hipMemsetAsync(sys->dense_cols.p, 0, kDenseCols * 3 * nc * sizeof(double), st));
    LGF_HIP(hipMemsetAsync(sys->dense_cols.as<double>() + kDenseCols * 6 * nc, 0, kDenseCols * nc * sizeof(double), st));
    for (int j = 0; j < n; j += kDenseCols)
        if ((rc = schur_dense_cols(sys, j, std::min(kDenseCols, n - j), C, (long)ld, st))) return rc;
    LGF_HIP(hipStreamSynchronize(st));
    return LGFIB_OK;
}

extern "C" int ib_system_factor(lgfib_ctx *ctx, ib_system *sys, int enable, lgfib_stream_t stream) {
    if (!ctx || !sys || sys->ctx != ctx) return fail(LGFIB_EINVAL, "ib_system_factor: bad context or system");
    LGF_HIP(hipSetDevice(ctx->device));
    if (!enable) {
        sys->factored = false;
        sys->wfac.release();
        return LGFIB_OK;
    }
    const size_t n = 3 * (size_t)sys->NL;
    if (n > 46000) return fail(LGFIB_EINVAL, "ib_system_factor: more than 46000 unknowns");
    sys->factored = false;
    DevBuf C;
    int rc;
    if ((rc = C.reserve(n * n * 8)) || (rc = sys->wfac.reserve(n * n * 8))) return rc;
    if ((rc = ib_schur_dense(ctx, sys, C.as<double>(), (int)n, stream))) return rc;
    if ((rc = chol_factor_f64(ctx, (int)n, C.as<double>(), (long)n, sys->wfac.as<double>(), (long)n,
                              (hipStream_t)stream)))
        return rc;
    sys->factored = true;
    return LGFIB_OK;
}

// ------------------------------------------------------------- IF-HERK step

struct ib_herk {
    lgfib_ctx *ctx = nullptr;
    int s = 0, NL = 0, B = 0, nflow = 0;
    double A = 0.0;
    bool direct = false, have_prev = false;
    std::vector<double> at, ct, stage_a;   // shifted tableau, nodes, H parameter of each stage
    std::vector<ib_system *> systems;      // one per distinct stage parameter (owned)
    std::vector<ib_flow *> flows;
    std::vector<int> stage_k;              // system / flow of each stage
    std::vector<int32_t> fblocks;
    double conv_dt = 0.0;                  // dt / dx of the nonlinear term (0: Stokes)
    double U[3] = {0.0, 0.0, 0.0};         // frame velocity in u_a = u + U
    DevBuf fields;   // (s + 4) face fields: h, tmp, r, Q lam - g of each stage, g
    DevBuf forces;   // s marker vectors: the stages' forces of the last step
};

extern "C" void ib_herk_destroy(ib_herk *hk) {
    if (!hk) return;
    for (auto *fl : hk->flows) ib_flow_destroy(fl);
    for (auto *sy : hk->systems) ib_system_destroy(sy);
    delete hk;
}

extern "C" int ib_herk_tableau(int scheme, int *s, double *at, double *ct) {
    if (!s || !at || !ct || scheme < 0 || scheme > 3) return fail(LGFIB_EINVAL, "ib_herk_tableau: bad argument");
    const double r3 = std::sqrt(3.0);
    // explicit tableaus (A, b, c) of App. B; the shifted form is
    // at_{ij} = A_{i+1,j} (i < s), at_{sj} = b_j, ct_i = c_{i+1}, ct_s = 1
    static const int ns[4] = {3, 3, 3, 4};
    double Am[4][4] = {}, b[4] = {}, c[4] = {};
    switch (scheme) {
    case 0:
        Am[1][0] = 0.5;
        Am[2][0] = r3 / 3, Am[2][1] = (3 - r3) / 3;
        b[0] = (3 + r3) / 6, b[1] = -r3 / 3, b[2] = (3 + r3) / 6;
        c[1] = 0.5, c[2] = 1.0;
        break;
    case 1:
        Am[1][0] = 1.0 / 3;
        Am[2][0] = -1.0, Am[2][1] = 2.0;
        b[1] = 0.75, b[2] = 0.25;
        c[1] = 1.0 / 3, c[2] = 1.0;
        break;
    case 2:
        Am[1][0] = 8.0 / 15;
        Am[2][0] = 0.25, Am[2][1] = 5.0 / 12;
        b[0] = 0.25, b[2] = 0.75;
        c[1] = 8.0 / 15, c[2] = 2.0 / 3;
        break;
    default:   // the classical four-stage method
        Am[1][0] = 0.5;
        Am[2][1] = 0.5;
        Am[3][2] = 1.0;
        b[0] = 1.0 / 6, b[1] = 1.0 / 3, b[2] = 1.0 / 3, b[3] = 1.0 / 6;
        c[1] = 0.5, c[2] = 0.5, c[3] = 1.0;
        break;
    }
    const int n = ns[scheme];
    *s = n;
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < n; ++j) at[i * n + j] = i + 1 < n ? Am[i + 1][j] : b[j];
        ct[i] = i + 1 < n ? c[i + 1] : 1.0;
    }
    return LGFIB_OK;
}

extern "C" int ib_herk_create(lgfib_ctx *ctx, int kernel, const double *X, int NL, int B, const int32_t *body_blocks,
                              int nbody, const int32_t *flow_blocks, int nflow, double A, int s, const double *at,
                              const double *ct, int direct, ib_herk **out) {
    if (!out) return fail(LGFIB_EINVAL, "ib_herk_create: null output");
    *out = nullptr;
    if (!ctx || !at || !ct || !flow_blocks || nflow < 1) return fail(LGFIB_EINVAL, "ib_herk_create: bad argument");
    if (s < 1 || s > 8) return fail(LGFIB_EINVAL, "ib_herk_create: s must lie in [1, 8]");
    if (!(A >= 0.0) || A > 4.0) return fail(LGFIB_EINVAL, "ib_herk_create: A must lie in [0, 4]");
    double prev = 0.0;
    for (int i = 0; i < s; ++i) {
        if (!(ct[i] >= prev) || ct[i] > 1.0) return fail(LGFIB_EINVAL, "ib_herk_create: nodes must be nondecreasing in [0, 1]");
        if (!(std::fabs(at[i * s + i]) > 0.0)) return fail(LGFIB_EINVAL, "ib_herk_create: zero diagonal coefficient");
        for (int j = i + 1; j < s; ++j)
            if (at[i * s + j] != 0.0) return fail(LGFIB_EINVAL, "ib_herk_create: tableau must be lower triangular");
        prev = ct[i];
    }
    auto hk = std::unique_ptr<ib_herk, void (*)(ib_herk *)>(new ib_herk, ib_herk_destroy);
    hk->ctx = ctx;
    hk->s = s;
    hk->NL = NL;
    hk->B = B;
    hk->nflow = nflow;
    hk->A = A;
    hk->direct = direct != 0;
    hk->at.assign(at, at + s * s);
    hk->ct.assign(ct, ct + s);
    hk->fblocks.assign(flow_blocks, flow_blocks + 3 * (size_t)nflow);
    int rc;
    prev = 0.0;
    for (int i = 0; i < s; ++i) {
        const double a = (ct[i] - prev) * A;
        prev = ct[i];
        hk->stage_a.push_back(a);
        int k = -1;
        for (int q = 0; q < i; ++q)
            if (std::fabs(hk->stage_a[q] - a) <= 1e-14 * std::max(1.0, std::fabs(a))) k = hk->stage_k[q];
        if (k < 0) {
            ib_system *sy = nullptr;
            if ((rc = ib_system_create(ctx, kernel, X, NL, B, body_blocks, nbody, a, &sy))) return rc;
            hk->systems.push_back(sy);
            if (hk->direct && (rc = ib_system_factor(ctx, sy, 1, nullptr))) return rc;
            ib_flow *fl = nullptr;
            if ((rc = ib_flow_create(ctx, sy, flow_blocks, nflow, &fl))) return rc;
            hk->flows.push_back(fl);
            k = (int)hk->systems.size() - 1;
        }
        hk->stage_k.push_back(k);
    }
    const size_t nf = 3 * (size_t)nflow * B * B * B, nl = 3 * (size_t)NL;
    if ((rc = hk->fields.reserve((size_t)(s + 4) * nf * 8)) || (rc = hk->forces.reserve((size_t)s * nl * 8)))
        return rc;
    *out = hk.release();
    return LGFIB_OK;
}

extern "C" int ib_herk_step(lgfib_ctx *ctx, ib_herk *hk, double *u, const double *ub, double *f, double rtol,
                            int maxit, int prec, ib_solve_stats_t *stats, lgfib_stream_t stream) {
    if (!ctx || !hk || hk->ctx != ctx) return fail(LGFIB_EINVAL, "ib_herk_step: bad context or step");
    if (!u || !ub || !f) return fail(LGFIB_EINVAL, "ib_herk_step: null vector");
    if (!hk->direct && prec != LGF_F32 && prec != LGF_F64) return fail(LGFIB_EINVAL, "ib_herk_step: bad prec");
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const int s = hk->s, B = hk->B, nb = hk->nflow;
    const size_t nf = 3 * (size_t)nb * B * B * B, nl = 3 * (size_t)hk->NL;
    const int32_t *bl = hk->fblocks.data();
    double *base = hk->fields.as<double>();
    double *h = base, *tmp = base + nf, *r = base + 2 * nf;
    std::vector<double *> q(s);
    for (int j = 0; j < s; ++j) q[j] = base + (3 + j) * nf;
    double *g = base + (3 + s) * nf;
    const bool conv = hk->conv_dt > 0.0;
    const double *ustage = u;   // u^{i-1}: the step's input, then each stage's solution (left in r)
    const double *hcur = u;     // h^i: the step's input until it has been propagated into h
    if (stats) *stats = ib_solve_stats_t{};
    int rc, solve_rc = LGFIB_OK;
    for (int i = 0; i < s; ++i) {
        const double ap = i > 0 ? hk->stage_a[i - 1] : 0.0;
        if (ap > 0.0) {   // h <- H^{i-1} h, Q lam^j <- H^{i-1} Q lam^j
            if ((rc = lgf_if_apply(ctx, ap, B, bl, nb, bl, nb, 3, LGF_F64, hcur, tmp, stream))) return rc;
            std::swap(h, tmp);
            hcur = h;
            for (int j = 0; j < i; ++j) {
                if ((rc = lgf_if_apply(ctx, ap, B, bl, nb, bl, nb, 3, LGF_F64, q[j], tmp, stream))) return rc;
                std::swap(q[j], tmp);
            }
        }
        // g^i = -at_ii dt N~(u^{i-1}) (Eq. ibifherk_g), before r is overwritten
        if (conv && (rc = lamb_apply(ctx, B, bl, nb, hk->U, -hk->at[i * s + i] * hk->conv_dt, LGF_F64, ustage, g, st)))
            return rc;
        // r = h - sum_j (at_ij / at_jj) (Q lam^j - g^j) + g^i
        HerkTerms terms{};
        for (int j = 0; j < i; ++j) {
            terms.c[j] = -hk->at[i * s + j] / hk->at[j * s + j];
            terms.q[j] = terms.c[j] == 0.0 ? nullptr : q[j];
        }
        hipLaunchKernelGGL(k_combine, dim3(nblocks(nf, 256)), dim3(256), 0, st, r, hcur, terms,
                           (const double *)(conv ? g : nullptr), nf);
        LGF_HIP(hipGetLastError());
        // the stage's force stays where the next step's solve starts from; its
        // propagated field is Q lam^i - g^i; the last stage's u is the step's
        double *fi = hk->forces.as<double>() + i * nl;
        ib_solve_stats_t si{};
        rc = flow_stage(ctx, hk->flows[hk->stage_k[i]], r, i == s - 1 ? u : r, ub + i * nl, fi,
                        (!hk->direct && hk->have_prev) ? fi : nullptr, rtol, maxit,
                        hk->direct ? IB_SOLVE_DIRECT : prec, &si, nullptr, conv ? g : nullptr, q[i], st);
        if (rc && rc != LGFIB_ENOCONV) return rc;
        if (rc) solve_rc = rc;
        ustage = r;
        if (stats) {
            stats->iterations += si.iterations;
            stats->restarts += si.restarts;
            stats->fallback += si.fallback;
            stats->ms += si.ms;
            stats->graphs = si.graphs;
            stats->rel_residual = std::max(stats->rel_residual, si.rel_residual);
        }
    }
    hipLaunchKernelGGL(k_scale, dim3(nblocks(nl, 256)), dim3(256), 0, st, f,
                       (const double *)(hk->forces.as<double>() + (s - 1) * nl), 1.0 / hk->at[(s - 1) * s + s - 1], nl);
    LGF_HIP(hipGetLastError());
    LGF_HIP(hipStreamSynchronize(st));
    hk->have_prev = true;
    return solve_rc;
}

extern "C" int ib_herk_convection(lgfib_ctx *ctx, ib_herk *hk, double dt, const double *U) {
    if (!ctx || !hk || hk->ctx != ctx) return fail(LGFIB_EINVAL, "ib_herk_convection: bad context or step");
    if (!(dt >= 0.0) || !std::isfinite(dt)) return fail(LGFIB_EINVAL, "ib_herk_convection: dt must be finite and >= 0");
    if (U && !(std::isfinite(U[0]) && std::isfinite(U[1]) && std::isfinite(U[2])))
        return fail(LGFIB_EINVAL, "ib_herk_convection: non-finite frame velocity");
    hk->conv_dt = dt;
    for (int a = 0; a < 3; ++a) hk->U[a] = U ? U[a] : 0.0;
    return LGFIB_OK;
}

namespace lgfib {
// g <- g / gamma where gamma != 0, else 0
__global__ void k_div_guard(double *__restrict__ g, const double *__restrict__ gamma, size_t n) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) g[t] = gamma[t] != 0.0 ? g[t] / gamma[t] : 0.0;
}
__global__ void k_fill(double *__restrict__ y, double v, size_t n) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] = v;
}
}  // namespace lgfib

extern "C" int ib_force_smooth(lgfib_ctx *ctx, ib_system *sys, const double *f, double *fhat, lgfib_stream_t stream) {
    if (!ctx || !sys || sys->ctx != ctx) return fail(LGFIB_EINVAL, "ib_force_smooth: bad context or system");
    if (!f || !fhat) return fail(LGFIB_EINVAL, "ib_force_smooth: null vector");
    LGF_HIP(hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    const IbPlan &P = *sys->plan;
    const size_t nf = 3 * (size_t)sys->nblk * sys->B * sys->B * sys->B, nl = 3 * (size_t)sys->NL;
    int rc;
    if (!sys->gamma.p) {   // gamma = R 1
        if ((rc = sys->gamma.reserve(nf * 8))) return rc;
        double *ones = sys->tmp.as<double>();
        hipLaunchKernelGGL(k_fill, dim3(nblocks(nl, 256)), dim3(256), 0, st, ones, 1.0, nl);
        LGF_HIP(hipGetLastError());
        if ((rc = launch_regularize<double, double>(ctx, P, 1.0, ones, sys->gamma.as<double>(), st))) return rc;
    }
    double *g = sys->af[1].as<double>();
    if ((rc = launch_regularize<double, double>(ctx, P, 1.0, f, g, st))) return rc;
    hipLaunchKernelGGL(k_div_guard, dim3(nblocks(nf, 256)), dim3(256), 0, st, g, (const double *)sys->gamma.as<double>(),
                       nf);
    LGF_HIP(hipGetLastError());
    return launch_interpolate<double, double>(ctx, P, g, fhat, st);
}
