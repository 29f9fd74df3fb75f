"""GPU parity of the multilevel interpolation evaluator of u = dx^2 G * f
(Sec. 2.2, Eq. dpoisson_conv) through the C ABI.

- On a kernel that is an even polynomial of degree 2 per axis (< p) the
  evaluator is exact: the GPU result equals the brute-force sum, which pins
  the GPU's tree, interaction lists and interpolation weights.
- On G_L the GPU equals the oracle's evaluator (the same approximation) to
  FP64 rounding, <= 1e-12 of the largest value, on ragged sets that span
  several levels, for B = 4 (p = 4) and B = 8 (p = 4, 5, 6).
- At full size (the near-surface shell of a sphere of diameter 128 cells,
  1640 blocks of 8^3) against the exact sum on sampled cells, within the
  method's error the oracle shows on such sets.
"""
import numpy as np
import pytest

import oracle
import workloads
from oracle import fmm

torch = pytest.importorskip("torch")
import paper_1604_01814_amd as lg  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = lg.Context(0)
    yield c
    c.close()


def _rand_set(seed, n, region, shift=(0, 0, 0)):
    g = np.random.Generator(np.random.PCG64(seed))
    allb = np.array(list(np.ndindex(*region)), dtype=np.int32)[:, ::-1] - np.array([5, 2, 3], dtype=np.int32)
    return allb[np.sort(g.choice(len(allb), n, replace=False))] + np.asarray(shift, dtype=np.int32), g


def _poly_table(ext):
    z, y, x = np.meshgrid(*[np.arange(e + 1, dtype=np.float64) for e in ext[::-1]], indexing="ij")
    return 0.7 - 0.2 * x * x + 0.1 * y * y + 0.05 * z * z - 0.01 * x * x * z * z


def _gpu(ctx, tbl, B, p, src, f, tgt, dx=1.0, pair_prec=None):
    ml = lg.lgf_ml_create(ctx, tbl, B, p, src, tgt, pair_prec=pair_prec)
    f = f if f.ndim == 5 else f[None]
    fd = torch.from_numpy(np.ascontiguousarray(f)).cuda()
    u = torch.full((fd.shape[0], len(tgt), B, B, B), np.nan, dtype=torch.float64, device="cuda")
    ml.apply(fd, u, dx)
    torch.cuda.synchronize()
    info = ml.info()
    ml.close()
    return u.cpu().numpy(), info


@pytest.mark.parametrize("B,p", [(4, 4), (8, 4), (8, 5), (8, 6)])
def test_exact_for_an_even_polynomial_kernel(ctx, B, p):
    src, g = _rand_set(B + p, 40 if B == 4 else 16, (12, 7, 8))
    tgt, _ = _rand_set(B + p + 1, 30 if B == 4 else 12, (12, 7, 8), (2, 0, -1))
    ext = [int(v) for v in fmm.ml_table_extent(np.concatenate([src, tgt]), B)]
    tab = _poly_table(ext)
    tbl = lg.lgf_table_upload(ctx, tab)
    f = g.standard_normal((len(src), B, B, B))
    got, info = _gpu(ctx, tbl, B, p, src, f, tgt, dx=0.5)
    assert info["levels"] >= 2 and info["m2l_pairs"] > 0
    ref = fmm.direct_conv(fmm.even_table_kernel(tab), src, f, tgt, B, dx=0.5)
    assert np.max(np.abs(got[0] - ref)) < 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("B,p", [(4, 4), (8, 4), (8, 5), (8, 6)])
def test_matches_the_oracle_evaluator_on_g_l(ctx, B, p):
    src, g = _rand_set(30 + B + p, 36 if B == 4 else 14, (12, 7, 8))
    tgt = np.concatenate([src[::3], _rand_set(31 + B + p, 6, (12, 7, 8), (1, 1, 0))[0]])
    tgt = np.unique(tgt, axis=0)
    ext = [int(v) for v in fmm.ml_table_extent(np.concatenate([src, tgt]), B)]
    tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, ext)
    f = g.standard_normal((2, len(src), B, B, B))
    got, info = _gpu(ctx, tbl, B, p, src, f, tgt, dx=0.25)
    assert info["levels"] >= 2
    kern = fmm.even_table_kernel(oracle.lgf_table(*ext))
    for c in range(2):
        ref = fmm.ml_conv(kern, src, f[c], tgt, B, p, dx=0.25)
        assert np.max(np.abs(got[c] - ref)) < 1e-12 * np.max(np.abs(ref)), c


@pytest.mark.parametrize("src,tgt", [
    ([[0, 0, 0]], [[3, 0, 0]]),                          # no level above the blocks, one far pair
    ([[0, 0, 0], [1, 0, 0]], [[2, 0, 0], [-2, 1, 1]]),   # near and far targets, one level
    ([[0, 0, 0], [-9, 4, 2]], [[-9, 4, 2], [5, -3, 0]]),  # far apart: several levels, sparse
])
def test_small_and_far_apart_sets(ctx, src, tgt):
    B, p = 8, 4
    src, tgt = np.array(src, np.int32), np.array(tgt, np.int32)
    ext = [int(v) for v in fmm.ml_table_extent(np.concatenate([src, tgt]), B)]
    f = np.random.Generator(np.random.PCG64(len(src) + 7)).standard_normal((len(src), B, B, B))
    tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, ext)
    got, _ = _gpu(ctx, tbl, B, p, src, f, tgt)
    ref = fmm.ml_conv(fmm.even_table_kernel(oracle.lgf_table(*ext)), src, f, tgt, B, p)
    assert np.max(np.abs(got[0] - ref)) < 1e-12 * np.max(np.abs(ref))
    tp = lg.lgf_table_upload(ctx, _poly_table(ext))
    got, _ = _gpu(ctx, tp, B, p, src, f, tgt)
    ref = fmm.direct_conv(fmm.even_table_kernel(_poly_table(ext)), src, f, tgt, B)
    assert np.max(np.abs(got[0] - ref)) < 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("drop_src,drop_tgt", [(3, 50), (50, 3), (0, 0)])
def test_neighbour_products_over_several_pair_tiles(ctx, drop_src, drop_tgt):
    """Full neighbourhoods with more than 128 pairs for several displacements
    (tile remainders) and more sources than targets or fewer, on a kernel that
    differs by axis and that the evaluator represents exactly."""
    B, p = 8, 4
    box = np.array(list(np.ndindex(6, 5, 6)), dtype=np.int32)[:, ::-1] - np.array([2, 1, 4], dtype=np.int32)
    g = np.random.Generator(np.random.PCG64(90 + drop_src))
    src = box[np.sort(g.permutation(len(box))[drop_src:])]
    tgt = box[np.sort(g.permutation(len(box))[drop_tgt:])]
    ext = [int(v) for v in fmm.ml_table_extent(box, B)]
    tab = _poly_table(ext)
    tbl = lg.lgf_table_upload(ctx, tab)
    f = g.standard_normal((len(src), B, B, B))
    got, _ = _gpu(ctx, tbl, B, p, src, f, tgt)
    sel = g.permutation(len(tgt))[:6]
    ref = fmm.direct_conv(fmm.even_table_kernel(tab), src, f, tgt[sel], B)
    assert np.max(np.abs(got[0][sel] - ref)) < 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", [lg.LGF_F64, lg.LGF_F32])
def test_neighbours_of_an_infinite_cell(ctx, prec):
    """The neighbour sum of 8^3 blocks runs on sums and differences of a block's
    cells, the definition meets every cell on its own: with a kernel of positive
    values an infinity reaches each cell of its neighbours as that infinity, two
    of opposite sign as NaN, and cells whose sum alone overflows stay finite.  A
    second component without such cells is what it is without them (bars: FP64
    and FP32 products as above and below)."""
    B, p = 8, 4
    src = np.array(list(np.ndindex(7, 2, 2)), dtype=np.int32)
    ext = [int(v) for v in fmm.ml_table_extent(src, B)]
    tab = np.abs(oracle.lgf_table(*ext)) + 1e-3
    tbl = lg.lgf_table_upload(ctx, tab)
    g = np.random.Generator(np.random.PCG64(91))
    f = g.standard_normal((len(src), B, B, B))
    clean, _ = _gpu(ctx, tbl, B, p, src, f, src, pair_prec=prec)
    bar = 1e-12 if prec == lg.LGF_F64 else 2e-6
    near = src[:, 0] <= 1
    # 0.9 of the largest value of the products' type in a cell and in its mirror image
    top = 0.9 * (np.finfo(np.float64).max if prec == lg.LGF_F64 else float(np.finfo(np.float32).max))
    for cells, want in (([(3, 4, 5, np.inf)], np.inf), ([(0, 0, 0, -np.inf)], -np.inf),
                        ([(1, 1, 1, np.inf), (6, 2, 0, -np.inf)], np.nan), ([(2, 2, 2, np.nan)], np.nan)):
        h = f.copy()
        for z, y, x, v in cells:
            h[0, z, y, x] = v
        got, _ = _gpu(ctx, tbl, B, p, src, np.stack([h, f]), src, pair_prec=prec)
        assert np.max(np.abs(got[1] - clean[0])) < bar * np.max(np.abs(clean[0]))
        assert np.array_equal(got[0][near], np.full(got[0][near].shape, want), equal_nan=True), cells
    h = f.copy()
    h[0, 1, 2, 0] = h[0, 1, 2, 7] = top
    got, _ = _gpu(ctx, tbl, B, p, src, h, src, pair_prec=prec)
    ref = fmm.direct_conv(fmm.even_table_kernel(tab), src[:1], h[:1] / top, src[near], B)   # the others: 1e-38 of it
    assert np.max(np.abs(got[0][near] / top - ref)) < bar * np.max(np.abs(ref))


@pytest.mark.parametrize("p", [4, 5, 6])
def test_fp32_pair_products(ctx, p):
    """M2L and the neighbour sum as FP32 matrix products: within 2e-6 of the
    largest value from the oracle's FP64 evaluator (FP32 rounding of the
    matrices, charges and sources, FP32 sums)."""
    B = 8
    src, g = _rand_set(50 + p, 14, (12, 7, 8))
    tgt = np.unique(np.concatenate([src[::2], _rand_set(51 + p, 5, (12, 7, 8), (0, 1, 1))[0]]), axis=0)
    ext = [int(v) for v in fmm.ml_table_extent(np.concatenate([src, tgt]), B)]
    tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, ext)
    f = g.standard_normal((len(src), B, B, B))
    got, _ = _gpu(ctx, tbl, B, p, src, f, tgt, pair_prec=lg.LGF_F32)
    ref = fmm.ml_conv(fmm.even_table_kernel(oracle.lgf_table(*ext)), src, f, tgt, B, p)
    err = np.max(np.abs(got[0] - ref)) / np.max(np.abs(ref))
    assert 0.0 < err < 2e-6, err


def test_tree_counts_match_the_oracle(ctx):
    """Levels, clusters, node pairs and neighbour pairs of the GPU plan equal
    the oracle's counts (integers, exactly) on a ragged set and on the
    416-block shell of a sphere of diameter 64."""
    B = 8
    shell = workloads.shell_blocks(64.0, B)
    src, _ = _rand_set(70, 30, (12, 7, 8))
    tgt, _ = _rand_set(71, 25, (12, 7, 8), (3, -1, 2))
    for s_, t_ in ((src, tgt), (shell, shell)):
        ext = [int(v) for v in fmm.ml_table_extent(np.concatenate([s_, t_]), B)]
        tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, ext)
        ml = lg.lgf_ml_create(ctx, tbl, B, 4, s_, t_)
        info = ml.info()
        ml.close()
        want = fmm.ml_counts(s_, t_)
        assert {k: info[k] for k in want} == want


def test_argument_checks(ctx):
    B = 8
    blocks = workloads.cube_blocks(2)
    tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, (15, 15, 15))
    for Bb, p, code in ((16, 4, lg.LGFIB_EINVAL), (4, 5, lg.LGFIB_EINVAL), (8, 7, lg.LGFIB_EINVAL), (8, 3, lg.LGFIB_EINVAL)):
        with pytest.raises(lg.LgfibError) as e:
            lg.lgf_ml_create(ctx, tbl, Bb, p, blocks, blocks)
        assert e.value.code == code
    with pytest.raises(lg.LgfibError) as e:       # FP32 pair products need 8^3 blocks
        lg.lgf_ml_create(ctx, tbl, 4, 4, blocks, blocks, pair_prec=lg.LGF_F32)
    assert e.value.code == lg.LGFIB_EINVAL
    with pytest.raises(lg.LgfibError) as e:       # the top clusters reach past the table
        lg.lgf_ml_create(ctx, tbl, B, 4, blocks, np.array([[9, 0, 0]], np.int32))
    assert e.value.code == lg.LGFIB_ERANGE
    with pytest.raises(lg.LgfibError) as e:
        lg.lgf_ml_create(ctx, tbl, B, 4, np.concatenate([blocks, blocks[:1]]), blocks)
    assert e.value.code == lg.LGFIB_EDUP_BLOCK
    # no sources: zero; no targets: nothing to do
    got, _ = _gpu(ctx, tbl, B, 4, np.zeros((0, 3), np.int32), np.zeros((0, B, B, B)), blocks)
    assert np.all(got == 0.0)
    ml = lg.lgf_ml_create(ctx, tbl, B, 4, blocks, np.zeros((0, 3), np.int32))
    ml.apply(torch.zeros((1, 8, B, B, B), dtype=torch.float64, device="cuda"),
             torch.zeros((1, 0, B, B, B), dtype=torch.float64, device="cuda"))
    ml.close()
    # neighbours only: the leaf sum alone, exact
    f = np.random.Generator(np.random.PCG64(3)).standard_normal((8, B, B, B))
    got, info = _gpu(ctx, tbl, B, 4, blocks, f, blocks)
    assert info["m2l_pairs"] == 0
    cells = workloads.block_cells(blocks, B)
    ref = oracle.conv_direct(oracle.lgf_table(15, 15, 15), cells, f.reshape(-1), cells)
    assert np.max(np.abs(got.reshape(-1) - ref)) < 1e-12 * np.max(np.abs(ref))


def test_sphere_shell_full_size_against_the_exact_sum(ctx):
    """1640 blocks of 8^3 within one block of a sphere surface of diameter
    128 cells, sources = targets; sampled target cells against the exact
    direct sum.  Bars: 3e-4 (p = 4), 1e-4 (p = 5) and 1e-5 (p = 6) of the
    largest sampled value, the oracle's error bounds on sparse sets."""
    B = 8
    blocks = workloads.shell_blocks(128.0, B)
    assert len(blocks) == 1640
    f = workloads.normal_sources(len(blocks), B, config=6).reshape(len(blocks), B, B, B).astype(np.float64)
    ext = [int(v) for v in fmm.ml_table_extent(blocks, B)]
    tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, ext)
    g = np.random.Generator(np.random.PCG64(128))
    sample = np.sort(g.choice(len(blocks) * B ** 3, 48, replace=False))
    cells = workloads.block_cells(blocks, B)
    span = [int(v) for v in (blocks.max(0) - blocks.min(0) + 1) * B - 1]
    ref = oracle.conv_direct(oracle.lgf_table(*span), cells, f.reshape(-1), cells[sample])
    for p, tol in ((4, 3e-4), (5, 1e-4), (6, 1e-5)):
        got, info = _gpu(ctx, tbl, B, p, blocks, f, blocks)
        assert info["levels"] == 3
        err = np.max(np.abs(got.reshape(-1)[sample] - ref)) / np.max(np.abs(ref))
        assert err < tol, (p, err)


def test_largest_sphere_shell_against_the_exact_sum(ctx):
    """26,120 blocks of 8^3 around a sphere of diameter 512 cells, which the
    box-FFT path cannot take (span 576 cells after rounding): sampled target
    cells against the exact direct sum.  Bars from the errors the bench
    measures over every cell of the smaller shells: 6e-4 (p = 4, FP32 pair
    products) and 3e-5 (p = 6)."""
    B = 8
    blocks = workloads.shell_blocks(512.0, B)
    assert len(blocks) == 26120
    f = workloads.normal_sources(len(blocks), B, config=7).reshape(len(blocks), B, B, B).astype(np.float64)
    ext = [int(v) for v in fmm.ml_table_extent(blocks, B)]
    tbl = lg.lgf_table_build(ctx, lg.LGF_KIND_L, 0.0, ext)
    g = np.random.Generator(np.random.PCG64(512))
    sample = np.sort(g.choice(len(blocks) * B ** 3, 24, replace=False))
    cells = workloads.block_cells(blocks, B)
    span = [int(v) for v in (blocks.max(0) - blocks.min(0) + 1) * B - 1]
    print("oracle table", span, flush=True)
    ref = oracle.conv_direct(oracle.lgf_table(*span), cells, f.reshape(-1), cells[sample])
    for p, prec, tol in ((4, lg.LGF_F32, 6e-4), (6, lg.LGF_F64, 3e-5)):
        got, info = _gpu(ctx, tbl, B, p, blocks, f, blocks, pair_prec=prec)
        assert info["levels"] == 5
        err = np.max(np.abs(got.reshape(-1)[sample] - ref)) / np.max(np.abs(ref))
        print("p = %d: %.2e" % (p, err), flush=True)
        assert err < tol, (p, err)

