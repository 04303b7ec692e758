"""The tiled gather's ways through a tile, against the direct gather and the oracle.

How many lanes share a particle follows from the particles of a work item, and
whether a block slides or is copied anew from the tiles that follow each other, so
the clouds here give every count around those limits: a few to more than one
round of a workgroup in each tile, one crowded tile (several chunks of 2048 and
several items), a column of tiles along axis 0, and tiles cut by the grid's end.
Every variant performs the same arithmetic, so tiled and direct agree to the last
bit; the oracle's bound is the one of the other gather tests.
"""
import numpy as np
import pytest

from gpu_common import log, dev, host, rel_err, TOL_F64, TOL_F32

pytestmark = pytest.mark.gpu


def _cloud(n, seed):
    """Particles per 8^3 tile from 1 to 300, 5000 in one tile, and a column along axis 0."""
    rng = np.random.default_rng(seed)
    h = 2 * np.pi / np.array(n)
    tiles = [(i, j, k) for i in range(-(-n[0] // 8)) for j in range(-(-n[1] // 8)) for k in range(-(-n[2] // 8))]
    counts = (1, 8, 10, 11, 16, 17, 20, 21, 22, 32, 33, 42, 43, 64, 65, 84, 85, 128, 129, 256, 257, 300)
    out = []
    for q, t in enumerate(tiles):
        lo = np.array(t) * 8 * h
        hi = np.minimum(np.array(t) * 8 + 8, n) * h
        c = 5000 if q == len(tiles) // 2 else counts[q % len(counts)]
        out.append(lo + (hi - lo) * rng.random((c, 3)))
    column = rng.random((500, 3)) * np.array([2 * np.pi, 4 * h[1], 4 * h[2]])
    pos = np.concatenate(out + [column])
    return pos[rng.permutation(len(pos))]


@pytest.mark.parametrize("n,C,N,coef", [
    ((36, 24, 48), 3, 6, "f32"), ((36, 24, 48), 1, 6, "f32"), ((18, 36, 24), 3, 4, "f32"),
    ((36, 24, 48), 3, 6, "bf16"), ((24, 36, 16), 1, 4, "bf16"),
    ((36, 24, 16), 3, 6, "f64"), ((18, 12, 24), 1, 4, "f64"), ((12, 12, 12), 3, 6, "f32")])
def test_tile_populations(n, C, N, coef):
    import paper_1201_4060_amd as bsi
    from oracle import evaluate
    log(f"paths n={n} C={C} N={N} coef={coef}")
    dt = {"f64": bsi.BSI_F64, "f32": bsi.BSI_F32, "bf16": bsi.BSI_BF16}[coef]
    pos = _cloud(n, seed=sum(n) + N)
    grid = np.random.default_rng(5).standard_normal((C,) + n)
    with bsi.Context(0) as ctx, bsi.Field(ctx, n, C, N, dt) as f:
        f.set_coefficients(dev(grid))
        want_u, want_g = evaluate(host(f.get_coefficients()).astype(np.float64), pos, N)
        ref = None
        for cfg in ((0, 0), (8, 0), (8, 256), (4, 0), (8, 0)):   # the direct gather first; twice the same plan
            c = bsi.EvalConfig(sort_tile=cfg[0], block=256, xcd_remap=1, variant=0 if cfg[0] else 1,
                               tile_block=cfg[1])
            u, g = (host(t) for t in f.eval(dev(pos), cfg=c))
            if ref is None:
                ref = u, g
                tol = TOL_F64 if coef == "f64" else TOL_F32
                assert np.max(rel_err(u, want_u)) < tol and np.max(rel_err(g, want_g)) < tol
            assert np.array_equal(u, ref[0]) and np.array_equal(g, ref[1]), cfg


@pytest.mark.parametrize("n,C,N,coef,basis", [
    (48, 3, 6, "f32", "bspline"), (48, 1, 6, "bf16", "bspline"), (36, 3, 6, "bf16", "bspline"),
    (24, 3, 4, "f64", "lagrange"), (64, 3, 6, "f64", "bspline"), (32, 3, 4, "f32", "hermite"),
    (16, 1, 2, "f32", "lagrange")])
def test_direct_lanes(n, C, N, coef, basis):
    """Evaluations without a configuration (the choice by particle count) and direct ones on one
    or several lanes per particle: counts around a wavefront's 10 or 16 particles, around the
    choices' limits, particles at the last cells of the grid and without a cell, value alone."""
    import paper_1201_4060_amd as bsi
    log(f"direct n={n} C={C} N={N} coef={coef} {basis}")
    dt = {"f64": bsi.BSI_F64, "f32": bsi.BSI_F32, "bf16": bsi.BSI_BF16}[coef]
    kw = {"bspline": {}, "lagrange": dict(basis=bsi.BSI_BASIS_LAGRANGE, prefilter=bsi.BSI_PREFILTER_NONE),
          "hermite": dict(basis=bsi.BSI_BASIS_HERMITE, prefilter=bsi.BSI_PREFILTER_NONE)}[basis]
    rng = np.random.default_rng(n + N)
    gn = 2 * n if basis == "hermite" else n
    grid = rng.standard_normal((C, gn, gn, gn))
    last = 2 * np.pi * (1 - np.array([1e-9, 0.3 / n, 0.9 / n]))
    with bsi.Context(0) as ctx, bsi.Field(ctx, n, C, N, dt, **kw) as f:
        f.set_coefficients(dev(grid))
        for P in (1, 9, 10, 11, 15, 16, 17, 64, 1003, 24577, 32767, 32768, 49152, 49153, 70001):
            pos = rng.uniform(0, 2 * np.pi, (P, 3))
            pos[:: 7] = last
            if P > 20:
                pos[5] = np.nan
                pos[P - 1, 1] = np.inf
            d = dev(pos)
            ref = None
            for c in (bsi.EvalConfig(sort_tile=8, block=256, xcd_remap=1, variant=0), None,
                      bsi.EvalConfig(sort_tile=0, block=256, xcd_remap=0, variant=1),
                      bsi.EvalConfig(sort_tile=8, block=256, xcd_remap=1, variant=1)):
                u, g = (host(t) for t in f.eval(d, cfg=c))
                v = host(f.eval(d, grad=False, cfg=c)[0])
                ref = (u, g) if ref is None else ref
                assert np.array_equal(u, ref[0], equal_nan=True) and np.array_equal(g, ref[1], equal_nan=True), (P, c)
                assert np.array_equal(v, ref[0], equal_nan=True), (P, c)


@pytest.mark.parametrize("coef", ["f32", "f64"])
def test_crowded_key_ranges(coef):
    # 10^6 particles over 32^3 tiles: key ranges of 32 tiles, some with about 1024, 2048, 4096, 8192
    # and 40000 particles (the sizes where the binning sorts a range another way)
    import torch
    import paper_1201_4060_amd as bsi
    n, N = 256, 4
    rng = np.random.default_rng(17)
    # a brick of 4^3 tiles is two ranges: corners of bricks far apart
    out = [rng.random((700000, 3)) * 2 * np.pi]
    for q, c in enumerate((300, 1300, 1400, 3300, 3400, 7400, 7500, 15900, 40000, 90000)):
        lo = np.array([q % 4, q // 4, q % 3]) * 2 * np.pi / 4
        out.append(lo + rng.random((c, 3)) * np.array([32, 32, 16]) * 2 * np.pi / n)
    pos = np.concatenate(out + [np.full((5000, 3), np.nan)])
    pos = np.concatenate([pos, rng.random((1000000 - len(pos), 3)) * 2 * np.pi])
    pos = dev(pos[rng.permutation(len(pos))])
    grid = dev(rng.standard_normal((1, n, n, n)))
    with bsi.Context(0) as ctx, bsi.Field(ctx, n, 1, N, bsi.BSI_F32 if coef == "f32" else bsi.BSI_F64) as f:
        f.set_coefficients(grid)
        want = f.eval(pos, cfg=bsi.EvalConfig(sort_tile=0, block=256, xcd_remap=1, variant=1))
        for rounds in (0, 1):
            got = f.eval(pos, cfg=bsi.EvalConfig(sort_tile=8, block=256, xcd_remap=1, variant=0, item_rounds=rounds))
            for a, b in zip(got, want):
                assert torch.equal(torch.nan_to_num(a, nan=7e7), torch.nan_to_num(b, nan=7e7))
        assert f.nonfinite_count() == 3 * 5000
