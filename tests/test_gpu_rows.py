"""Density from the neighbour-list rows at their ragged lengths: rows that end
anywhere within a block of entries, empty lanes, last chunks of one particle,
for each smoothing kernel, lanes per particle and precision, against the
oracle (FP64 1e-12; mixed 2e-6 in h, 1e-5 in rho and Omega: FP32 pair terms
of about 6e-8 each, a few ten per lane)."""
import numpy as np
import pytest

import oracle
from paper_1909_07439_amd import inputs, sph

from gpu_util import gpu_eval, rel_err, say

pytestmark = pytest.mark.gpu


def cloud(n, kernel, seed):
    """n particles of a jittered ball in an open box: every row length from
    the surface's to the centre's."""
    rng = np.random.default_rng(seed)
    s = int(np.ceil((6.0 * n / np.pi) ** (1.0 / 3.0))) + 2
    c = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij"), -1).reshape(-1, 3) - 0.5 * (s - 1)
    c = c[np.argsort((c ** 2).sum(1), kind="stable")[:n]]
    d = 0.5 / s
    pos = 0.5 + d * (c + rng.uniform(-0.3, 0.3, c.shape))
    cfg = inputs.lattice(4)
    cfg.update(n=n, periodic=(0, 0, 0), workload=f"cloud{n}", id=np.arange(n, dtype=np.int64),
               m=np.full(n, 1.0 / n), u=np.ones(n), h=np.full(n, cfg["hfact"] * d))
    for a, k in enumerate("xyz"):
        cfg[k] = np.ascontiguousarray(pos[:, a])
        cfg["v" + k] = np.zeros(n)
        cfg["a" + k] = np.zeros(n)
    cfg["dudt"] = np.zeros(n)
    return inputs.with_kernel(cfg, kernel)


@pytest.mark.parametrize("precision", [sph.SPH_PREC_FP64, sph.SPH_PREC_MIXED])
@pytest.mark.parametrize("n_group", [4, 8])
@pytest.mark.parametrize("kernel", ["m4", "m6", "wc6"])
@pytest.mark.parametrize("n", [9, 65, 1003])
def test_density_of_ragged_rows(n, kernel, n_group, precision):
    cfg = cloud(n, kernel, 7 + n)
    cfg["n_group"] = n_group
    o = oracle.evaluate(cfg, oracle.make_params(cfg))
    out, ctx, _, info = gpu_eval(cfg, precision)
    sph.sph_check(ctx)
    tol = dict(h=1e-12, rho=1e-12, omega=1e-12) if precision == sph.SPH_PREC_FP64 else \
        dict(h=2e-6, rho=1e-5, omega=1e-5)
    for k, t in tol.items():
        e = float(rel_err(out[k], o[k]).max())
        say(f"  {k}: {e:.2e}")
        assert e <= t, (k, e)


@pytest.mark.parametrize("kernel", ["m4", "wc6"])
@pytest.mark.parametrize("n", [9, 1003, 8191, 8192, 8193])
def test_force_of_ragged_rows_fp64(n, kernel):
    """Either side of the particle count up to which more lanes share a row;
    tolerance as of the density, relative to the pair terms' magnitudes."""
    cfg = cloud(n, kernel, 11 + n)
    rng = np.random.default_rng(n)
    for k in ("vx", "vy", "vz"):
        cfg[k] = rng.normal(0.0, 0.1, n)
    o = oracle.evaluate(cfg, oracle.make_params(cfg))
    out, ctx, _, info = gpu_eval(cfg)
    sph.sph_check(ctx)
    assert info["stats"]["force_pairs"] == int(o["nneigh_force"].sum())
    for k, nk in (("ax", "anorm"), ("ay", "anorm"), ("az", "anorm"), ("dudt", "unorm")):
        e = float((np.abs(out[k] - o[k]) / np.maximum(o[nk], 1e-300)).max())
        say(f"  {k}: {e:.2e}")
        assert e <= 1e-12, (k, e)


def blobs(n, seed, clump=0):
    """Two jittered blobs in opposite corners of an open box (the curve jumps
    between them), with `clump` particles of one at one point: coincident
    keys, so a level-21 leaf of that many particles."""
    cfg = cloud(n, "m4", seed)
    rng = np.random.default_rng(seed)
    for k in "xyz":
        x = 0.2 + 0.2 * (cfg[k] - 0.25)
        x[n // 2:] += 0.6
        cfg[k] = np.ascontiguousarray(x)
    cfg["h"] = 0.2 * cfg["h"]
    if clump:
        at = rng.integers(0, n // 2)
        for k in "xyz":
            cfg[k][:clump] = cfg[k][at]
    return cfg


@pytest.mark.parametrize("precision", [sph.SPH_PREC_FP64, sph.SPH_PREC_MIXED])
@pytest.mark.parametrize("n_group", [4, 8])
@pytest.mark.parametrize("n,clump", [(1, 0), (8, 0), (70, 0), (1500, 0), (1500, 65), (1500, 110)])
def test_rows_hold_the_walks_sets(n, clump, n_group, precision):
    """The pairs the rows give are the exact sets of the group walk: one group,
    several wavefronts per group, units cut at a jump of the curve, and leaves
    of more than 64 coincident particles (clump 110: more than a row holds with
    its other neighbours, so flagged groups)."""
    cfg = blobs(n, 3 + n, clump)
    cfg["n_group"] = n_group
    say(f"[rows] n={n} clump={clump} n_group={n_group} precision={precision}")
    parts = sph.Particles(cfg)
    ctx = sph.Context(sph.make_params(cfg, precision, h_tol=-1.0), n)
    sph.sph_build_tree(ctx, parts)
    sph.sph_density(ctx, parts)
    sph.sph_check(ctx)
    for mode in (0, 1):
        off, idx = sph.sph_list_pairs(ctx, parts, mode)
        woff, widx = sph.sph_neighbours(ctx, parts, mode)
        np.testing.assert_array_equal(off, woff)
        np.testing.assert_array_equal(idx, widx)
    ctx.close()


@pytest.mark.parametrize("precision", [sph.SPH_PREC_FP64, sph.SPH_PREC_MIXED])
def test_outgrown_rows_give_the_same_bits_again(precision):
    """Groups whose h outgrows their rows: which wavefront flags one first must
    not show in the results or in the counts."""
    cfg = inputs.lattice(40, jitter=0.3)
    cfg["h"] = cfg["h"] * np.random.default_rng(3).uniform(0.85, 1.1, cfg["n"])
    seen = []
    for _ in range(2):
        parts = sph.Particles(cfg)
        ctx = sph.Context(sph.make_params(cfg, precision), cfg["n"])
        sph.sph_build_tree(ctx, parts)
        sph.sph_density(ctx, parts)
        sph.sph_force(ctx, parts)
        stats = sph.sph_stats(ctx)
        assert stats["groups_h_outgrew"] > 100
        seen.append((parts.numpy("h", "rho", "ax", "dudt"), stats))
    for k, v in seen[0][0].items():
        np.testing.assert_array_equal(v, seen[1][0][k], err_msg=k)
    for k in ("groups_h_outgrew", "density_pairs", "density_pair_sums", "density_candidates"):
        assert seen[0][1][k] == seen[1][1][k], k
