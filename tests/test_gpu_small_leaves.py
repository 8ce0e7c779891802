"""Rows on trees with leaves of one or two particles, where a group reaches
more than 512 leaves: no group is left to the walking kernels, and the adjoint
takes the set (against the gradient oracle, with the bound of the other FP64
gradients: 1e-9 of each field's largest)."""
import numpy as np
import pytest

from oracle import adjoint as adj
from paper_1909_07439_amd import inputs, sph

from gpu_util import say

pytestmark = pytest.mark.gpu


def evaluate(cfg, precision, n_leaf):
    ctx = sph.Context(sph.make_params(cfg, precision, n_leaf=n_leaf), cfg["n"])
    parts = sph.Particles(cfg)
    sph.sph_build_tree(ctx, parts)
    sph.sph_density(ctx, parts)
    sph.sph_force(ctx, parts)
    sph.sph_check(ctx)
    return ctx, parts


@pytest.mark.parametrize("precision", [sph.SPH_PREC_FP64, sph.SPH_PREC_MIXED])
@pytest.mark.parametrize("n_leaf", [1, 2])
@pytest.mark.parametrize("side", [20, 24])
def test_rows_of_many_leaves(side, n_leaf, precision):
    say(f"[leaves] {side}^3 n_leaf={n_leaf} precision={precision}")
    cfg = inputs.with_kernel(inputs.lattice(side, jitter=0.2), "wc6")
    cfg["h"] = 0.99 * cfg["h"]
    ctx, parts = evaluate(cfg, precision, n_leaf)
    stats = sph.sph_stats(ctx)
    assert stats["groups_rows_overflow"] == 0, stats
    for mode in (0, 1):
        off, idx = sph.sph_list_pairs(ctx, parts, mode)
        woff, widx = sph.sph_neighbours(ctx, parts, mode)
        np.testing.assert_array_equal(off, woff)
        np.testing.assert_array_equal(idx, widx)
    ctx.close()


def test_adjoint_of_many_leaves():
    cfg = inputs.with_kernel(inputs.lattice(24, jitter=0.2, velocities=True), "wc6")
    rng = np.random.default_rng(24)
    up = {k: rng.normal(size=cfg["n"]) for k in ("ax", "ay", "az", "dudt")}
    want, _ = adj.eval_vjp(cfg, up)
    ctx, parts = evaluate(cfg, sph.SPH_PREC_FP64, 1)
    cot = sph.Cotangents(cfg["n"])
    for k, v in up.items():
        cot.t[k].copy_(sph.Particles({"x": v}).t["x"])
    sph.sph_eval_adjoint(ctx, parts, cot)
    sph.sph_check(ctx)
    ctx.close()
    for k in ("x", "y", "z", "vx", "vy", "vz", "u"):
        e = float(np.abs(cot.t[k].cpu().numpy() - want[k]).max() / np.abs(want[k]).max())
        say(f"  {k}: {e:.1e}")
        assert e <= 1e-9, (k, e)


@pytest.mark.parametrize("n_group", [4, 8])
@pytest.mark.parametrize("kernel", ["m6", "wc6"])
def test_lists_of_a_leaf_per_particle(kernel, n_group):
    """64^3 lattice sites: cells of 8 particles, so leaves of one up to n_leaf
    7 and of eight from 8 on; the leaf-list space is shared by all groups."""
    cfg = inputs.with_kernel(inputs.lattice(64, jitter=0.2), kernel)
    cfg["n_group"] = n_group
    pairs = set()
    for n_leaf in (1, 7, 8):
        say(f"[leaves] 64^3 {kernel} n_group={n_group} n_leaf={n_leaf}")
        ctx, _ = evaluate(cfg, sph.SPH_PREC_FP64, n_leaf)
        stats = sph.sph_stats(ctx)
        assert stats["groups_rows_overflow"] == 0, (n_leaf, stats)
        pairs.add((stats["density_pairs"], stats["force_pairs"]))
        ctx.close()
    assert len(pairs) == 1, pairs
