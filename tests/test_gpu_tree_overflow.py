"""A tree that does not fit the node arrays (close pairs, one particle per
leaf: a chain of some 17 cells for every pair) is reported, and the passes on
it read no row: the first density, force, export and adjoint of a context come
without rows of an earlier tree to fall back on."""
import numpy as np
import pytest

from paper_1909_07439_amd import inputs, sph

from gpu_util import say

pytestmark = pytest.mark.gpu


def close_pairs(n):
    cfg = inputs.lattice(4)
    rng = np.random.default_rng(n)
    at = 0.1 + 0.8 * rng.random((n // 2, 3))
    x = np.concatenate([at, at + 1e-6])
    cfg.update(n=n, workload=f"pairs{n}", id=np.arange(n), m=np.full(n, 1.0 / n), u=np.ones(n),
               h=np.full(n, 1.2 * n ** (-1.0 / 3.0)), dudt=np.zeros(n))
    for a, k in enumerate("xyz"):
        cfg[k] = np.ascontiguousarray(x[:, a])
        cfg["v" + k] = np.zeros(n)
        cfg["a" + k] = np.zeros(n)
    return cfg


@pytest.mark.parametrize("precision", [sph.SPH_PREC_FP64, sph.SPH_PREC_MIXED])
@pytest.mark.parametrize("n", [2000, 20000])
def test_passes_on_a_tree_that_does_not_fit(n, precision):
    say(f"[overflow] n={n} precision={precision}")
    cfg = close_pairs(n)
    ctx = sph.Context(sph.make_params(cfg, precision, n_leaf=1), n)
    parts = sph.Particles(cfg)
    sph.sph_build_tree(ctx, parts)
    with pytest.raises(sph.SphError) as e:
        sph.sph_check(ctx)
    assert e.value.status == sph.SPH_E_OVERFLOW
    assert sph.sph_stats(ctx)["n_groups"] == 0
    h = parts.numpy("h")["h"]
    sph.sph_density(ctx, parts)
    sph.sph_force(ctx, parts)
    for call in (lambda: sph.sph_list_pairs(ctx, parts, 0),
                 lambda: sph.sph_eval_adjoint(ctx, parts, sph.Cotangents(n))):
        with pytest.raises(sph.SphError) as e:
            call()
        assert e.value.status == sph.SPH_E_OVERFLOW
    sph.sph_check(ctx)
    np.testing.assert_array_equal(parts.numpy("h")["h"], h)
    with pytest.raises(sph.SphError) as e:
        sph.sph_step(ctx, parts, 1e-9, want_dt=True)
    assert e.value.status == sph.SPH_E_OVERFLOW
    # the context then takes a set whose tree fits
    good = inputs.lattice(12, jitter=0.1, velocities=True)
    out = []
    for c in (ctx, sph.Context(sph.make_params(good, precision, n_leaf=1), n)):
        p = sph.Particles(good)
        sph.sph_build_tree(c, p)
        sph.sph_density(c, p)
        sph.sph_force(c, p)
        sph.sph_check(c)
        out.append(p.numpy("h", "rho", "ax", "dudt"))
        c.close()
    for k, v in out[0].items():
        np.testing.assert_array_equal(v, out[1][k], err_msg=k)
