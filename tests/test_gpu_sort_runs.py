"""Runs of equal leading key bits longer than a block orders by rank: sorted by
a block each up to 4096 keys, by passes over everything beyond; keys and
permutation are those of a stable sort by the whole keys, bit for bit.  And
what such sets cost."""
import numpy as np
import pytest

import oracle
from paper_1909_07439_amd import inputs, sph

from gpu_util import say

pytestmark = pytest.mark.gpu


def config(x, name):
    n = x.shape[0]
    return dict(inputs.DEFAULTS, box_lo=(0, 0, 0), box_len=(1, 1, 1), periodic=(0, 0, 0),
                x=x[:, 0].copy(), y=x[:, 1].copy(), z=x[:, 2].copy(), m=np.full(n, 1.0 / n),
                h=np.full(n, 1e-4), n=n, workload=f"{name}{n}")


def clumps(sizes, n, seed, width, equal=0):
    """Clumps of the given sizes among uniform particles, n in all, in random
    memory order; `equal` particles of each clump at one point."""
    rng = np.random.default_rng(seed)
    x = rng.random((n, 3))
    at = 0
    for size in sizes:
        # within one cell of level 12: one run for every pass count up to four
        corner = rng.integers(0, 4096, 3) / 4096.0
        x[at:at + size] = corner + (0.3 + width * rng.random((size, 3))) / 4096.0
        x[at:at + equal] = x[at]
        at += size
    return x[rng.permutation(n)]


@pytest.mark.parametrize("sizes,n,equal", [
    ((64, 65, 66), 5000, 0), ((255, 256, 257, 1023, 1024, 1025), 9000, 100),
    ((4095, 4096), 30000, 0), ((4096, 300), 30000, 300), ((4097, 65), 30000, 0),
    ((4096,) * 9 + (65,) * 200, 70001, 0), ((3000,), 3001, 0), ((2048, 2048), 4097, 65),
    ((20000, 5000, 65), 300001, 4500), ((4100,) * 260, 1080000, 0)])
@pytest.mark.parametrize("width", [0.4, 1e-4])
def test_long_runs_are_sorted_by_whole_keys(sizes, n, equal, width):
    say(f"[runs] {sizes[:6]} n={n} equal={equal} width={width}")
    cfg = config(clumps(sizes, n, len(sizes) + n, width, equal), "runs")
    ctx = sph.Context(sph.make_params(cfg), n)
    parts = sph.Particles(cfg)
    sph.sph_build_tree(ctx, parts)
    sph.sph_check(ctx)
    keys, perm = sph.sph_get_keys(ctx, n)
    ok = oracle.keys(cfg["x"], cfg["y"], cfg["z"], oracle.make_params(cfg))
    operm = oracle.sort(ok)
    np.testing.assert_array_equal(perm, operm)
    np.testing.assert_array_equal(keys, ok[operm])
    # again from the sorted order: every run is in order
    sph.sph_build_tree(ctx, parts)
    keys, perm = sph.sph_get_keys(ctx, n)
    np.testing.assert_array_equal(perm, np.arange(n))
    np.testing.assert_array_equal(keys, ok[operm])
    ctx.close()


def plummer(n, a):
    rng = np.random.default_rng(n)
    r = a / np.sqrt((0.98 * rng.random(n)) ** (-2.0 / 3.0) - 1.0)
    v = rng.normal(size=(n, 3))
    v /= np.linalg.norm(v, axis=1)[:, None]
    return np.clip(0.5 + r[:, None] * v, 0.001, 0.999)


@pytest.mark.parametrize("n,a", [(60000, 0.003), (400000, 0.003), (1000000, 0.001)])
def test_runs_of_every_length_next_to_each_other(n, a):
    """A cluster's centre: runs for one block, for several and for the rank,
    with shared cache lines, sorted in the same launches."""
    say(f"[runs] cluster n={n} a={a}")
    cfg = config(plummer(n, a), "cluster")
    ok = oracle.keys(cfg["x"], cfg["y"], cfg["z"], oracle.make_params(cfg))
    operm = oracle.sort(ok)
    ctx = sph.Context(sph.make_params(cfg), n)
    for _ in range(3):
        sph.sph_build_tree(ctx, sph.Particles(cfg))
        sph.sph_check(ctx)
        keys, perm = sph.sph_get_keys(ctx, n)
        np.testing.assert_array_equal(perm, operm)
        np.testing.assert_array_equal(keys, ok[operm])
    ctx.close()


def sort_time(x, name):
    """Median over a few builds (a delay of the host must not count)."""
    cfg = config(x, name)
    ctx = sph.Context(sph.make_params(cfg), cfg["n"])
    sets = [sph.Particles(cfg) for _ in range(17)]
    times = []
    for p in sets:
        sph.sph_build_tree(ctx, p)
        times.append(sph.sph_timings(ctx)["keys_sort"])
    ctx.close()
    return float(np.median(times[2:]))


def test_a_dense_cluster_costs_no_more_than_all_passes():
    """30,000 particles: a uniform set takes three passes, a preparation and
    the run kernels; all eight passes over it would take 1.7 times as long
    (80 us, measured, against 47).  A cluster whose density spans six orders
    of magnitude, and a body that fills 1e-8 of its box, take no longer than
    that."""
    rng = np.random.default_rng(1)
    flat = sort_time(rng.random((30000, 3)), "uniform")
    for name, x in (("cluster", plummer(30000, 0.01)),
                    ("body", 0.5 + 1e-3 * (2.0 * rng.random((30000, 3)) - 1.0))):
        t = sort_time(x, name)
        say(f"[sort time] {name}: {1e3 * t:.1f} us, uniform {1e3 * flat:.1f} us")
        assert t <= 1.7 * flat, (name, t, flat)
