"""The key sort orders leading bits, then short runs, then (long runs out of
order) everything: keys and permutation must be those of a stable sort by the
whole keys, bit for bit, at the sizes and runs where the parts meet."""
import numpy as np
import pytest

import oracle
from paper_1909_07439_amd import inputs, sph

from gpu_util import say

pytestmark = pytest.mark.gpu


def cells(rng, n, size, width):
    """n points in clumps of `size` within `width`, in random memory order."""
    c = rng.random(((n + size - 1) // size, 3)) * 0.9 + 0.05
    x = np.repeat(c, size, axis=0)[:n] + width * rng.random((n, 3))
    return x[rng.permutation(n)]


def positions(kind, n):
    rng = np.random.default_rng(n)
    if kind == "uniform":
        return rng.random((n, 3))
    if kind == "few":  # runs of three, some across tile edges
        return cells(rng, n, 3, 2e-6)
    if kind == "full":  # runs up to the longest that a block orders
        return cells(rng, n, 64, 1e-6)
    if kind == "over":  # runs just longer: all bits sorted
        return cells(rng, n, 65, 1e-6)
    if kind == "ball":  # one run holds nearly all
        x = 0.3 + 1e-4 * rng.random((n, 3))
        x[: n // 100 + 1] = rng.random((n // 100 + 1, 3))
        return x[rng.permutation(n)]
    if kind == "corner":  # a small part of the box: its top bits do not vary
        return 1e-3 * rng.random((n, 3))
    if kind == "equal":  # a long run of equal keys is in order already
        x = rng.random((n, 3))
        x[rng.permutation(n)[: n // 3]] = 0.7
        return x
    raise ValueError(kind)


@pytest.mark.parametrize("box", [(1.0, 1.0, 1.0), (1.0, 1e-3, 1e-2)], ids=["cube", "needle"])
@pytest.mark.parametrize("kind", ["uniform", "few", "full", "over", "ball", "corner", "equal"])
@pytest.mark.parametrize("n", [2, 130, 1024, 1025, 2048, 2049, 4096, 4097, 6200, 70001])
def test_sort_is_the_stable_sort_of_whole_keys(n, kind, box):
    say(f"[sort] {kind} n={n} box={box}")
    x = positions(kind, n) * np.asarray(box)
    cfg = dict(inputs.DEFAULTS, box_lo=(0, 0, 0), box_len=box, periodic=(1, 1, 1),
               x=x[:, 0].copy(), y=x[:, 1].copy(), z=x[:, 2].copy(), m=np.full(n, 1.0 / n),
               h=np.full(n, 1e-4), n=n, workload=f"{kind}{n}")
    ctx = sph.Context(sph.make_params(cfg), n)
    parts = sph.Particles(cfg)
    sph.sph_build_tree(ctx, parts)
    keys, perm = sph.sph_get_keys(ctx, n)
    ok = oracle.keys(cfg["x"], cfg["y"], cfg["z"], oracle.make_params(cfg))
    operm = oracle.sort(ok)
    np.testing.assert_array_equal(perm, operm)
    np.testing.assert_array_equal(keys, ok[operm])
    np.testing.assert_array_equal(parts.numpy("x")["x"], cfg["x"][operm])
    sph.sph_check(ctx)


@pytest.mark.parametrize("n", [1, 1024, 1025, 4096, 4097, 16384, 16385])
def test_permute_moves_every_field(n):
    rng = np.random.default_rng(n)
    cfg = dict(inputs.DEFAULTS, box_lo=(0, 0, 0), box_len=(1, 1, 1), periodic=(1, 1, 1), n=n,
               workload=f"permute{n}", **{k: rng.random(n) for k in ("x", "y", "z", "m", "u", "h",
                                                                     "vx", "vy", "vz")})
    ctx = sph.Context(sph.make_params(cfg), n)
    parts = sph.Particles(cfg)
    before = parts.numpy("x", "y", "z", "m", "u", "h", "vx", "vy", "vz")
    sph.sph_build_tree(ctx, parts)
    _, perm = sph.sph_get_keys(ctx, n)
    after = parts.numpy("id", *before)
    np.testing.assert_array_equal(after["id"], perm)
    for k, v in before.items():
        np.testing.assert_array_equal(after[k], v[perm], err_msg=k)
