"""Phase timings after more calls than a phase keeps."""
import pytest

from paper_1909_07439_amd import inputs, sph

pytestmark = pytest.mark.gpu


def test_full_phases_leave_room_for_the_others():
    """1024 launches per phase are kept; phases that first run after that
    still are."""
    cfg = inputs.lattice(6, jitter=0.1, velocities=True)
    parts = sph.Particles(cfg)
    ctx = sph.Context(sph.make_params(cfg), cfg["n"])
    sph.sph_build_tree(ctx, parts)
    sph.sph_density(ctx, parts)
    sph.sph_force(ctx, parts)
    for _ in range(1500):
        sph.sph_step(ctx, parts, 1e-6)
    cot = sph.Cotangents(cfg["n"])
    cot.t["x"].fill_(1.0)
    for _ in range(2):
        sph.sph_step_adjoint(ctx, parts, 1e-6, cot)
    sph.sph_check(ctx)
    t = sph.sph_timings(ctx)
    for k, v in t.items():
        assert v > 0.0, k
    assert t["adjoint"] >= t["adjoint_force"]
    assert t["step"] >= t["lists"] + t["density"] + t["force"]
    ctx.close()
