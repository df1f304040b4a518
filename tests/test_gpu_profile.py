"""Profiling hooks: every launch of a solve is in its class."""
import pytest

import seeded_inputs as si
from tests.gpu_util import gauge, make_ctx, to_dev

pytestmark = pytest.mark.gpu
DIMS = (6, 6, 4, 6)


@pytest.fixture(autouse=True)
def _two_kernels(monkeypatch):
    for v in ("OVL_STENCIL_VARIANT", "OVL_AUTOTUNE", "OVL_AUTOTUNE_CACHE"):
        monkeypatch.delenv(v, raising=False)
    monkeypatch.setenv("OVL_FUSED", "0")


# Profiling switched on before the first solve, whose tuning runs belong to no
# class: the classes hold the launches of the solve alone, one stencil and one
# update per iteration queued, and as many again in a second profiled solve.
@pytest.mark.parametrize("form", [1, 2])
def test_profiling_a_solve_that_tunes(form):
    ctx = make_ctx(DIMS, gauge(DIMS, 0.3, 6), nq=16, form=form)
    b = to_dev(si.gaussian_sources(DIMS, 2, first_seed=61))
    counts = []
    for _ in range(2):
        ctx.set_profiling(True)
        _, st = ctx.apply_sign(b)
        p = ctx.profile()
        ctx.set_profiling(False)
        chunks = -(-st.iterations // 16)
        assert p["stencil64"][1] == p["vector64"][1] == 16 * chunks
        assert p["sweep64"][1] == (chunks if form == 1 else 0)
        assert p["basis_sum"][1] == (1 if form == 2 else 0)
        assert p["iter64"] == p["iter32"] == p["stencil32"] == (0.0, 0, 0.0)
        assert all(ms >= 0.0 and nb >= 0.0 for ms, _, nb in p.values())
        counts.append({k: v[1] for k, v in p.items()})
    assert counts[0] == counts[1]
    ctx.close()


# The two-pass form's second pass: its additions to s, one per 8 iterations
# queued and precision, are the basis-sum class; with the replayed stencil
# (variant 17) no update runs in it, with the repeated one (0) as many as in the
# first pass.  Bytes: every residual of either source read once, s read and
# written per window.
@pytest.mark.parametrize("variant", [0, 17])
def test_two_pass_sum_is_profiled(variant, monkeypatch):
    monkeypatch.setenv("OVL_STENCIL_VARIANT", str(variant))
    ctx = make_ctx(DIMS, gauge(DIMS, 0.3, 6), nq=16, form=3)
    b = to_dev(si.gaussian_sources(DIMS, 1, first_seed=61))
    ctx.set_profiling(True)
    _, st = ctx.apply_sign(b)
    p = ctx.profile()
    ctx.set_profiling(False)
    its = 16 * -(-st.iterations // 16)
    assert p["stencil64"][1] == 2 * its
    assert p["vector64"][1] == (its if variant == 17 else 2 * its)
    assert p["basis_sum"][1] == its // 8 and p["basis_sum"][0] > 0.0
    n12 = 12 * 6 * 6 * 4 * 6
    assert p["basis_sum"][2] == n12 * (16 * st.iterations + 32 * -(-st.iterations // 8))
    ctx.close()
