"""Shifted solutions rebuilt a few at a time: the vector kernel (at most 4 shifts,
lattices from 32768 sites) against the matrix form."""
import pytest

import seeded_inputs as si
from tests.gpu_util import gauge, make_ctx, to_dev

pytestmark = pytest.mark.gpu


# Chunks on both sides of its shift limit and lattices on both sides of its size
# limit (28672 and 32768 sites), against all 12 shifts at once: the same solves
# and slots, the sums over some 200 slots and the shifts in another order.
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dims", [(16, 16, 16, 7), (16, 16, 16, 8)])
def test_few_shifts_at_a_time(dims, precision, monkeypatch):
    monkeypatch.setenv("OVL_FUSED", "0")
    monkeypatch.setenv("OVL_AUTOTUNE", "0")
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), 1.4, 0.1, 6, precision=precision,
                   form=2, tol=1e-12, switch_res=1e-4)
    phi = to_dev(si.gaussian_sources(dims, 1, first_seed=31))
    ref, S, st = ctx.force(phi, kind=1)
    assert precision == 0 or st.fp32_iterations > 0
    for chunk in (1, 2, 3, 4, 5):
        G, _, _ = ctx.force(phi, kind=1, shift_chunk=chunk)
        err = float((G - ref).abs().max() / ref.abs().max())
        assert err < 1e-12, (chunk, err)
    ctx.close()
