"""Kernels at the sizes where their tiling can go wrong: edges of tiles,
remainders, the smallest and largest of a range."""
import functools

import pytest

import seeded_inputs as si
from oracle.contour import nodes
from oracle.force import force as oracle_force
from tests.gpu_util import CIRCLE, assert_close, gauge, make_ctx, to_dev

pytestmark = pytest.mark.gpu


def setup_module(module):
    from paper_2204_01583_amd import ovl
    ovl.load()


@functools.lru_cache(maxsize=None)
def _force_reference(dims, nq):
    phi = si.gaussian_sources(dims, 1, first_seed=31)[0]
    z, c = nodes(nq, *CIRCLE)
    return oracle_force(gauge(dims, 0.3, 6), phi, 1.4, 0.1, z, c, method="dense")


# Rebuilt shifted solutions: 68 shifts in chunks on both sides of the 16-, 32-
# and 64-shift tiles.  Tolerances: the shifted solutions carry the solver's
# 1e-13 and, mixed, the FP32 drift of about 1e-7 x the switch point 1e-4.  The
# one-kernel iteration switches one slot earlier, so a step of four slots
# holds FP64 and FP32 ones.
@pytest.mark.parametrize("precision,fused,tol", [(0, "0", 1e-10), (1, "0", 1e-8), (1, "1", 1e-8)])
@pytest.mark.parametrize("chunk", [1, 15, 16, 17, 32, 33, 64, 65, 0])
def test_rebuilt_solutions_at_tile_edges(precision, fused, tol, chunk, monkeypatch):
    monkeypatch.setenv("OVL_FUSED", fused)
    dims, nq = (2, 2, 4, 4), 34
    G_ref, _, S_ref = _force_reference(dims, nq)
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), 1.4, 0.1, nq, precision=precision, form=2,
                   tol=1e-13 if precision == 0 else 1e-12)
    phi = to_dev(si.gaussian_sources(dims, 1, first_seed=31))
    G, S, st = ctx.force(phi, kind=1, shift_chunk=chunk)
    assert precision == 0 or st.fp32_iterations > 0
    assert abs(S - S_ref) / S_ref < (1e-11 if precision == 0 else 1e-8)
    assert_close(G.cpu().numpy(), G_ref, tol, f"G p{precision} fused {fused} chunk {chunk}")
    ctx.close()
