"""Kernels at the sizes where their tiling can go wrong: edges of tiles,
remainders, the smallest and largest of a range."""
import functools

import numpy as np
import pytest

import seeded_inputs as si
from oracle.contour import nodes
from oracle.force import force as oracle_force
from oracle.wilson import hermitian_wilson
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


@functools.lru_cache(maxsize=None)
def _dense(dims):
    return hermitian_wilson(gauge(dims, 0.3, 6), 1.4).toarray()


# The shift sweep: shift counts around a block's four waves, the 64 lanes of
# one and the 256 of a block, padding sites (90 sites), two sources, both sweep
# forms, FP64 and mixed; tolerances of the sign tests at these precisions.
@pytest.mark.parametrize("precision,tol", [(0, 1e-11), (1, 1e-10)])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 5, 64, 65, 257])
def test_sweep_shift_counts(form, n, precision, tol):
    dims = (3, 5, 2, 3)
    z, c = nodes(258, *CIRCLE)
    z, c = z[::2][:n], c[::2][:n]
    b = si.gaussian_sources(dims, 2, first_seed=41)
    H = _dense(dims)
    lam, Q = np.linalg.eigh(H)
    f = (c[:, None] / (z[:, None] - lam[None, :])).sum(0)
    ref = np.stack([Q @ (f * (Q.conj().T @ v.ravel())) for v in b]).reshape(b.shape)
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), precision=precision, form=form, tol=1e-12)
    ctx.set_nodes(z, c)
    s, st = ctx.apply_sign(to_dev(b))
    assert_close(s.cpu().numpy(), ref, tol, f"form {form}, {n} shifts, {st.iterations} iterations")
    ctx.close()


# Iteration limits that end inside a sweep: the last iterate equals the stored
# basis form's, which sums the same iterations in another order.
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("maxiter", [1, 15, 16, 17, 31])
def test_sweep_ends_inside_a_chunk(form, maxiter):
    dims = (3, 5, 2, 3)
    b = to_dev(si.gaussian_sources(dims, 2, first_seed=43))
    out = {}
    for fm in (form, 2):
        ctx = make_ctx(dims, gauge(dims, 0.3, 6), nq=16, form=fm, tol=1e-12, maxiter=maxiter)
        s, st = ctx.apply_sign(b, allow_not_converged=True)
        assert st.iterations == maxiter and st.n_active_end > 0
        out[fm] = s.cpu().numpy()
        ctx.close()
    assert_close(out[form], out[2], 1e-12, f"form {form}, {maxiter} iterations")


# The split iteration: lattices below, at and above one 64-site tile, shift
# counts around its 256-shift slices, both link formats, both basis forms.
@pytest.mark.parametrize("precision,tol", [(0, 1e-11), (1, 1e-10)])
@pytest.mark.parametrize("form,links", [(2, "two-row"), (2, "full"), (3, "two-row")])
@pytest.mark.parametrize("dims,n,nsrc", [((2, 2, 2, 2), 2, 1), ((4, 4, 2, 2), 256, 2),
                                         ((3, 5, 2, 3), 258, 3), ((5, 3, 3, 4), 600, 1)])
def test_split_iteration(dims, n, nsrc, form, links, precision, tol, monkeypatch):
    if links == "full":
        monkeypatch.setenv("OVL_LINKS", "full")
    z, c = nodes(600, *CIRCLE)
    z, c = z[::2][:n], c[::2][:n]
    b = si.gaussian_sources(dims, nsrc, first_seed=47)
    lam, Q = np.linalg.eigh(_dense(dims))
    f = (c[:, None] / (z[:, None] - lam[None, :])).sum(0)
    ref = np.stack([Q @ (f * (Q.conj().T @ v.ravel())) for v in b]).reshape(b.shape)
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), precision=precision, form=form, tol=1e-12)
    ctx.set_nodes(z, c)
    s, st = ctx.apply_sign(to_dev(b))
    assert st.stencil_variant64 == 2000 + (links == "two-row")
    assert_close(s.cpu().numpy(), ref, tol, f"{dims} x {nsrc}, form {form}, {n} shifts")
    ctx.close()


# Both sides of the split iteration's size limit: the same result from either
# iteration.
@pytest.mark.parametrize("precision,tol", [(0, 1e-11), (1, 1e-10)])
@pytest.mark.parametrize("dims,nsrc,split", [((16, 16, 8, 18), 1, True), ((16, 17, 8, 17), 1, False),
                                             ((8, 8, 8, 12), 6, True), ((8, 8, 8, 12), 7, False)])
def test_split_iteration_limit(dims, nsrc, split, precision, tol, monkeypatch):
    b = to_dev(si.gaussian_sources(dims, nsrc, first_seed=53))
    out = []
    for fused in ("", "0"):
        monkeypatch.setenv("OVL_FUSED", fused)
        monkeypatch.setenv("OVL_AUTOTUNE", "0")
        ctx = make_ctx(dims, gauge(dims, 0.3, 6), nq=16, precision=precision, form=2, tol=1e-12)
        s, st = ctx.apply_sign(b)
        assert (st.stencil_variant64 >= 2000) == (split and fused == "")
        out.append(s.cpu().numpy())
        ctx.close()
    assert_close(out[0], out[1], tol, f"{dims} x {nsrc}")


# H_W on the caller's layout: lattices below, at and beyond one 64-site block,
# every boundary sign, both link formats; against the oracle's matrix, at the
# tolerances of the operator tests.
@pytest.mark.parametrize("links", ["two-row", "full"])
@pytest.mark.parametrize("dims,nrhs,bc", [((2, 2, 2, 2), 1, (1, 1, 1, -1)),
                                          ((4, 4, 2, 2), 2, (-1, 1, -1, 1)),
                                          ((3, 5, 2, 3), 3, (1, -1, 1, -1)),
                                          ((6, 6, 4, 6), 5, (1, 1, 1, -1))])
def test_hw_direct_edges(dims, nrhs, bc, links, monkeypatch):
    if links == "full":
        monkeypatch.setenv("OVL_LINKS", "full")
    U = gauge(dims, 0.3, 6)
    H = hermitian_wilson(U, 1.4, bc=bc)
    b = si.gaussian_sources(dims, nrhs, first_seed=59)
    ref = np.stack([(H @ v.ravel()).reshape(v.shape) for v in b])
    ctx = make_ctx(dims, U, bc=bc)
    assert_close(ctx.apply_hw(to_dev(b)).cpu().numpy(), ref, 1e-14, f"{dims} FP64 {links}")
    ctx.close()


# Both sides of its rule for the block order (192 MiB of vectors), against the
# tiled stencil.
@pytest.mark.parametrize("dims,nrhs", [((16, 16, 16, 16), 16), ((16, 16, 16, 17), 16)])
def test_hw_direct_matches_the_tiled_stencil(dims, nrhs, monkeypatch):
    import torch
    ctx = make_ctx(dims, gauge(dims, 0.3, 6))
    b = torch.randn((nrhs,) + ctx.site_shape + (4, 3), dtype=torch.complex128, device="cuda")
    got = ctx.apply_hw(b)
    monkeypatch.setenv("OVL_STENCIL_VARIANT", "0")
    ref = ctx.apply_hw(b)
    assert float((got - ref).abs().max() / ref.abs().max()) < 1e-14
    ctx.close()


# The two-pass form's replayed second pass (LDS-tile variants 16 and 17) and the
# repeated one (variant 0): the same s as the stored basis form, whose sum runs
# over the same residuals in the same order, so a residual that differed in its
# last bit would show.  Mixed, the slot converted at the switch is added from
# its FP64 value, eps32 x 1e-3 of it away.  Padding sites, several sources,
# iteration limits inside a stretch of 8.
@pytest.mark.parametrize("links", ["two-row", "full"])
@pytest.mark.parametrize("variant", [0, 16, 17])
@pytest.mark.parametrize("precision,maxiter,tol", [(0, 4000, 1e-14), (0, 13, 1e-14), (1, 4000, 1e-12)])
def test_two_pass_replay(variant, links, precision, maxiter, tol, monkeypatch):
    monkeypatch.setenv("OVL_STENCIL_VARIANT", str(variant))
    if links == "full":
        monkeypatch.setenv("OVL_LINKS", "full")
    dims, nsrc = (6, 6, 4, 6), 3
    b = to_dev(si.gaussian_sources(dims, nsrc, first_seed=61))
    out = []
    for form in (2, 3):
        ctx = make_ctx(dims, gauge(dims, 0.3, 6), nq=16, precision=precision, form=form, tol=1e-12,
                       maxiter=maxiter, switch_res=1e-3)
        for _ in range(2):  # the second solve replays the captured graphs
            s, st = ctx.apply_sign(b, allow_not_converged=True)
        assert precision == 0 or st.fp32_iterations > 0
        out.append(s.cpu().numpy())
        ctx.close()
    assert_close(out[1], out[0], tol, f"variant {variant} {links} precision {precision}")
