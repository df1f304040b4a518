"""The stencil and update kernels, which every larger solve runs, on lattices
small enough for the oracle: tests of the solver repeated with OVL_FUSED=0 and
each solve's stats saying that this iteration ran."""
import inspect
import itertools

import pytest

from tests import test_gpu_batch as batch
from tests import test_gpu_force as force
from tests import test_gpu_kernel_edges as edges
from tests import test_gpu_parity as parity
from tests.gpu_util import gauge, make_ctx, to_dev
from tests.test_gpu_parity import eig_4x4  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu

SOLVES = [parity.test_sign_4x4_fp64_all_forms, parity.test_sign_4x4_mixed,
          parity.test_dov_4x4_multi_rhs, parity.test_sign_8x8, parity.test_deterministic,
          parity.test_true_residual_single_node, parity.test_true_residual_contour,
          parity.test_single_contour_against_oracle,
          parity.test_spectral_bounds_and_suggested_contour,
          parity.test_sign_ragged_lattice_below_one_tile,
          parity.test_sign_partial_layout_tile_two_sources,
          parity.test_inband_residual_check_matches_synchronous_check,
          parity.test_mixed_repeats_in_fp64_when_the_check_fails,
          parity.test_maximum_shift_counts_against_the_oracle,
          batch.test_graph_replay_equals_eager, batch.test_lookahead_equals_chunk_by_chunk,
          batch.test_twopass_equals_basis, batch.test_batched_uneven_lattices,
          batch.test_batched_single_contour_matches_single_solves,
          batch.test_batch_jobs_finishing_at_very_different_times,
          edges.test_sweep_shift_counts, edges.test_sweep_ends_inside_a_chunk,
          force.test_force_partial_tile_and_boundaries, force.test_force_mixed_matches_fp64]


def _cases():
    """(test, arguments) for every parametrisation of SOLVES, and again with
    stencil variant 17 where the two-pass form runs (its second pass then
    replays the stencil; variant 0 repeats stencil and update)."""
    out = []
    for fn in SOLVES:
        marks = [m.args for m in getattr(fn, "pytestmark", []) if m.name == "parametrize"]
        axes = []
        for names, values in marks:
            names = [n.strip() for n in names.split(",")]
            axes.append([dict(zip(names, v if len(names) > 1 else (v,))) for v in values])
        for combo in itertools.product(*axes):
            kw = {k: v for d in combo for k, v in d.items()}
            two_pass = kw.get("form") == 3 or fn in (batch.test_twopass_equals_basis,
                                                     parity.test_sign_partial_layout_tile_two_sources)
            for variant in ("", "17") if two_pass else ("",):
                name = "-".join([fn.__name__[5:]] + [f"{k}{v}".replace(" ", "") for k, v in kw.items()]
                                + (["v17"] if variant else []))
                out.append(pytest.param(fn, kw, variant, id=name))
    return out


@pytest.fixture
def two_kernels(monkeypatch):
    """Contexts that keep the stencil and update kernels, untuned; returns the
    stencil choices of the solves made."""
    from paper_2204_01583_amd import ovl
    for v in ("OVL_STENCIL_VARIANT", "OVL_AUTOTUNE_CACHE", "OVL_LINKS"):
        monkeypatch.delenv(v, raising=False)
    monkeypatch.setenv("OVL_FUSED", "0")
    monkeypatch.setenv("OVL_AUTOTUNE", "0")
    seen = []

    def noting(fn):
        def call(*a, **kw):
            r = fn(*a, **kw)
            if r[-1].n_shifts:
                seen.append(r[-1].stencil_variant64)
            return r
        return call

    for name in ("apply_sign", "apply_dov", "force"):
        monkeypatch.setattr(ovl.Context, name, noting(getattr(ovl.Context, name)))
    monkeypatch.setattr(ovl, "apply_sign_batched", noting(ovl.apply_sign_batched))
    return seen


@pytest.mark.timeout(900)
@pytest.mark.parametrize("fn,kw,variant", _cases())
def test_solver_on_two_kernels(fn, kw, variant, two_kernels, monkeypatch, request):
    if variant:
        monkeypatch.setenv("OVL_STENCIL_VARIANT", variant)
    kw = dict(kw)
    for p in inspect.signature(fn).parameters:
        if p not in kw:
            kw[p] = request.getfixturevalue(p)
    fn(**kw)
    assert two_kernels and all(v < 1000 for v in two_kernels)
    if variant:
        assert all(v % 28 == int(variant) for v in two_kernels)


# The two-pass form regenerates its residuals bit for bit: the second pass that
# replays the recorded scalars (variants 16 and 17) and the one that repeats
# stencil and update (0 and 1) add the same residuals to the sum, each pair of
# variants summing the hops alike.
@pytest.mark.parametrize("links", ["two-row", "full"])
@pytest.mark.parametrize("repeat,replay", [(0, 16), (1, 17)])
@pytest.mark.parametrize("precision,dims,nsrc", [(0, (6, 6, 4, 6), 3), (1, (6, 6, 4, 6), 3),
                                                 (0, (3, 5, 2, 3), 2), (1, (12, 8, 8, 10), 2)])
def test_replayed_residuals_are_the_repeated_ones(repeat, replay, links, precision, dims, nsrc,
                                                  two_kernels, monkeypatch):
    import seeded_inputs as si
    if links == "full":
        monkeypatch.setenv("OVL_LINKS", "full")
    b = to_dev(si.gaussian_sources(dims, nsrc, first_seed=61))
    out = []
    for v in (repeat, replay):
        monkeypatch.setenv("OVL_STENCIL_VARIANT", str(v))
        ctx = make_ctx(dims, gauge(dims, 0.3, 6), nq=16, precision=precision, form=3, tol=1e-12,
                       switch_res=1e-3)
        s, st = ctx.apply_sign(b)
        assert precision == 0 or st.fp32_iterations > 0
        out.append(s)
        ctx.close()
    assert bool((out[0] == out[1]).all())
