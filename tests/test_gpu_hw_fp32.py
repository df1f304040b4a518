"""ovl_apply_hw_fp32 returns the same bits on every context: the tuner picks
among stencil variants that sum the hops in one order."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle.wilson import hermitian_wilson
from tests.gpu_util import assert_close, gauge, make_ctx, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _tuned(monkeypatch):
    for v in ("OVL_STENCIL_VARIANT", "OVL_AUTOTUNE", "OVL_AUTOTUNE_CACHE", "OVL_LINKS"):
        monkeypatch.delenv(v, raising=False)


# Both sides of every line of the size rule, with the variant whose bits the
# call returns (two-row links, then full ones).  The rule's groups: 0 one lane
# per site, 1 one lane with two hops per step, 8 two lanes, 9 both.
SIZES = [((4, 4, 2, 2), 2, None, 9), ((5, 4, 3, 3), 1, 9, 9), ((4, 4, 4, 4), 4, 8, 9),
         ((10, 6, 14, 9), 3, 8, 9), ((8, 8, 8, 8), 12, 8, 9), ((10, 6, 14, 9), 6, 9, 9),
         ((16, 16, 16, 16), 1, 8, 9), ((16, 16, 16, 12), 2, 1, 1), ((16, 16, 16, 12), 6, 1, 0),
         ((16, 16, 16, 16), 8, 0, 0)]


@pytest.mark.parametrize("links", ["two-row", "full"])
@pytest.mark.parametrize("dims,nrhs,two,full", SIZES)
def test_bits_do_not_depend_on_the_tuner(dims, nrhs, two, full, links, monkeypatch):
    import torch
    variant = two
    if links == "full":
        monkeypatch.setenv("OVL_LINKS", "full")
        variant = full
    gen = torch.Generator(device="cuda").manual_seed(7)
    U = gauge(dims, 0.3, 6)
    b = None
    got = []
    for _ in range(4):
        ctx = make_ctx(dims, U)
        if b is None:
            b = torch.view_as_complex(torch.randn((nrhs,) + ctx.site_shape + (4, 3, 2),
                                                  generator=gen, dtype=torch.float64, device="cuda"))
        got.append(ctx.apply_hw_fp32(b))
        assert torch.equal(got[-1], ctx.apply_hw_fp32(b))
        ctx.close()
    for g in got[1:]:
        assert torch.equal(g, got[0])
    if variant is None:  # at most one tile: the full links' sums
        monkeypatch.setenv("OVL_LINKS", "full")
        variant = full
    group = [v for v in range(24) if (v & 9) == variant and not (variant == 9 and v & 2)]
    for v in group:
        monkeypatch.setenv("OVL_STENCIL_VARIANT", str(v))
        ctx = make_ctx(dims, U)
        assert torch.equal(ctx.apply_hw_fp32(b), got[0]), f"variant {v}"
        ctx.close()


# A field that is not SU(3) loaded where an SU(3) field was: the stored third
# rows are read, not rebuilt; and back.
def test_field_kind_changes_on_one_context():
    dims = (6, 6, 4, 6)
    b = to_dev(si.gaussian_sources(dims, 2, first_seed=59))
    fields = [gauge(dims, 0.3, 6), 1.1 * gauge(dims, 0.3, 7), gauge(dims, 0.3, 8)]
    ctx = make_ctx(dims, fields[0], nq=16, form=2)
    ctx.set_residual_check(1)
    for U in fields:
        ctx.set_gauge(to_dev(U))
        H = hermitian_wilson(U, 1.4)
        ref = np.stack([(H @ v.ravel()).reshape(v.shape) for v in b.cpu().numpy()])
        assert_close(ctx.apply_hw_fp32(b).cpu().numpy(), ref, 2e-6, "FP32")
        # the residual check's operator is the solve's
        _, st = ctx.apply_sign(b)
        assert st.max_true_rel_res < 1e-11
    ctx.close()
