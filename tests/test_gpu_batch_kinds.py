"""Batches of contexts created under different OVL_FUSED settings: the batch
runs one iteration kind that all of them allow."""
import pytest

import seeded_inputs as si
from tests.gpu_util import assert_close, gauge, make_ctx, to_dev

pytestmark = pytest.mark.gpu
DIMS = [(4, 4, 4, 6), (3, 5, 4, 6)]


def _contexts(kinds, form, monkeypatch):
    out = []
    for i, k in enumerate(kinds):
        monkeypatch.setenv("OVL_FUSED", k)  # read when a context is created
        out.append(make_ctx(DIMS[i], gauge(DIMS[i], 0.3, 30 + i), nq=16, form=form))
    monkeypatch.setenv("OVL_FUSED", "")
    return out


@pytest.fixture(autouse=True)
def _env(monkeypatch):
    monkeypatch.delenv("OVL_STENCIL_VARIANT", raising=False)
    monkeypatch.setenv("OVL_AUTOTUNE", "0")


# OVL_FUSED=0 beside unset in every form, OVL_FUSED=1 (which only the basis
# forms heed) beside unset in the sweep forms: the stencil and update kernels.
# The batch equals single solves on contexts of that kind at the tolerance of the
# sign tests.
@pytest.mark.parametrize("kinds,form", [(("0", ""), 0), (("", "0"), 1), (("0", ""), 2),
                                        (("", "0"), 3), (("1", ""), 0), (("", "1"), 1)])
def test_unlike_contexts_in_one_batch(kinds, form, monkeypatch):
    from paper_2204_01583_amd import ovl
    ins = [to_dev(si.gaussian_sources(d, 2, first_seed=300 + i)) for i, d in enumerate(DIMS)]
    ctxs = _contexts(kinds, form, monkeypatch)
    outs, st = ovl.apply_sign_batched(ctxs, ins)
    assert st.stencil_variant64 < 1000
    refs = _contexts(("0", "0"), form, monkeypatch)
    for c, b, o in zip(refs, ins, outs):
        ref, _ = c.apply_sign(b)
        assert_close(o.cpu().numpy(), ref.cpu().numpy(), 1e-11, f"form {form} {kinds}")
    for c in ctxs + refs:
        c.close()


# The one-lane-per-site fused iteration beside another kind stays refused.
@pytest.mark.parametrize("kinds", [("1", ""), ("0", "1")])
@pytest.mark.parametrize("form", [2, 3])
def test_fused_beside_another_kind_is_refused(kinds, form, monkeypatch):
    from paper_2204_01583_amd import ovl
    ctxs = _contexts(kinds, form, monkeypatch)
    ins = [to_dev(si.gaussian_sources(d, 2)) for d in DIMS]
    with pytest.raises(ovl.OvlError) as e:
        ovl.apply_sign_batched(ctxs, ins)
    assert e.value.status == ovl.E_ARG
    for c in ctxs:
        c.close()
