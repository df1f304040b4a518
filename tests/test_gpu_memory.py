"""Solves where memory is short: the sweep and two-pass forms fall back from
their ring of residuals to one or two buffers, so that what fits without the
ring is solved."""
import pytest

from oracle.contour import nodes
from tests.gpu_util import CIRCLE, gauge, make_ctx

pytestmark = pytest.mark.gpu
GB = 1 << 30


# 16^4, so that each of the source's vectors is 12.6 MB; the card is filled up to
# what the form needs without a ring plus 1.25 GB and two outputs.  A sweep or sum
# after every 1 or 2 iterations adds the same terms in another order: tolerances
# of the sign tests.
@pytest.mark.parametrize("form,precision,J,nsrc,variant,tol", [
    (0, 0, 4, 32, 0, 1e-11), (1, 0, 4, 32, 0, 1e-11), (0, 1, 4, 32, 0, 1e-10),
    (1, 1, 4, 32, 0, 1e-10), (1, 0, 65, 16, 0, 1e-11), (3, 0, 4, 32, 0, 1e-11),
    (3, 0, 4, 32, 17, 1e-11), (3, 1, 4, 32, 17, 1e-10)])
def test_solves_without_room_for_the_ring(form, precision, J, nsrc, variant, tol, monkeypatch):
    import torch
    monkeypatch.setenv("OVL_STENCIL_VARIANT", str(variant))
    dims = (16, 16, 16, 16)
    z, c = nodes(130, *CIRCLE)
    z, c = z[10:10 + J], c[10:10 + J]
    gen = torch.Generator(device="cuda").manual_seed(3)
    b = torch.view_as_complex(torch.randn((nsrc, 16, 16, 16, 16, 4, 3, 2), generator=gen,
                                          dtype=torch.float64, device="cuda"))
    vec = b.numel() * 16
    sweep = form != 3
    per_shift = (J if sweep else 0) + (J if form == 0 else 0)
    half = 0.5 * (1 if precision else 0)
    need = 4 + (1 if sweep else 2) + per_shift + half * ((1 if sweep else 2) + 1 + (J if sweep else 0))
    ring = need + (1 + half) * (15 if sweep else 6)
    leave = int((need + 2) * vec + 1.25 * GB)  # (two outputs)
    assert ring * vec > leave  # the ring does not fit
    out, st, taken = {}, {}, {}
    for short in (False, True):
        ctx = make_ctx(dims, gauge(dims, 0.3, 6), precision=precision, form=form, tol=1e-12,
                       maxiter=600, switch_res=1e-3)
        ctx.set_nodes(z, c)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        hog = None
        if short:
            free = torch.cuda.mem_get_info()[0]
            hog = torch.empty(free - leave, dtype=torch.uint8, device="cuda")
        before = torch.cuda.mem_get_info()[0]
        try:
            s, st[short] = ctx.apply_sign(b)
            taken[short] = before - torch.cuda.mem_get_info()[0]
            out[short] = s.clone()
        finally:
            s = hog = None  # (a traceback would keep it)
            torch.cuda.empty_cache()
            ctx.close()
    print(f"taken {taken[False] / vec:.1f} and {taken[True] / vec:.1f} vectors")
    assert taken[False] > (ring - 0.5) * vec and taken[True] < (need + 3) * vec
    assert st[True].iterations == st[False].iterations
    assert precision == 0 or st[True].fp32_iterations > 0
    err = float((out[True] - out[False]).abs().max() / out[False].abs().max())
    print(f"form {form} precision {precision}, {J} shifts: element-wise {err:.2e}")
    assert err < tol


# Many shifts: the ring is a tenth of the solve, and used as long as all of it
# fits, beyond half of what is free.
def test_many_shifts_keep_the_ring():
    import torch
    dims, J, nsrc = (16, 16, 16, 16), 130, 16
    z, c = nodes(130, *CIRCLE)
    b = torch.ones((nsrc, 16, 16, 16, 16, 4, 3), dtype=torch.complex128, device="cuda")
    vec = b.numel() * 16
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), form=1, tol=1e-10, maxiter=32)
    ctx.set_nodes(z[:J], c[:J])
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    leave = int((20 + J + 1 + 4) * vec + 1.5 * GB)
    free = torch.cuda.mem_get_info()[0]
    hog = torch.empty(free - leave, dtype=torch.uint8, device="cuda")
    before = torch.cuda.mem_get_info()[0]
    assert (20 + J) * vec > 0.5 * before
    try:
        ctx.apply_sign(b, allow_not_converged=True)
        taken = before - torch.cuda.mem_get_info()[0]
    finally:
        hog = None  # noqa: F841
        torch.cuda.empty_cache()
        ctx.close()
    print(f"taken {taken / vec:.1f} vectors")
    assert taken > (20 + J - 0.5) * vec


# A solve that cannot fit at all returns OVL_E_OOM, leaves no HIP error for the
# caller's next launch to find, and the context solves what fits afterwards.
@pytest.mark.parametrize("form", [0, 1])
def test_out_of_memory_leaves_nothing_behind(form):
    import torch
    from paper_2204_01583_amd import ovl
    dims = (16, 16, 16, 16)
    z, c = nodes(512, *CIRCLE)
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), form=form, tol=1e-10)
    ctx.set_nodes(z, c)  # 1024 shifts x 32 sources: 412 GB of directions
    b = torch.zeros((32, 16, 16, 16, 16, 4, 3), dtype=torch.complex128, device="cuda")
    with pytest.raises(ovl.OvlError) as e:
        ctx.apply_sign(b)
    assert e.value.status == ovl.E_OOM
    assert float(torch.ones(1000, device="cuda").mul(2).sum()) == 2000.0
    ctx.set_nodes(z[:2], c[:2])
    b[:1] = 1.0
    _, st = ctx.apply_sign(b[:1])
    assert st.n_active_end == 0
    ctx.close()


# The basis form's slots: a chunk of 32 slots that cannot be allocated is
# refused each time it is asked for, and a smaller solve on the same context
# runs.  Tensors and vectors of 700 sources take 62 GB, a chunk 282 GB.
def test_out_of_memory_in_the_basis_slots():
    import torch
    from paper_2204_01583_amd import ovl
    dims, nsrc = (16, 16, 16, 16), 700
    ctx = make_ctx(dims, gauge(dims, 0.3, 6), nq=4, form=2, tol=1e-10, maxiter=600)
    b = torch.zeros((nsrc, 16, 16, 16, 16, 4, 3), dtype=torch.complex128, device="cuda")
    b[0] = 1.0
    for _ in range(2):
        with pytest.raises(ovl.OvlError) as e:
            ctx.apply_sign(b)
        assert e.value.status == ovl.E_OOM
    s, st = ctx.apply_sign(b[:1])
    assert st.n_active_end == 0 and bool(torch.isfinite(torch.view_as_real(s)).all())
    ctx.close()
