"""Lattices beyond 32-bit byte offsets: H_W takes them, what runs on the tiled
stencils refuses them."""
import pytest

from oracle.gamma import gamma5, gammas

pytestmark = pytest.mark.gpu


def _field(site_shape):
    """SU(3) links diag(e^{ia}, e^{ib}, e^{-i(a+b)}), a and b random per link."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    U = torch.zeros((4,) + site_shape + (3, 3), dtype=torch.complex128, device="cuda")
    for mu in range(4):
        a = torch.randn(site_shape + (2,), generator=gen, dtype=torch.float64, device="cuda")
        U[mu, ..., 0, 0] = torch.polar(torch.ones_like(a[..., 0]), a[..., 0])
        U[mu, ..., 1, 1] = torch.polar(torch.ones_like(a[..., 0]), a[..., 1])
        U[mu, ..., 2, 2] = torch.polar(torch.ones_like(a[..., 0]), -a[..., 0] - a[..., 1])
    return U


def _hw_slice(diag, b, t, m0):
    """H_W b on time slice t, from the diagonals [mu] -> [Lt][Lz][Ly][Lx][3] of
    the links (antiperiodic in time)."""
    import torch
    kappa = 1.0 / (2.0 * (4.0 - m0))
    Lt = b.shape[0]
    g5 = torch.from_numpy(gamma5()).cuda()
    one = torch.eye(4, dtype=torch.complex128, device="cuda")

    def spin(M, x):
        return (M[:, :, None] * x[..., None, :, :]).sum(-2)

    acc = torch.zeros_like(b[t])
    for mu, gm in enumerate(torch.from_numpy(gammas()).cuda()):
        if mu < 3:
            dim = 2 - mu
            u = diag[mu][t][..., None, :]
            f = u * torch.roll(b[t], -1, dim)
            w = torch.roll(u.conj() * b[t], 1, dim)
        else:
            s, p = (-1.0 if t == Lt - 1 else 1.0), (-1.0 if t == 0 else 1.0)
            f = s * diag[3][t][..., None, :] * b[(t + 1) % Lt]
            w = p * diag[3][(t - 1) % Lt][..., None, :].conj() * b[(t - 1) % Lt]
        acc += spin(one - gm, f) + spin(one + gm, w)
    return spin(g5, b[t] - kappa * acc)


# 30.4 million sites: a source's vector and, in the full form, one direction's
# links pass 2^32 bytes.  Three FP64 roundings per term as on small lattices.
@pytest.mark.parametrize("links", ["two-row", "full"])
def test_hw_beyond_32_bit_offsets(links, monkeypatch):
    import torch
    from paper_2204_01583_amd import ovl
    for v in ("OVL_STENCIL_VARIANT", "OVL_LINKS"):
        monkeypatch.delenv(v, raising=False)
    if links == "full":
        monkeypatch.setenv("OVL_LINKS", "full")
    dims = (64, 64, 64, 116)
    site_shape = dims[::-1]
    U = _field(site_shape)
    ctx = ovl.Context(dims, bc=(1, 1, 1, -1), device=0)
    ctx.set_gauge(U)
    ctx.set_masses(1.4, 0.1)
    ctx.set_nodes([1 + 0.5j], [1.0])
    diag = [torch.stack([U[mu, ..., i, i] for i in range(3)], -1) for mu in range(4)]
    del U
    torch.cuda.empty_cache()
    gen = torch.Generator(device="cuda").manual_seed(6)
    b = torch.view_as_complex(torch.randn((1,) + site_shape + (4, 3, 2), generator=gen,
                                          dtype=torch.float64, device="cuda"))
    out = ctx.apply_hw(b)[0]
    out32 = ctx.apply_hw_fp32(b)[0] if links == "two-row" else None
    for t in (0, 1, 70, 85, 86, 114, 115):  # 2^32 bytes end in slice 85 of a vector
        ref = _hw_slice(diag, b[0], t, 1.4)
        assert float((out[t] - ref).abs().max() / ref.abs().max()) < 1e-14, t
        if out32 is not None:
            assert float((out32[t] - ref).abs().max() / ref.abs().max()) < 1e-6, t
    del out, out32

    def refused(f):
        with pytest.raises(ovl.OvlError) as e:
            f()
        assert e.value.status == ovl.E_ARG and "30408704 sites" in str(e.value)

    for form in range(4):
        ctx.set_solver(0, form)
        refused(lambda: ctx.apply_sign(b))
    refused(lambda: ctx.force(b))
    refused(lambda: ovl.apply_sign_batched([ctx], [b]) and None)
    refused(lambda: ctx.bench_kernel(0, 1, 1))
    monkeypatch.setenv("OVL_STENCIL_VARIANT", "0")
    refused(lambda: ctx.apply_hw(b))
    ctx.close()
