"""The direction-wave H_w kernel (one wave per direction, taken by small batches whose launch shape nobody chose)
against the FP64 oracle: site counts around its 64-site blocks and around the 64 blocks from which the XCDs take
contiguous runs, every boundary condition, both link formats, both operators, the fused epilogue and the largest
batch of the rule."""
import numpy as np
import pytest
import torch

import synth
from oracle import api

pytestmark = pytest.mark.gpu
MW = -1.5


def _ctx(L, bc, U, q, eta):
    from paper_1111_6288_amd import ov
    ctx = ov.Context(L, bc, MW)
    ctx.upload_gauge(torch.from_numpy(U).cuda())
    ctx.set_fields(q, eta)
    return ctx


def _rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


SHAPES = [((2, 2, 2, 2), (2, 2, 2, 2)), ((3, 3, 7, 3), (0, 1, 2, 0)), ((4, 4, 2, 2), (0, 0, 0, 1)),
          ((5, 13, 2, 7), (2, 0, 1, 2)), ((9, 13, 5, 7), (1, 2, 0, 2)), ((8, 8, 8, 8), (2, 0, 0, 2)),
          ((17, 3, 9, 9), (0, 0, 2, 1))]


@pytest.mark.parametrize("L,bc", SHAPES)
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-14), ("fp32", 2e-6), ("bf16", 2e-2)])
def test_dirwaves_match_oracle(L, bc, prec, tol):
    q, eta, n = (2 / 3, -1 / 3), (0.2, -0.4), 3
    rng = np.random.default_rng(11)
    f = [0, 1, 1]
    x = synth.gaussian_spinors(L, n, 8)
    su3 = synth.su3_links(L, 0.5, 41)
    for U in (su3, su3 * np.exp(1j * rng.uniform(-1, 1, (4, synth.volume(L), 1, 1)))):
        ctx = _ctx(L, bc, U, q, eta)
        assert ctx.link_format()[0] is (U is su3)
        for op, k in (("HW", 1), ("DW", 0)):
            y = ctx.dslash(torch.from_numpy(x).cuda(), f, op=op, prec=prec).cpu().numpy()
            for j in range(n):
                ref = api.dslash(api.Lattice(L, bc, MW, U, q[f[j]] * eta[f[j]]), x[j], k)
                assert _rel(y[j], ref) < tol, (op, j)
        ctx.close()


@pytest.mark.parametrize("L,bc,nrhs", [((3, 3, 7, 3), (0, 1, 2, 0), 1), ((4, 4, 4, 4), (0, 0, 0, 1), 37),
                                       ((8, 8, 8, 8), (2, 0, 0, 2), 9), ((9, 13, 5, 7), (1, 2, 0, 2), 4)])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5), ("bf16", 6e-2)])
def test_dirwaves_epilogue_against_site_kernel(L, bc, nrhs, prec, tol):
    """The fused Clenshaw step: D(m) through the direction waves and through a chosen site-parallel shape."""
    U = synth.su3_links(L, 0.3, 5)
    ctx = _ctx(L, bc, U, (2 / 3, 2 / 3), (1e-3, -1e-3))
    ctx.set_sign_params(12, 0.02, 6.5)
    x = torch.from_numpy(synth.gaussian_spinors(L, nrhs, 3)).cuda()
    f, m = [j % 2 for j in range(nrhs)], [0.05 * (j % 3) for j in range(nrhs)]
    y = ctx.dov_apply(x, f, m, prec=prec)
    for kind in ("dslash", "clenshaw"):
        ctx.set_launch_config(prec, kind, rhs_per_thread=1, block=128)
    z = ctx.dov_apply(x, f, m, prec=prec)
    assert float((y - z).abs().max() / z.abs().max()) < tol
    ctx.close()


def test_dirichlet_neighbours_are_not_read_into_the_result():
    """An infinity beyond a Dirichlet boundary stays where it is: hops across it are dropped, not multiplied by 0."""
    L, bc = (6, 4, 4, 6), (2, 0, 0, 2)
    U = synth.su3_links(L, 0.3, 5)
    ctx = _ctx(L, bc, U, (2 / 3,), (0.1,))
    x = synth.gaussian_spinors(L, 1, 3)
    x[0, 0] = np.inf   # site (0, 0, 0, 0): x and t wrap to sites that must not see it
    y = ctx.dslash(torch.from_numpy(x).cuda(), [0], prec="fp64").cpu().numpy()
    bad = {int(s) for s in np.nonzero(~np.isfinite(y[0]).all(axis=(1, 2)))[0]}
    lx, ly, lz, _ = L
    want = {0, 1, lx, lx * (ly - 1), lx * ly, lx * ly * (lz - 1), lx * ly * lz}   # itself, +x, +-y, +-z, +t
    assert bad == want
    ctx.close()


@pytest.mark.parametrize("L,bc", [((16, 16, 16, 32), (2, 0, 0, 2)), ((15, 14, 13, 34), (0, 1, 2, 0))])
def test_unchosen_launches_give_the_bits_of_a_chosen_shape(L, bc):
    """Batches around every boundary of the launch rule, against two right-hand sides per thread: the same bits."""
    U = synth.su3_links(L, 0.3, 5)
    ctx = _ctx(L, bc, U, (2 / 3, -1 / 3), (1e-3, -1e-3))
    V = synth.volume(L)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn((13, V, 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    cases = [(p, n, True) for p, ns in (("fp64", (1, 3, 4, 5, 9)), ("fp32", (1, 4, 7, 8, 9, 13)),
                                        ("bf16", (1, 2, 3, 5, 9, 13))) for n in ns] + [("fp64", 5, False), ("fp32", 9, False)]
    got = {}
    for prec, n, rec in cases:
        ctx.set_link_reconstruct(rec)
        got[prec, n, rec] = ctx.dslash(x[:n].contiguous(), [j % 2 for j in range(n)], prec=prec)
    for prec in ("fp64", "fp32", "bf16"):
        ctx.set_launch_config(prec, "dslash", rhs_per_thread=2, block=128)
    for prec, n, rec in cases:
        ctx.set_link_reconstruct(rec)
        ref = ctx.dslash(x[:n].contiguous(), [j % 2 for j in range(n)], prec=prec)
        assert torch.equal(got[prec, n, rec], ref), (prec, n, rec)
    ctx.close()


@pytest.mark.parametrize("su3", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_shared_links_under_capture(su3, prec):
    """Link-sharing launches first met inside a graph capture (nine-entry FP64 links stage more than 64 KiB of LDS):
    replays between eager work equal the eager result, and a chosen site-parallel shape, bit for bit."""
    L, n = (8, 8, 8, 16), 60
    U = synth.su3_links(L, 0.3, 17)
    if not su3:
        U = U * np.exp(1j * np.random.default_rng(2).uniform(-1, 1, (4, synth.volume(L), 1, 1)))
    ctx = _ctx(L, (2, 0, 0, 2), U, (2 / 3, 2 / 3), (1e-3, -1e-3))
    assert ctx.link_format()[0] is su3
    ctx.set_sign_params(6, 0.02, 6.5)
    x = torch.from_numpy(synth.gaussian_spinors(L, n, 3)).cuda()
    f = [j % 2 for j in range(n)]
    ctx.set_graphs(1)
    got = []
    for _ in range(3):
        got.append(ctx.dov_apply(x, f, mass=[0.1] * n, prec=prec).clone())
        ctx.dslash(x, f, prec=prec)
        torch.cuda.synchronize()
    ctx.set_graphs(0)
    eager = ctx.dov_apply(x, f, mass=[0.1] * n, prec=prec).clone()
    for kind in ("dslash", "clenshaw"):
        ctx.set_launch_config(prec, kind, rhs_per_thread=2, block=128)
    site = ctx.dov_apply(x, f, mass=[0.1] * n, prec=prec)
    for g in got:
        assert torch.equal(g, eager)
    assert torch.equal(eager, site)
    ctx.close()
