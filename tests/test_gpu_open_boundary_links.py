"""Links across a Dirichlet boundary belong to no hop: whatever finite numbers they hold, also numbers beyond the range
of FP32 and BF16 storage, the result is the one with unit matrices in their place, bit for bit."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

# launch shapes; None is the library's own choice
SHAPES = [None, dict(rhs_per_thread=2, block=128), dict(rhs_per_thread=1, wshare=4), dict(rhs_per_thread=2, wshare=2),
          dict(rhs_per_thread=1, block=256, site_order=2)]


def _links(L, bc, su3, unused):
    """Random links with `unused` in place of the links across the Dirichlet boundaries."""
    U = synth.su3_links(L, 0.4, 29)
    if not su3:
        U = U * np.exp(1j * np.random.default_rng(3).uniform(-1, 1, (4, synth.volume(L), 1, 1)))
    U = np.ascontiguousarray(U).reshape((4, L[3], L[2], L[1], L[0], 3, 3))
    for mu in range(4):
        if bc[mu] == 2:
            at = [mu, slice(None), slice(None), slice(None), slice(None)]
            at[4 - mu] = L[mu] - 1
            U[tuple(at)] = unused
    return torch.from_numpy(U.reshape(4, -1, 3, 3)).cuda()


@pytest.mark.parametrize("su3", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("L,bc,n", [((3, 4, 5, 6), (2, 1, 2, 2), 1), ((3, 4, 5, 6), (2, 0, 2, 2), 3),
                                    ((4, 4, 8, 16), (2, 2, 0, 2), 240), ((8, 8, 8, 16), (2, 0, 2, 1), 60)])
def test_links_across_open_boundaries_are_not_read_into_the_result(L, bc, n, prec, su3):
    from paper_1111_6288_amd import ov
    f = [j % 2 for j in range(n)]
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((n, synth.volume(L), 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    for shape in SHAPES:
        y = []
        for unused in (np.eye(3), np.diag([1e300, 1.0, 1e300])):   # both satisfy u_2 = conj(u_0 x u_1)
            ctx = ov.Context(L, bc, -1.5)
            ctx.upload_gauge(_links(L, bc, su3, unused))
            assert ctx.link_format()[0] is su3
            ctx.set_fields((2 / 3, -1 / 3), (0.2, -0.4))
            if shape:
                ctx.set_launch_config(prec, "dslash", **shape)
            y += [ctx.dslash(x, f, op=op, prec=prec) for op in ("HW", "DW")]
            ctx.close()
        assert torch.isfinite(torch.view_as_real(y[0])).all()
        assert torch.equal(y[0], y[2]) and torch.equal(y[1], y[3]), shape
