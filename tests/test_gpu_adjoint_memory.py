"""The two memory paths of the sign adjoint: H_w b_k of a replayed segment kept, or applied again.  Both against the
oracle, bit for bit against each other, and the workspace that each takes."""
import numpy as np
import pytest
import torch

import synth
from oracle import api

pytestmark = pytest.mark.gpu
MW, Q, ETA, N, EPS, NORM = -1.5, 2 / 3, 0.05, 24, 0.03, 6.5


def _rel(a, b):
    return np.abs(a - b).max() / np.abs(b).max()


def _backward(L, bc, U, V, lam, x, g, K, nbytes, want_links=True):
    """(gU, geta, gx, device bytes the call added)."""
    from paper_1111_6288_amd import ov
    ctx = ov.Context(L, bc, MW)
    ctx.upload_gauge(torch.from_numpy(U).cuda())
    ctx.set_fields((Q,), (ETA,))
    ctx.set_sign_params(N, EPS, NORM)
    if V is not None:
        ctx.upload_eigvecs(0, torch.from_numpy(V).cuda(), lam)
    if nbytes is not None:
        ctx.set_adjoint_memory(nbytes)
    before = ctx.memory_used()
    out = ctx.sign_backward(0, torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda(), ckpt_every=K,
                            want_U=want_links, want_eta=want_links)
    used = ctx.memory_used() - before
    ctx.close()
    return (*out, used)


@pytest.mark.parametrize("K", [1, 5, 64])
@pytest.mark.parametrize("L,bc,l", [((4, 4, 2, 6), (2, 0, 0, 2), 3), ((4, 4, 4, 4), (0, 0, 0, 1), 0)])
def test_both_memory_paths_match_the_oracle(L, bc, l, K):
    U = synth.su3_links(L, 0.4, 41)
    V = synth.random_orthonormal(L, l, 2) if l else None
    lam = np.linspace(-1, 1, l) if l else None
    x, g = synth.gaussian_spinors(L, 2, 13)
    fields = min(K, N) * 192 * ((synth.volume(L) + 63) // 64 * 64)   # bytes of the kept H_w b_k
    kept = _backward(L, bc, U, V, lam, x, g, K, fields)
    again = _backward(L, bc, U, V, lam, x, g, K, fields - 1)
    assert kept[3] == again[3] + fields
    assert torch.equal(kept[0], again[0]) and kept[1] == again[1] and torch.equal(kept[2], again[2])
    sp = api.SignParams(N, EPS, NORM, V, lam)
    rU, re, rx = api.sign_backward(api.Lattice(L, bc, MW, U, Q * ETA), sp, Q, x, g)
    assert _rel(again[0].cpu().numpy(), rU) < 1e-12
    assert abs(again[1] - re) <= 1e-12 * max(abs(re), 1e-12 * np.abs(rU).max())
    assert _rel(again[2].cpu().numpy(), rx) < 1e-12
    # nothing is kept for the gradient of x alone, which has no sweep
    assert _backward(L, bc, U, V, lam, x, g, K, fields, want_links=False)[3] == again[3]


def test_workspace_stays_bounded_by_default():
    """400 products of 25 MB exceed the default of 8 GiB: the workspace holds the vectors alone."""
    from paper_1111_6288_amd import ov
    L, n = (16, 16, 16, 32), 400
    ctx = ov.Context(L, (2, 0, 0, 2), MW)
    ctx.upload_gauge(torch.eye(3, dtype=torch.complex128, device="cuda").expand(4, synth.volume(L), 3, 3).contiguous())
    ctx.set_fields((Q,), (ETA,))
    ctx.set_sign_params(n, 0.5 / n ** 2, 8.5)
    field = 192 * synth.volume(L)
    assert n * field > 8 << 30
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, g = torch.randn((2, synth.volume(L), 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    before = ctx.memory_used()
    ctx.sign_backward(0, x, g, ckpt_every=n)
    assert ctx.memory_used() - before < (n + 40) * field
    with pytest.raises(ov.OvError):
        ctx.set_adjoint_memory(-1)
    ctx.close()
