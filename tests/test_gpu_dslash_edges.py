"""Branches of the dslash launches that the small lattices of the other tests do not take: vectors that stream past the
caches (four direction waves with non-temporal streams), extents above 128, and the rounding of BF16 storage."""
import numpy as np
import pytest
import torch

import synth
from oracle import api

pytestmark = pytest.mark.gpu


def _ctx(L, bc, U, mw=-1.5):
    from paper_1111_6288_amd import ov
    ctx = ov.Context(L, bc, mw)
    ctx.upload_gauge(U if torch.is_tensor(U) else torch.from_numpy(U).cuda())
    ctx.set_fields((2 / 3, -1 / 3), (0.2, -0.4))
    return ctx


def _su3(V, gen):
    """Random SU(3) links on the device: orthonormal rows, the third as their conjugated cross product."""
    a = torch.randn((4 * V, 3, 3), dtype=torch.complex128, device="cuda", generator=gen)
    r0 = a[:, 0] / torch.linalg.vector_norm(a[:, 0], dim=1, keepdim=True)
    r1 = a[:, 1] - (r0.conj() * a[:, 1]).sum(1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=1, keepdim=True)
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1, dim=1).conj()], dim=1).reshape(4, V, 3, 3)


@pytest.mark.parametrize("su3", [True, False])
@pytest.mark.parametrize("L,bc", [((24, 24, 24, 48), (2, 0, 0, 2)), ((20, 18, 15, 41), (0, 1, 2, 2))])
def test_streaming_vectors_give_the_bits_of_a_chosen_shape(L, bc, su3):
    """One and two vectors, plain (own output and the caller's) and fused launches, on z-slabs and in canonical order."""
    V = synth.volume(L)
    gen = torch.Generator(device="cuda").manual_seed(7)
    U = _su3(V, gen)
    if not su3:
        U = U * torch.exp(1j * torch.rand((4, V, 1, 1), dtype=torch.float64, device="cuda", generator=gen))
    ctx = _ctx(L, bc, U.contiguous())
    assert ctx.link_format()[0] is su3
    ctx.set_sign_params(3, 0.02, 8.5)
    x = torch.randn((2, V, 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    got = {}
    runs = [(p, n) for p in ("fp64", "fp32", "bf16") for n in (1, 2)]
    def run(prec, n):
        xs, f = x[:n].contiguous(), [0, 1][:n]
        return [ctx.dslash(xs, f, op=op, prec=prec) for op in ("HW", "DW")] + [ctx.dov_apply(xs, f, [0.1] * n, prec=prec)]
    for r in runs:
        got[r] = run(*r)
    hint = {r: ctx.launch_plan(r[0], "dslash", r[1]) for r in runs}
    assert all(hint[p, n]["kernel"] == "directions" for p in ("fp64", "fp32") for n in (1, 2))
    if V > 400000:
        assert hint["fp64", 1]["stream_hint"] == hint["fp32", 2]["stream_hint"] == 1
    for prec in ("fp64", "fp32", "bf16"):
        for kind in ("dslash", "clenshaw"):
            ctx.set_launch_config(prec, kind, rhs_per_thread=2, block=128)
    for r in runs:
        for a, b in zip(got[r], run(*r)):
            assert torch.equal(a, b), r
    ctx.close()


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-14), ("fp32", 2e-6), ("bf16", 2e-2)])
@pytest.mark.parametrize("L", [(129, 2, 3, 2), (2, 200, 2, 3), (3, 2, 257, 2), (2, 2, 2, 300), (1000, 2, 2, 2)])
def test_long_extents_match_oracle(L, prec, tol):
    """Site coordinates come from products whose shift depends on the extent from 129 on."""
    bc = (2, 1, 0, 1)
    U = synth.su3_links(L, 0.4, 3)
    ctx = _ctx(L, bc, U)
    x = synth.gaussian_spinors(L, 5, 8)
    y = ctx.dslash(torch.from_numpy(x).cuda(), [0] * 5, prec=prec).cpu().numpy()
    lat = api.Lattice(L, bc, -1.5, U, 2 / 3 * 0.2)
    for j in (0, 4):
        ref = api.dslash(lat, x[j], 1)
        assert np.abs(y[j] - ref).max() / np.abs(ref).max() < tol
    ctx.close()


@pytest.mark.parametrize("n", [1, 300])
def test_bf16_storage_rounds_to_nearest_even(n):
    """With links of zero and diagonal 1 D_w copies a site whose neighbours are zero: FP32 numbers of every kind as BF16
    storage holds them, by the packing kernel and by the stores of both stencils (one vector: direction waves, 300:
    shared links).  The numbers stand on the even sites; an odd one receives 0 * inf where they overflow."""
    L = (4, 4, 4, 8)
    V = synth.volume(L)
    ctx = _ctx(L, (2, 2, 2, 2), np.zeros((4, V, 3, 3), dtype=np.complex128), mw=-3.0)
    assert ctx.launch_plan("bf16", "dslash", n)["kernel"] == ("directions" if n == 1 else "share")
    s = np.arange(V)
    even = torch.from_numpy((s % 4 + s // 4 % 4 + s // 16 % 4 + s // 64) % 2 == 0)
    m = V // 2 * 24
    bits = torch.arange(m, dtype=torch.int64) * (2 ** 32 // m)   # subnormals, infinities and NaN among them
    first = torch.tensor([0x3F800000, 0x3F810000, 0x00000001, 0x00010000, 0x007F0000, 0x7F7F0000, 0x7F800000, 0x7FC00000])
    ties = torch.cat([first + d for d in (0, 0x7FFF, 0x8000, 0x8001)] + [first + 0x80000000])
    bits[:ties.numel()] = ties
    f = (bits - (bits >= 2 ** 31) * 2 ** 32).to(torch.int32).view(torch.float32)
    x = torch.zeros((V, 4, 3, 2), dtype=torch.float64)
    x[even] = f.to(torch.float64).reshape(-1, 4, 3, 2)
    want = x[even].to(torch.float32).to(torch.bfloat16).to(torch.float64).cuda()
    y = ctx.dslash(torch.view_as_complex(x).cuda().expand(n, -1, -1, -1).contiguous(), [0] * n, op="DW", prec="bf16")
    for j in (0, n - 1):
        got = torch.view_as_real(y[j])[even.cuda()]
        assert torch.equal(torch.isnan(got), torch.isnan(want))
        assert torch.equal(got.nan_to_num(0.0, float("inf"), float("-inf")),
                           want.nan_to_num(0.0, float("inf"), float("-inf")))
    ctx.close()


@pytest.mark.parametrize("su3", [True, False])
@pytest.mark.parametrize("L,bc", [((8, 8, 8, 16), (2, 1, 0, 2)), ((6, 5, 7, 10), (1, 2, 0, 1))])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_every_launch_shape_gives_the_bits_of_the_rule(L, bc, prec, su3):
    """Plain and fused launches of a batch, whichever kernel and shape runs them; in FP64 and FP32 also a vector alone and
    in a batch (BF16 rounds the phase of a single vector another way)."""
    U = synth.su3_links(L, 0.4, 3)
    if not su3:
        U = U * np.exp(1j * np.random.default_rng(3).uniform(-1, 1, (4, synth.volume(L), 1, 1)))
    ctx = _ctx(L, bc, np.ascontiguousarray(U))
    ctx.set_sign_params(4, 0.02, 8.5)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn((60, synth.volume(L), 4, 3), dtype=torch.complex128, device="cuda", generator=gen)
    one = dict(rhs_split=1, wshare=1, site_order=0)
    shapes = [dict(one, rhs_per_thread=nr, block=bl, site_order=o) for nr in (1, 2, 4, 8) for bl in (64, 256) for o in (0, 1, 3)]
    shapes += [dict(one, rhs_per_thread=nr, block=128, rhs_split=q, wshare=w) for nr in (1, 2) for q in (1, 2, 4)
               for w in (1, 2, 4, 8)]
    shapes += [dict(one, rhs_per_thread=nr, block=128, rhs_split=8) for nr in (1, 2) if prec != "bf16"]
    shapes += [dict(one, rhs_per_thread=1, block=bl, site_order=2) for bl in (256, 512)]

    def run(n):
        xs, f = x[:n].contiguous(), [j % 2 for j in range(n)]
        return ctx.dslash(xs, f, prec=prec), ctx.dov_apply(xs, f, [0.1] * n, prec=prec)
    ref = {n: run(n) for n in (1, 2, 5, 12, 60)}
    if prec != "bf16":
        assert all(torch.equal(r[0], ref[60][0][:n]) for n, r in ref.items())
    for s in shapes:
        for kind in ("dslash", "clenshaw"):
            ctx.set_launch_config(prec, kind, **s)
        for n, r in ref.items():
            assert all(torch.equal(a, b) for a, b in zip(r, run(n))), (s, n)
    ctx.close()
