"""Dslash launches whose shape nobody chose, and those whose shape somebody did: what they reserve, report and run."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
BYTES = {"fp64": 16, "fp32": 8, "bf16": 4}


def _ctx(L, bc=(2, 0, 0, 2)):
    from paper_1111_6288_amd import ov
    ctx = ov.Context(L, bc, -1.5)
    ctx.upload_gauge(torch.from_numpy(synth.su3_links(L, 0.3, 5)).cuda())
    ctx.set_fields((2 / 3, -1 / 3), (1e-3, -1e-3))
    return ctx


def _x(L, n):
    gen = torch.Generator(device="cuda").manual_seed(2)
    return torch.randn((n, synth.volume(L), 4, 3), dtype=torch.complex128, device="cuda", generator=gen)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("L,n", [((4, 4, 4, 8), 3), ((8, 8, 8, 16), 60)])
def test_dslash_reserves_no_output_batch_that_it_does_not_write(L, n, prec):
    """Direction waves and shared links write the caller's output: the workspace holds the packed input alone."""
    ctx = _ctx(L)
    before = ctx.memory_used()
    ctx.dslash(_x(L, n), prec=prec)
    assert ctx.memory_used() - before < 1.5 * n * 12 * BYTES[prec] * synth.volume(L) + 65536
    ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("L,n", [((4, 4, 4, 8), 3), ((8, 8, 8, 16), 60)])
def test_profile_counts_the_bytes_of_the_layout_that_is_written(L, n, prec):
    """ov_prof_query: two-row links, the packed input and the output, complex128 where the kernel writes the caller's."""
    ctx = _ctx(L)
    x = _x(L, n)
    S, V = BYTES[prec], synth.volume(L)
    for chosen, out in ((False, 16), (True, S)):
        if chosen:   # this shape leaves the output to the unpacking pass
            ctx.set_launch_config(prec, "dslash", rhs_per_thread=2, block=128)
        ctx.prof_enable(True)
        ctx.dslash(x, prec=prec)
        assert ctx.prof_query("dslash")[0::2] == (1, V * (24.0 * S + n * 12.0 * (S + out)))
        ctx.prof_enable(False)
    ctx.close()
