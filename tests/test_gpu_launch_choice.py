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


def test_launch_plan_names_what_runs():
    ctx = _ctx((8, 8, 8, 16))
    kernel = {(p, n): ctx.launch_plan(p, "dslash", n)["kernel"] for p in BYTES for n in (1, 2, 12, 60)}
    assert kernel["fp64", 2] == kernel["fp32", 12] == kernel["bf16", 12] == "directions"   # small batches
    assert kernel["fp64", 60] == kernel["fp32", 60] == kernel["bf16", 60] == "share"       # more than the caches hold
    stored = ctx.get_launch_config("fp32", "clenshaw")
    assert not any(ctx.launch_plan(p, k, n)["chosen"] for p in BYTES for k in ("dslash", "clenshaw") for n in (1, 60))
    assert ctx.get_launch_config("fp32", "clenshaw") == stored
    for cfg, name in ((dict(rhs_per_thread=2, block=512), "sites"), (dict(rhs_per_thread=1, wshare=8), "share"),
                      (dict(rhs_per_thread=2, wshare=4), "share_multi"), (dict(site_order=2, wshare=1), "march")):
        ctx.set_launch_config("fp32", "clenshaw", **cfg)
        p = ctx.launch_plan("fp32", "clenshaw", 60)
        assert p["chosen"] and p["kernel"] == name
    # the shape follows the batch and the lattice: two vectors need no eight waves, a z extent of 4 no slabs
    ctx.set_launch_config("fp32", "clenshaw", rhs_per_thread=1, wshare=8, site_order=1)
    assert ctx.launch_plan("fp32", "clenshaw", 2)["wshare"] == 2
    ctx.close()
    ctx = _ctx((8, 8, 4, 16))
    ctx.set_launch_config("fp32", "dslash", site_order=1)
    assert ctx.launch_plan("fp32", "dslash", 2)["site_order"] == 0
    assert not ctx.launch_plan("fp32", "clenshaw", 2)["chosen"]
    for bad in (("fp32", "dslash", 0),):
        with pytest.raises(Exception):
            ctx.launch_plan(*bad)
    ctx.close()


def test_setting_the_value_in_place_chooses_nothing():
    ctx = _ctx((8, 8, 8, 16))
    rule = ctx.launch_plan("fp32", "clenshaw", 4)
    ctx.set_site_order("fp32", 0)
    ctx.set_occupancy("fp32", 0)
    assert ctx.launch_plan("fp32", "clenshaw", 4) == rule and not rule["chosen"]
    ctx.set_occupancy("fp32", 2)
    plan = ctx.launch_plan("fp32", "clenshaw", 4)
    assert plan["chosen"] and plan["blocks_per_cu"] == 2
    ctx.set_site_order("fp32", 0)   # nor does it take a choice back
    assert ctx.launch_plan("fp32", "clenshaw", 4) == plan
    ctx.set_site_order("fp64", 1)
    assert ctx.launch_plan("fp64", "dslash", 4)["site_order"] == 1
    ctx.close()


def test_a_shape_can_be_limited_to_its_batch_and_dropped(tmp_path):
    L, n = (8, 8, 8, 16), 24
    ctx = _ctx(L)
    x = _x(L, 30)
    rule = {m: ctx.launch_plan("fp64", "dslash", m) for m in (1, 12, 13, 24, 47, 48)}
    ref = {m: ctx.dslash(x[:m].contiguous()) for m in (12, 24)}
    ctx.set_launch_config("fp64", "dslash", rhs_per_thread=2, block=64)
    assert all(ctx.launch_plan("fp64", "dslash", m)["chosen"] for m in rule)   # a setter speaks of every batch
    ctx.set_launch_batch("fp64", "dslash", n)
    for m, p in rule.items():
        q = ctx.launch_plan("fp64", "dslash", m)
        assert (q["chosen"] and q["block"] == 64) if 12 < m < 48 else q == p
    for m, y in ref.items():   # 12 vectors by the rule, 24 by the shape
        assert torch.equal(ctx.dslash(x[:m].contiguous()), y)
    ctx.set_launch_config("fp64", "dslash", block=128)
    assert ctx.launch_plan("fp64", "dslash", 1)["chosen"]
    ctx.set_launch_batch("fp64", "dslash", -1)
    assert all(ctx.launch_plan("fp64", "dslash", m) == p for m, p in rule.items())
    with pytest.raises(Exception):
        ctx.set_launch_batch("fp64", "dslash", -2)
    # a record, limited to its batch and not
    rec = tmp_path / "shapes.jsonl"
    rec.write_text('{"arch": "gfx950", "L": [8, 8, 8, 16], "prec": 0, "nrhs": 24, "kind": "dslash", "rhs_per_thread": 2, '
                   '"block": 64, "site_order": 0, "blocks_per_cu": 0, "ms_per_launch": 0.1}\n')
    assert ctx.load_tuning(str(rec), "fp64", n, near_only=True) == ["dslash"]
    assert [ctx.launch_plan("fp64", "dslash", m)["chosen"] for m in (1, 24)] == [False, True]
    assert ctx.load_tuning(str(rec), "fp64", n) == ["dslash"]
    assert [ctx.launch_plan("fp64", "dslash", m)["chosen"] for m in (1, 24)] == [True, True]
    ctx.close()


def test_the_last_record_of_a_kind_holds(tmp_path):
    ctx = _ctx((8, 8, 8, 16))
    rule = ctx.launch_plan("fp32", "clenshaw", 24)
    head = '{"arch": "gfx950", "L": [8, 8, 8, 16], "prec": 1, "nrhs": 24, "kind": "clenshaw", "rhs_per_thread": 2, '
    shape = head + '"block": 64, "site_order": 0, "blocks_per_cu": 0, "ms_per_launch": 0.1, "ms_unchosen": 0.2}\n'
    keep = head + '"block": 256, "site_order": 0, "blocks_per_cu": 0, "ms_per_launch": 0.2, "ms_unchosen": 0.1}\n'
    rec = tmp_path / "shapes.jsonl"
    rec.write_text(shape + keep)
    ctx.set_launch_config("fp32", "clenshaw", rhs_per_thread=4, block=128)   # nor does an earlier choice stay
    assert "clenshaw" in ctx.load_tuning(str(rec), "fp32", 24)
    assert ctx.launch_plan("fp32", "clenshaw", 24) == rule
    rec.write_text(keep + shape)
    assert "clenshaw" in ctx.load_tuning(str(rec), "fp32", 24)
    assert ctx.launch_plan("fp32", "clenshaw", 24)["block"] == 64
    ctx.close()


@pytest.mark.parametrize("prec,n", [("fp64", 3), ("fp32", 12), ("bf16", 24)])
def test_autotune_keeps_the_rule_unless_a_shape_is_ahead(prec, n, tmp_path):
    import json
    L, path = (8, 8, 8, 16), tmp_path / "shapes.jsonl"
    ctx = _ctx(L)
    x = _x(L, n)
    ref = ctx.dslash(x, prec=prec)
    rule = {k: ctx.launch_plan(prec, k, n) for k in ("dslash", "clenshaw")}
    ctx.autotune(prec, n, str(path))
    recs = [json.loads(line) for line in path.read_text().splitlines()]
    assert [r["kind"] for r in recs] == ["dslash", "clenshaw"]
    plan = {k: ctx.launch_plan(prec, k, n) for k in rule}
    for r in recs:
        ahead = r["ms_per_launch"] / r["ms_unchosen"]   # the file rounds to a nanosecond
        assert (r["chosen"] == 1 and ahead < 0.981) or (r["chosen"] == 0 and ahead > 0.979)
        assert plan[r["kind"]]["chosen"] == bool(r["chosen"])
        assert r["chosen"] or plan[r["kind"]] == rule[r["kind"]]
    assert torch.equal(ctx.dslash(x, prec=prec), ref)
    ctx.close()
    ctx = _ctx(L)
    assert ctx.load_tuning(str(path), prec, n) == ["dslash", "clenshaw"]
    assert {k: ctx.launch_plan(prec, k, n) for k in rule} == plan
    ctx.close()
