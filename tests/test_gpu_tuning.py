"""The tuning of the hop: what dwa_get_tuning reports is what dwa_set_tuning takes, and what
the autotuner measures is what the context runs."""

import json

import pytest

from paper_1501_04950_amd import dwa, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def context(dims, Ls, batch=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(synth.su3_field(dims, 0.5, 7)).cuda())
    if batch:
        ctx.reserve_batch(batch)
    return ctx


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("Ls", [5, 6, 8, 10, 14])
def test_tuning_round_trip(Ls, prec, tmp_path):
    """The default, an autotuned and a dense configuration go back through set_tuning; a
    cache file written by one call of the autotuner serves the next one."""
    ctx = context((4, 4, 4, 6), Ls)
    print(f"[gpu] tuning round trip Ls={Ls} {prec}", flush=True)
    t = ctx.get_tuning(prec)
    ctx.set_tuning(prec, *t)
    assert ctx.get_tuning(prec) == t
    cache = str(tmp_path / "tune.json")
    first = ctx.autotune(prec, reps=2, cache=cache)
    assert not first["cached"] and first["us"] is not None
    second = ctx.autotune(prec, reps=2, cache=cache)
    t = (first["ns"], first["order"], first["nf"], first["dense"])
    assert second["cached"] and ctx.get_tuning(prec) == t
    ctx.set_tuning(prec, *t)
    ctx.set_tuning(prec, 8, "slab", 1, True)
    t = ctx.get_tuning(prec)
    assert t == (8, "slab", 1, True)
    ctx.set_tuning(prec, *t)
    ctx.close()


def test_refused_cache_entry_is_tuned_again(tmp_path):
    """A stored tile that the library does not take (16 at an L_s of one tile) is a miss."""
    ctx = context((4, 4, 4, 4), 6)
    cache = str(tmp_path / "tune.json")
    ctx.autotune("f64", reps=2, cache=cache)
    data = json.load(open(cache))
    (key,) = data
    data[key]["ns"] = 16
    json.dump(data, open(cache, "w"))
    res = ctx.autotune("f64", reps=2, cache=cache)
    assert not res["cached"] and res["ns"] == 8
    assert json.load(open(cache))[key]["ns"] == 8
    assert ctx.autotune("f64", reps=2, cache=cache)["cached"]
    ctx.close()


def test_fields_per_block_are_timed_by_the_hop_that_has_them(monkeypatch):
    """The autotuner's times of the fields per block are the site-block hop's, also where this
    batch runs the wave hop (which takes about 0.6 of its time here and leaves larger ones to
    it); none are taken where the wave hop runs every batch."""
    dims, Ls = (4, 4, 4, 4), 4
    ctx = context(dims, Ls, 12)
    monkeypatch.setenv("DWA_NO_WAVE_HOP", "1")
    ref = context(dims, Ls, 12)
    us = [1e9, 1e9]
    for _ in range(3):
        for k, c in enumerate((ctx, ref)):
            t = c.autotune("bf16", reps=30)["candidates"]
            us[k] = min([us[k]] + [e["us"] for e in t if e["nrhs"] > 1 and e["us"] >= 0])
    print(f"[gpu] fields per block: {us[0]:.1f} us, without the wave hop {us[1]:.1f}", flush=True)
    assert us[0] > 0.8 * us[1]
    ctx.close()
    ref.close()
    monkeypatch.delenv("DWA_NO_WAVE_HOP")
    ctx = context(dims, 9, 12)
    t = ctx.autotune("bf16", reps=2)
    assert t["nf"] == 1 and {e["nrhs"] for e in t["candidates"]} == {1}
    ctx.close()


def test_wave_solve_does_not_depend_on_the_order():
    """The wave hop's walk follows from the lattice, so its sums do not move with a tuning."""
    dims, Ls = (4, 2, 16, 8), 9
    ctx = context(dims, Ls)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rhs = ctx.half_field("f64")
    rhs.copy_(torch.randn(rhs.shape, dtype=rhs.dtype, device="cuda", generator=gen))
    xs = []
    for order in ("slab", "lex", "zdom"):
        ctx.set_tuning("f64", 8, order)
        xs.append(ctx.cgne_solve(rhs, tol=1e-12, maxiter=40, check_every=8)[0].clone())
    assert torch.equal(xs[0], xs[1]) and torch.equal(xs[0], xs[2])
    ctx.close()


@pytest.mark.parametrize("variable", ["DWA_DENSE_MIX", "DWA_NO_WAVE_HOP"])
def test_no_gathered_links_without_the_wave_hop(variable, monkeypatch):
    """A context that never runs the wave hop holds no second copy of the links: 144 numbers
    per site of a parity in FP64 and BF16 (FP32 runs it on smaller lattices at this L_s)."""
    dims, Ls = (16, 16, 16, 16), 3
    need = 144 * 16**4 // 2 * (16 + 4)

    def held():
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
        used = before - torch.cuda.mem_get_info()[0]
        ctx.close()
        return used

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    held()  # (first-use allocations)
    full = held()
    monkeypatch.setenv(variable, "1")
    assert full - held() >= 0.9 * need
