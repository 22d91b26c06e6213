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
