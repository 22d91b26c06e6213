"""A field of a batched CGLS against its own solve, bit for bit."""

import pytest

from paper_1501_04950_amd import dwa, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# lattices of the wave hop and of the site blocks; batches on both sides of the sites from
# which a hop without norms gives a wave several sites (32768; BF16 8192)
CASES = [((4, 4, 4, 4), 8, 12, "f64"), ((8, 8, 8, 16), 9, 9, "f64"), ((8, 4, 4, 8), 12, 3, "f64"),
         ((8, 8, 8, 8), 12, 3, "f64"), ((8, 8, 8, 16), 9, 9, "f32"), ((8, 8, 8, 16), 12, 6, "bf16"),
         ((8, 4, 8, 8), 9, 70, "f64"), ((8, 4, 8, 8), 7, 140, "f32"), ((6, 4, 8, 8), 9, 70, "bf16"),
         ((10, 4, 4, 6), 9, 80, "bf16"), ((22, 2, 4, 4), 12, 110, "bf16"), ((12, 8, 12, 16), 9, 4, "bf16")]



@pytest.mark.parametrize("dims,Ls,n,inner", CASES)
def test_batch_follows_its_single_solves(dims, Ls, n, inner):
    """The same iterations of every source in one batch and alone, with one fold of a mixed
    solve at the end.  (Sources of whole numbers: their norms, by which a mixed solve scales
    them and which a batch sums on the host, are exact.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] batch bits {dims} Ls={Ls} {inner} x{n}", flush=True)
    ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(synth.su3_field(dims, 0.5, 7)).cuda())
    ctx.reserve_batch(n)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rhs = torch.stack([ctx.half_field("f64") for _ in range(n)]).contiguous()
    re, im = (torch.randint(-1, 2, rhs.shape, generator=gen, device="cuda").double() for _ in range(2))
    rhs.copy_(torch.complex(re, im))
    o = dict(tol=1e-12, inner_prec=inner, delta=1e-3, maxiter=24, check_every=4)
    xs, st, _ = dwa.cgne_solve_batch([(ctx, rhs)], **o)
    for k in range(n):
        x, s, _ = ctx.cgne_solve(rhs[k].contiguous(), **o)
        assert st[0][k]["iters"] == s["iters"] and st[0][k]["outer"] == s["outer"]
        assert torch.equal(xs[0][k], x), (k, float((xs[0][k] - x).abs().max() / x.abs().max()))
    ctx.close()


@pytest.mark.parametrize("what", ["up1", "up2", "hopall", "smix"])
@pytest.mark.parametrize("Ls", [8, 9])  # site-block kernels, wave hop
@pytest.mark.parametrize("inner", ["f64", "f32"])
def test_serial_launches_give_the_batch(inner, Ls, what, monkeypatch):
    """DWA_BATCH_SERIAL runs the named batched kernels field by field: the same solve."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] serial {what} {inner} Ls={Ls}", flush=True)
    dims, n = (8, 8, 8, 8), 3
    ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(synth.su3_field(dims, 0.3, 7)).cuda())
    ctx.reserve_batch(n)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rhs = torch.stack([ctx.half_field("f64") for _ in range(n)]).contiguous()
    rhs.copy_(torch.randn(rhs.shape, dtype=rhs.dtype, device="cuda", generator=gen))
    o = dict(tol=1e-6, inner_prec=inner, delta=0.1, maxiter=600, check_every=3)
    xs, st, rc = dwa.cgne_solve_batch([(ctx, rhs)], **o)
    monkeypatch.setenv("DWA_BATCH_SERIAL", what)
    ys, tt, rd = dwa.cgne_solve_batch([(ctx, rhs)], **o)
    assert rc == rd == dwa.DWA_OK
    assert [s["iters"] for s in st[0]] == [t["iters"] for t in tt[0]]
    assert torch.equal(xs[0], ys[0])
    ctx.close()


@pytest.mark.parametrize("dims,Ls,inner", [((4, 8, 16, 20), 4, "bf16"), ((4, 16, 32, 34), 8, "f32"), ((2, 16, 32, 66), 8, "bf16")])
def test_updates_of_both_chiralities(dims, Ls, inner):
    """Lattices whose CG updates take both chiralities in a thread: the solution against that
    of the dense kernels, and a zero source beside it in a batch."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] updates {dims} Ls={Ls} {inner}", flush=True)
    ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(synth.su3_field(dims, 0.3, 7)).cuda())
    ctx.reserve_batch(2)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rhs = torch.zeros((2,) + tuple(ctx.half_field("f64").shape), dtype=torch.complex128, device="cuda")
    rhs[0].copy_(torch.randn(rhs[0].shape, dtype=rhs.dtype, device="cuda", generator=gen))
    o = dict(tol=1e-9, inner_prec=inner, delta=0.1, check_every=5, maxiter=2000)
    x, s, rc = ctx.cgne_solve(rhs[0].contiguous(), **o)
    xs, _, rb = dwa.cgne_solve_batch([(ctx, rhs)], **o)
    ctx.set_tuning(inner, 8, "slab", 1, True)
    g, _, rg = ctx.cgne_solve(rhs[0].contiguous(), **o)
    assert rc == rb == rg == dwa.DWA_OK and not xs[0][1].abs().any()
    n = torch.linalg.vector_norm(g)
    assert torch.linalg.vector_norm(x - g) <= 1e-7 * n and torch.linalg.vector_norm(xs[0][0] - g) <= 1e-7 * n
    ctx.close()
