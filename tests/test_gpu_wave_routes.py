"""The wave hop's own forms: its tiled batches, several sites per wave and its walk, and the
site-major solvers of L_s = 6, 10 and 14."""

import numpy as np
import pytest

from oracle import redblack
from paper_1501_04950_amd import dwa, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6, "bf16": 2e-2}  # as in the parity tests


def context(dims, Ls, U, batch=0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(U).cuda())
    if batch:
        ctx.reserve_batch(batch)
    return ctx


# BF16 batches above 2 MB, which pass through the tiled store: L_s of the site blocks too
# (6144 sites at most for L_s = 8), rows of 1 to 11 sites, z of one plane group and of eight;
# 16 and 22 sites of x: eight of a wave in a row, and across rows
TILED = [((2, 2, 6, 2), 8, 240), ((10, 2, 2, 6), 8, 48), ((6, 2, 4, 2), 12, 80), ((14, 2, 2, 2), 12, 140),
         ((16, 2, 2, 4), 12, 40), ((16, 2, 16, 2), 16, 6), ((6, 2, 16, 2), 16, 16), ((22, 2, 2, 2), 16, 70),
         ((12, 6, 16, 2), 9, 7)]


@pytest.mark.parametrize("dims,Ls,n", TILED)
def test_tiled_batches(dims, Ls, n):
    """D_bb of such a batch and its norms against D_bb of one field read in place, which the
    oracle checks."""
    U = synth.su3_field(dims, 0.5, 3)
    rb = redblack.RedBlack(U, redblack.Params.make(dims, Ls, -1.8, 0.05, 0.8, np.full(Ls, 1.5), np.full(Ls, 0.5)))
    f = synth.gaussian_field5(dims, Ls, 11) * rb.black
    ctx = context(dims, Ls, U, n)
    print(f"[gpu] tiled wave batch {dims} Ls={Ls} x{n}", flush=True)
    x = ctx.pack(torch.from_numpy(f).cuda(), 0, "bf16")
    assert n * x.numel() * x.element_size() > 2 << 20
    xs = torch.stack([x * (1 + k % 3) for k in range(n)]).contiguous()
    ys, nrm = ctx.apply_Dbb_batch(xs, "bf16", norms=True)
    for k in range(3):
        y = ctx.apply_Dbb(xs[k].contiguous(), "bf16")
        for j in range(k, n, 3):
            assert torch.equal(ys[j], y), j
            want = float(y.double().square().sum())
            assert abs(nrm[j] - want) <= 1e-5 * want
    out = torch.zeros(f.shape, dtype=torch.complex128, device="cuda")
    ctx.unpack(ys[0], 0, "bf16", out=out)
    ref = rb.Dbb(f)
    assert np.linalg.norm(out.cpu().numpy() - ref) < TOL["bf16"] * np.linalg.norm(ref)
    ctx.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("dims,Ls,n", [((4, 2, 16, 2), 9, 3), ((6, 2, 16, 4), 7, 3), ((2, 4, 32, 2), 13, 2),
                                       ((16, 2, 2, 4), 7, 260), ((6, 2, 16, 4), 7, 180)])
def test_walk_and_sites_per_wave(dims, Ls, n, prec):
    """z-plane groups, and batches of 32768 sites and more, whose waves take several sites
    each: D_bb and D_bb^dag against the oracle, the batch bit for bit the single call."""
    U = synth.su3_field(dims, 0.5, 3)
    rb = redblack.RedBlack(U, redblack.Params.make(dims, Ls, -1.8, 0.05, 0.8, np.full(Ls, 1.5), np.full(Ls, 0.5)))
    f = synth.gaussian_field5(dims, Ls, 11) * rb.black
    ctx = context(dims, Ls, U, n)
    print(f"[gpu] wave walk {dims} Ls={Ls} {prec} x{n}", flush=True)
    x = ctx.pack(torch.from_numpy(f).cuda(), 0, prec)
    first = None
    for order in ("slab", "lex", "zdom"):
        ctx.set_tuning(prec, 8, order)
        got = ctx.apply_Dbb(x, prec), ctx.apply_Dbb_dag(x, prec)
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first)), order
    xs = torch.stack([x * (1 + k % 3) for k in range(n)]).contiguous()
    ys = ctx.apply_Dbb_batch(xs, prec)
    for k in range(min(n, 3)):
        y = ctx.apply_Dbb(xs[k].contiguous(), prec)
        assert all(torch.equal(ys[j], y) for j in range(k, n, 3))
    for half, ref in zip(first, (rb.Dbb(f), rb.Dbb_dag(f))):
        out = torch.zeros(f.shape, dtype=torch.complex128, device="cuda")
        ctx.unpack(half, 0, prec, out=out)
        assert np.linalg.norm(out.cpu().numpy() - ref) < TOL[prec] * np.linalg.norm(ref)
    ctx.close()


@pytest.mark.parametrize("inner,delta", [("f64", 0.1), ("f32", 0.02), ("bf16", 0.3)])
@pytest.mark.parametrize("Ls", [6, 10, 14])
def test_even_ls_solvers(Ls, inner, delta):
    """Site-major solvers of one source and of a batch against those of the dense kernels: both
    residuals are below tol, so the propagators agree to kappa * tol."""
    dims, tol, n = (4, 2, 4, 6), 1e-11, 3
    U = synth.su3_field(dims, 0.3, 5)
    ctx = context(dims, Ls, U, n)
    print(f"[gpu] wave solve Ls={Ls} {inner}", flush=True)
    V = int(np.prod(dims))
    eta = np.stack([synth.point_source(dims, 1, k // 3, k % 3) for k in range(n)]).reshape(n, V, 4, 3)
    eta = torch.from_numpy(eta).cuda()
    o = dict(tol=tol, inner_prec=inner, delta=delta, check_every=3)
    ys, st, rc = ctx.propagator_batch(eta, **o)
    assert rc == dwa.DWA_OK
    for k in range(n):
        y, s, rc = ctx.propagator(eta[k].contiguous(), **o)
        ctx.set_tuning(inner, 8, "slab", 1, True)
        g, sg, rcg = ctx.propagator(eta[k].contiguous(), **o)
        ctx.set_tuning(inner, 8, "slab", 1, False)
        assert rc == rcg == dwa.DWA_OK
        assert max(s["rel_resid"], sg["rel_resid"], st[k]["rel_resid"]) <= 1.01 * tol
        for a in (y, ys[k]):
            assert float(torch.linalg.vector_norm(a - g)) <= 1e-8 * float(torch.linalg.vector_norm(g))
    ctx.close()


# (lattice, L_s, precision, fields, whether the wave hop runs): both sides of the lines of
# dwa_internal.h's wave_max_sites
DBB_LINES = [((8, 8, 8, 8), 2, "f32", 8, True), ((8, 8, 8, 8), 3, "f32", 9, False), ((8, 8, 8, 8), 5, "f32", 32, True),
             ((8, 8, 8, 8), 4, "f64", 1, False), ((8, 8, 8, 8), 5, "f32", 33, False), ((8, 8, 8, 8), 7, "f32", 33, True),
             ((16, 8, 16, 24), 3, "f64", 1, True), ((16, 16, 16, 16), 3, "f64", 1, False),
             ((16, 16, 16, 16), 5, "f64", 1, True), ((16, 16, 16, 16), 2, "bf16", 1, True),
             ((8, 8, 8, 8), 12, "bf16", 42, True), ((8, 8, 8, 8), 12, "bf16", 43, False)]
SOLVE_LINES = [((6, 6, 6, 12), 3, "f32", True), ((8, 8, 8, 8), 3, "f32", False), ((8, 8, 8, 8), 3, "f64", True),
               ((8, 4, 4, 8), 8, "f64", True), ((8, 4, 4, 10), 8, "f64", False), ((4, 4, 4, 8), 4, "f64", True),
               ((4, 4, 4, 10), 4, "f64", False), ((8, 4, 4, 8), 6, "f32", True), ((8, 4, 4, 10), 6, "f32", False),
               ((8, 4, 8, 8), 10, "f64", True), ((8, 4, 8, 10), 14, "f64", False), ((8, 4, 8, 10), 12, "f32", False),
               ((8, 4, 8, 8), 12, "f32", True), ((8, 8, 8, 8), 5, "f32", True), ((8, 8, 8, 8), 8, "bf16", True),
               ((8, 8, 8, 10), 8, "bf16", False), ((8, 8, 8, 10), 12, "bf16", True)]


def both_routes(monkeypatch, dims, Ls, batch, call):
    U = synth.su3_field(dims, 0.5, 3)
    out = []
    for off in (False, True):
        if off:
            monkeypatch.setenv("DWA_NO_WAVE_HOP", "1")
        ctx = context(dims, Ls, U, batch)
        gen = torch.Generator(device="cuda").manual_seed(3)
        out.append(call(ctx, gen).clone())
        ctx.close()
    return out


@pytest.mark.parametrize("dims,Ls,prec,n,wave", DBB_LINES)
def test_lines_of_dbb(dims, Ls, prec, n, wave, monkeypatch):
    """The two hops round differently, so equal bits are the site-block hop's."""
    print(f"[gpu] D_bb line {dims} Ls={Ls} {prec} x{n}", flush=True)

    def call(ctx, gen):
        x = torch.stack([ctx.half_field(prec) for _ in range(n)]).contiguous()
        x.copy_(torch.randn(x.shape, dtype=torch.float32 if prec == "bf16" else x.dtype, device="cuda", generator=gen))
        return ctx.apply_Dbb_batch(x, prec) if n > 1 else ctx.apply_Dbb(x[0], prec)

    a, b = both_routes(monkeypatch, dims, Ls, n if n > 1 else 0, call)
    assert torch.equal(a, b) == (not wave)


@pytest.mark.parametrize("dims,Ls,inner,wave", SOLVE_LINES)
def test_lines_of_solvers(dims, Ls, inner, wave, monkeypatch):
    """A few iterations and one correction: bits as above."""
    print(f"[gpu] solve line {dims} Ls={Ls} {inner}", flush=True)

    def call(ctx, gen):
        rhs = ctx.half_field("f64")
        rhs.copy_(torch.randn(rhs.shape, dtype=rhs.dtype, device="cuda", generator=gen))
        return ctx.cgne_solve(rhs, tol=1e-12, inner_prec=inner, delta=1e-3, maxiter=8, check_every=8)[0]

    a, b = both_routes(monkeypatch, dims, Ls, 0, call)
    assert torch.equal(a, b) == (not wave)
