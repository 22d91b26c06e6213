"""The wave-per-site hop (D_bb, D_bb^dag and the solvers on the L_s and lattices that it
runs) against the CPU oracle and against the generic kernels, which dense matrices select."""

import numpy as np
import pytest

from oracle import redblack
from paper_1501_04950_amd import dwa, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# As in the parity tests: FP64 agrees to rounding, FP32 and BF16 storage to a few units of
# theirs (two hops and two roundings of a field).
TOL = {"f64": 1e-13, "f32": 2e-6, "bf16": 2e-2}


def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda", 0)


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


class Setup:
    def __init__(self, dims, Ls):
        rng = np.random.default_rng(Ls)
        b, c = rng.uniform(1.0, 2.0, Ls), rng.uniform(0.1, 0.9, Ls)
        self.dims, self.Ls = dims, Ls
        U = synth.su3_field(dims, 0.5, 3 + Ls)
        self.rb = redblack.RedBlack(U, redblack.Params.make(dims, Ls, -1.8, 0.05, 0.8, b, c))
        self.x = synth.gaussian_field5(dims, Ls, 11) * self.rb.black
        self.ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, b, c)
        self.ctx.set_links(torch.from_numpy(U).to(gpu()))

    def pack(self, prec):
        return self.ctx.pack(torch.from_numpy(self.x).to(gpu()), 0, prec)

    def full(self, half, prec):
        out = torch.zeros(self.x.shape, dtype=torch.complex128, device=gpu())
        self.ctx.unpack(half, 0, prec, out=out)
        return out.cpu().numpy()


# the shortest and longest L_s, odd ones, those with and without kernels of their own; x rows
# of 1, 2, 3, 4 and 5 sites, and site numbers that no tile divides
SHAPES = [((2, 2, 2, 6), 2), ((6, 2, 4, 2), 3), ((4, 4, 4, 4), 4), ((10, 2, 2, 6), 5), ((4, 2, 6, 2), 7),
          ((4, 4, 4, 4), 8), ((10, 6, 2, 4), 9), ((6, 2, 2, 4), 10), ((8, 2, 2, 10), 12), ((2, 2, 6, 2), 13),
          ((6, 6, 2, 2), 15), ((10, 2, 4, 2), 16)]


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("dims,Ls", SHAPES)
def test_wave_dbb(dims, Ls, prec):
    """D_bb and D_bb^dag against the oracle and the dense kernels; a batch that passes
    through the tiled relayout gives bitwise the output of one field read in place."""
    s = Setup(dims, Ls)
    ctx, x = s.ctx, s.pack(prec)
    print(f"[gpu] wave D_bb {dims} Ls={Ls} {prec}", flush=True)
    ns, order, nf = 8, "slab", 1  # (dense matrices run 8 sites per block)
    ctx.set_tuning(prec, ns, order, nf, 0)
    y, z = ctx.apply_Dbb(x, prec), ctx.apply_Dbb_dag(x, prec)
    ctx.set_tuning(prec, ns, order, nf, 1)
    gy, gz = ctx.apply_Dbb(x, prec), ctx.apply_Dbb_dag(x, prec)
    ref, ref_d = s.rb.Dbb(s.x), s.rb.Dbb_dag(s.x)
    fy, fz = s.full(y, prec), s.full(z, prec)
    e, ed = rel(fy, ref), rel(fz, ref_d)
    g, gd = rel(s.full(gy, prec), ref), rel(s.full(gz, prec), ref_d)
    print(f"    error {e:.2e}, dagger {ed:.2e} (dense {g:.2e}, {gd:.2e})", flush=True)
    assert max(e, ed) < TOL[prec] and max(g, gd) < TOL[prec]

    ctx.set_tuning(prec, ns, order, nf, 0)
    if Ls in (4, 8, 12, 16) or (Ls in (6, 10, 14) and prec != "bf16"):  # larger batches: site blocks
        ctx.close()
        return
    nbytes = x.numel() * x.element_size()
    n = max(3, (2 << 20) // nbytes + 1)
    ctx.reserve_batch(n)
    xs = torch.stack([x * (1 + k % 3) for k in range(n)]).contiguous()
    for f in (1, 2):
        ctx.set_tuning(prec, ns, order, f, 0)
        ys, nrm = ctx.apply_Dbb_batch(xs, prec, norms=True)
        for k in range(min(n, 6)):
            yk = ctx.apply_Dbb(xs[k].contiguous(), prec)
            assert torch.equal(ys[k], yk), (f, k)
            want = float((torch.view_as_real(yk) if yk.is_complex() else yk).double().square().sum())
            assert abs(nrm[k] - want) <= 1e-12 * want if prec == "f64" else abs(nrm[k] - want) <= 1e-5 * want
    ctx.close()


@pytest.mark.parametrize("inner,delta", [("f64", 0.1), ("f32", 0.02), ("bf16", 0.3)])
@pytest.mark.parametrize("mode", ["reliable", "defect"])
@pytest.mark.parametrize("dims,Ls", [((10, 2, 2, 6), 5), ((6, 4, 2, 4), 9), ((4, 4, 4, 4), 12)])
def test_wave_solvers(dims, Ls, mode, inner, delta):
    """Propagators (one source and a batch) of the site-major solvers against those of the
    dense kernels: both residuals are below tol, so the propagators agree to kappa * tol."""
    tol = 1e-11
    s = Setup(dims, Ls)
    ctx = s.ctx
    V = int(np.prod(dims))
    eta = np.stack([synth.point_source(dims, 1, k // 3, k % 3) for k in range(3)]).reshape(3, V, 4, 3)
    eta = torch.from_numpy(eta).to(gpu())
    o = dict(tol=tol, inner_prec=inner, delta=delta, check_every=3, mixed_mode=mode, maxiter=4000)
    print(f"[gpu] wave solve {dims} Ls={Ls} {inner} mode {mode}", flush=True)
    ctx.reserve_batch(3)
    ys, stats, rc = ctx.propagator_batch(eta, **o)
    assert rc == dwa.DWA_OK
    ns, order, nf = 8, "slab", 1  # (dense matrices run 8 sites per block)
    for k in range(3):
        ctx.set_tuning(inner, ns, order, nf, 0)
        y, st, rc = ctx.propagator(eta[k].contiguous(), **o)
        ctx.set_tuning(inner, ns, order, nf, 1)
        g, sg, rcg = ctx.propagator(eta[k].contiguous(), **o)
        assert rc == dwa.DWA_OK and rcg == dwa.DWA_OK
        assert max(st["rel_resid"], sg["rel_resid"], stats[k]["rel_resid"]) <= 1.01 * tol
        n = float(torch.linalg.vector_norm(g))
        d, db = float(torch.linalg.vector_norm(y - g)) / n, float(torch.linalg.vector_norm(ys[k] - g)) / n
        print(f"    source {k}: {st['iters']} / {sg['iters']} iterations, difference {d:.1e}, batch {db:.1e}", flush=True)
        assert max(d, db) <= 1e-8
    ctx.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("Ls", [6, 10, 14])
def test_even_ls_site_blocks(Ls, prec):
    """L_s = 6, 10, 14 beyond the wave hop's lattices: their site-block kernels (16 sites, the
    last block partly filled) against the oracle and the dense kernels, every block order
    and several fields per block bit for bit."""
    s = Setup((6, 6, 10, 6), Ls)
    ctx, x = s.ctx, s.pack(prec)
    print(f"[gpu] site-block D_bb Ls={Ls} {prec}", flush=True)
    ref, ref_d = s.rb.Dbb(s.x), s.rb.Dbb_dag(s.x)
    ctx.reserve_batch(3)
    xs = torch.stack([x * (1 + k) for k in range(3)]).contiguous()
    first = None
    for order in ("slab", "lex"):
        for nf in (1, 2):
            ctx.set_tuning(prec, 8, order, nf, 0)
            y, z = ctx.apply_Dbb(x, prec), ctx.apply_Dbb_dag(x, prec)
            ys = ctx.apply_Dbb_batch(xs, prec)
            first = first or (y, z, ys)
            assert all(torch.equal(a, b) for a, b in zip((y, z, ys), first))
            assert torch.equal(ys[0], y)
    e, ed = rel(s.full(first[0], prec), ref), rel(s.full(first[1], prec), ref_d)
    ctx.set_tuning(prec, 8, "slab", 1, 1)
    g = rel(s.full(ctx.apply_Dbb(x, prec), prec), ref)
    print(f"    error {e:.2e}, dagger {ed:.2e} (dense {g:.2e})", flush=True)
    assert max(e, ed, g) < TOL[prec]
    with pytest.raises(dwa.DwaError):
        ctx.set_tuning(prec, 16, "slab", 1, 0)
    ctx.close()
