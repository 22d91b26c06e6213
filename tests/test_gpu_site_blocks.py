"""The site-block hop in contexts that run no wave hop (DWA_NO_WAVE_HOP), on lattices and
batches that the wave hop serves otherwise: tiles, block orders and fields per block."""

import numpy as np
import pytest

from oracle import redblack
from paper_1501_04950_amd import dwa, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6, "bf16": 2e-2}  # as in the parity tests


@pytest.fixture(autouse=True)
def site_blocks_only(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("DWA_NO_WAVE_HOP", "1")


def context(dims, Ls, U, batch=0):
    ctx = dwa.Context(dims, Ls, -1.8, 0.05, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(U).cuda())
    if batch:
        ctx.reserve_batch(batch)
    return ctx


def fields(ctx, prec, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.stack([ctx.half_field(prec) for _ in range(n)]).contiguous()
    src = torch.randn(x.shape, dtype=torch.float32 if prec == "bf16" else x.dtype, device="cuda", generator=gen)
    return x.copy_(src)


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("dims,Ls", [((2, 2, 2, 2), 4), ((2, 2, 8, 6), 4), ((4, 4, 4, 4), 8), ((2, 2, 2, 6), 12),
                                     ((2, 2, 2, 6), 16), ((6, 2, 8, 2), 16), ((2, 2, 2, 6), 10), ((2, 2, 2, 6), 5)])
def test_tiles_match_oracle(dims, Ls, prec):
    """Every tile and order against the oracle, and bitwise among themselves; the last blocks
    are partly filled."""
    U = synth.su3_field(dims, 0.5, 3)
    rb = redblack.RedBlack(U, redblack.Params.make(dims, Ls, -1.8, 0.05, 0.8, np.full(Ls, 1.5), np.full(Ls, 0.5)))
    f = synth.gaussian_field5(dims, Ls, 11) * rb.black
    ctx = context(dims, Ls, U)
    print(f"[gpu] site blocks {dims} Ls={Ls} {prec}", flush=True)
    x = ctx.pack(torch.from_numpy(f).cuda(), 0, prec)
    first = None
    for ns in (8, 16, 32) if Ls in (4, 8, 12, 16) else (8,):
        for order in ("slab", "lex", "zdom"):
            ctx.set_tuning(prec, ns, order)
            got = ctx.apply_Dbb(x, prec), ctx.apply_Dbb_dag(x, prec)
            first = first or got
            assert all(torch.equal(a, b) for a, b in zip(got, first)), (ns, order)
    for half, ref in zip(first, (rb.Dbb(f), rb.Dbb_dag(f))):
        out = torch.zeros(f.shape, dtype=torch.complex128, device="cuda")
        ctx.unpack(half, 0, prec, out=out)
        e = np.linalg.norm(out.cpu().numpy() - ref) / np.linalg.norm(ref)
        assert e < TOL[prec]
    ctx.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("dims,Ls", [((8, 8, 8, 16), 12), ((10, 2, 2, 6), 16), ((10, 2, 2, 6), 6)])
def test_fields_per_block(dims, Ls, prec):
    """A batch's D_bb and norms are those of one field per block, bit for bit."""
    ctx = context(dims, Ls, synth.su3_field(dims, 0.5, 23), 5)
    print(f"[gpu] site blocks, fields per block {dims} Ls={Ls} {prec}", flush=True)
    x = fields(ctx, prec, 5, 29)
    ns, order, _, _ = ctx.get_tuning(prec)
    ref, ref_n = ctx.apply_Dbb_batch(x, prec, norms=True)
    for nf in (2, 3, 5, 16):
        ctx.set_tuning(prec, ns, order, nf)
        y, nrm = ctx.apply_Dbb_batch(x, prec, norms=True)
        assert torch.equal(y, ref) and nrm == ref_n, nf
    for k in range(5):
        assert torch.equal(ref[k], ctx.apply_Dbb(x[k].contiguous(), prec))
    ctx.close()


@pytest.mark.parametrize("inner", ["f32", "bf16"])
def test_fields_per_block_solve(inner, monkeypatch):
    """A batched solve with three fields per block, replayed and eager, is that with one."""
    dims, Ls, n = (4, 4, 4, 4), 8, 4
    ctx = context(dims, Ls, synth.su3_field(dims, 0.3, 5), n)
    print(f"[gpu] site blocks, batched solve {inner}", flush=True)
    V = int(np.prod(dims))
    eta = np.stack([synth.point_source(dims, 1, k // 3, k % 3) for k in range(n)]).reshape(n, V, 4, 3)
    eta = torch.from_numpy(eta).cuda()
    o = dict(tol=1e-9, inner_prec=inner, delta=0.1, check_every=3)
    ref, _, rc = ctx.propagator_batch(eta, **o)
    assert rc == dwa.DWA_OK
    ns, order, _, _ = ctx.get_tuning(inner)
    ctx.set_tuning(inner, ns, order, 3)
    y, _, rc = ctx.propagator_batch(eta, **o)
    assert rc == dwa.DWA_OK and torch.equal(y, ref)
    monkeypatch.setenv("DWA_BATCH_NO_GRAPH", "1")
    y, _, rc = ctx.propagator_batch(eta, **o)
    assert rc == dwa.DWA_OK and torch.equal(y, ref)
    ctx.close()
