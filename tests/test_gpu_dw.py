"""D_w on canonical fields: the direct kernel against the CPU oracle and against the packed
copies that overlapping arrays pass through."""

import ctypes

import numpy as np
import pytest

from oracle import wilson
from paper_1501_04950_amd import dwa, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# a single block of 16 sites, x rows shorter and longer than a block and no divisor of it,
# z in one group and in eight; fewer fields than waves, full blocks and a rest
@pytest.mark.parametrize("n", [1, 4, 5, 9])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 2, 2, 6), (10, 6, 2, 4), (6, 4, 8, 2), (22, 2, 16, 2)])
def test_dw_direct(dims, n):
    """24 products of order one a component and 8 sums: 1e-14 is ten times the rounding."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U = synth.su3_field(dims, 0.5, 5)
    f = synth.gaussian_source(dims, 7, leading=(n,))
    ctx = dwa.Context(dims, 9, -1.8, 0.1, 0.8, 1.5, 0.5)
    ctx.set_links(torch.from_numpy(U).cuda())
    x = torch.from_numpy(f).cuda()
    print(f"[gpu] D_w {dims} n={n}", flush=True)
    y = ctx.apply_Dw(x)
    z = x.clone()
    rc = dwa.lib().dwa_apply_Dw(ctx._h, ctypes.c_void_p(z.data_ptr()), ctypes.c_void_p(z.data_ptr()), n)
    assert rc == dwa.DWA_OK
    torch.cuda.synchronize()
    ref = wilson.dw(U, f, -1.8, dims)
    scale = np.linalg.norm(ref)
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-14 * scale
    assert np.linalg.norm(z.cpu().numpy() - ref) <= 1e-14 * scale
    ctx.close()
