"""The adjoint's staged kernels where their boxes and their brick order can go wrong: a grid smaller than a
box (wraps on every side), widths one and two points past a brick, odd widths from the narrowest staged one
(21) with the seam at every place in the last brick's rows, and numbers of brick layers that are not a
multiple of the order's groups of four (1, 5 and 10 of them); 19 is the widest direct width. One transposed
right-hand side and one adjoint step (which takes the gather's other forms) against the tape, at the bar of
the adjoint tests (1e-11 field by field)."""
import pytest
import torch

from tests.inputs import fuzz_direction, fuzz_state
from tests.test_gpu_adjoint import rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(8, 8, 8), (18, 9, 20), (19, 8, 9), (21, 8, 9), (33, 9, 8), (35, 10, 11), (47, 8, 8),
                               (16, 12, 37), (49, 11, 8)])
def test_sizes_against_the_tape(orc, n):
    import paper_2606_02053_amd as P
    L = tuple(0.3 * m for m in n)
    s = orc.Setup(n=n, L=L)
    u, lam = fuzz_state(n, seed=51), fuzz_direction(n, seed=52)
    dt = 0.25 * min(s.h)
    grid, params = P.make_grid(n, L), P.make_params()
    ws = torch.empty(P.cosmos_adjoint_workspace_bytes(grid), dtype=torch.uint8, device="cuda")
    ud, ld = torch.from_numpy(u).cuda(), torch.from_numpy(lam).cuda()
    out = torch.empty_like(ud)
    P.cosmos_rhs_vjp(grid, params, 0.2, ud, ld, out, ws)
    assert rel_err(out.cpu().numpy(), orc.vjp(s, u, lam, "rhs", t=0.2)) < 1e-11
    P.cosmos_adjoint_step(grid, params, 0.1, dt, ud, ld, out, ws)
    assert rel_err(out.cpu().numpy(), orc.vjp(s, u, lam, "step", t=0.1, dt=dt)) < 1e-11
