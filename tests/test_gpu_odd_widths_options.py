"""Odd widths with the options that the LDS-staged kernels carry: the scalar field (its own staged kernel, the
stage kernel's sources and the constraints with them) and the Kurganov-Tadmor scheme, from the narrowest staged
width (21), with 1, 3 and 5 columns in the last brick, and the widest direct width (19) beside them. Bars as in the
parity tests (1e-11 of the oracle field by field); state arrays at either 8-byte alignment give the same bits."""
import pytest
import torch

from tests.inputs import fuzz_scalar, fuzz_state
from tests.test_gpu_parity import err_fields, to_dev
from tests.test_gpu_scalar import err2, mk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2606_02053_amd as P
    return P


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("n", [(19, 9, 8), (21, 8, 9), (33, 9, 8), (35, 10, 11), (49, 8, 8)])
def test_odd_widths_with_the_scalar_field(P, orc, n, scheme):
    L = tuple(0.25 * m for m in n)
    s, sol = mk(P, orc, n, L, fluid_scheme=scheme)
    u, sc = fuzz_state(n, seed=71), fuzz_scalar(n, seed=72)
    sol.set_state(to_dev(u), t=0.2, s=to_dev(sc))
    du, ds = sol.rhs(t=0.2)
    ru, rs, _ = orc.rhs_sc(s, u, sc, t=0.2)
    assert err_fields(du.cpu().numpy(), ru)[0] < 1e-11
    assert err2(ds.cpu().numpy(), rs)[0] < 1e-11
    ub = torch.empty(u.size + 1, dtype=torch.float64, device="cuda")
    sb = torch.empty(sc.size + 1, dtype=torch.float64, device="cuda")
    um, sm = ub[1:], sb[1:]
    um.copy_(sol.u.reshape(-1))
    sm.copy_(sol.s.reshape(-1))
    du1, ds1 = torch.empty_like(du), torch.empty_like(ds)
    P.cosmos_rhs_scalar(sol.grid, sol.params, 0.2, um, sm, du1, ds1, sol.ws, sol.sws)
    assert torch.equal(du1, du) and torch.equal(ds1, ds)
    fields = {}
    for variant in (0, 1):
        sol.params.variant = variant
        _, H, M = sol.constraints(want_fields=True)
        fields[variant] = torch.cat([H.reshape(-1), M.reshape(-1)])
    sol.params.variant = 0
    assert torch.equal(fields[0], fields[1])
    dt = 0.25 * min(s.h)
    sol.step(dt)
    ru, rs, _ = orc.rk4_sc(s, u, sc, 0.2, dt, 1)
    assert err_fields(sol.u.cpu().numpy(), ru)[0] < 1e-11
    assert err2(sol.s.cpu().numpy(), rs)[0] < 1e-11


@pytest.mark.parametrize("n", [(19, 9, 8), (21, 8, 9), (33, 9, 8), (35, 10, 11), (49, 8, 8)])
def test_odd_widths_with_kurganov_tadmor(P, orc, n):
    L = tuple(0.25 * m for m in n)
    s, sol = orc.Setup(n=n, L=L, fluid_scheme=1), P.Solver(n, L, P.make_params(fluid_scheme=1))
    u = fuzz_state(n, seed=73)
    dt = 0.25 * min(s.h)
    rhs, _ = orc.rhs(s, u, t=0.2)
    one, _ = orc.rk4(s, u, 0.2, dt, 1)
    for tile in ((16, 4, 4), (16, 8, 2), (8, 8, 4), (8, 4, 8)):
        sol.params.tile_x, sol.params.tile_y, sol.params.tile_z = tile
        sol.set_state(to_dev(u), t=0.2)
        assert err_fields(sol.rhs().cpu().numpy(), rhs)[0] < 1e-11, tile
        sol.step(dt)
        assert err_fields(sol.u.cpu().numpy(), one)[0] < 1e-11, tile
