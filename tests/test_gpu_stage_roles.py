"""The two-role stage kernel at the sizes where it can go wrong: a grid smaller than the halo box
(wraps on every side), one point past a brick along each axis, bricks whose box crosses one face
only, and several bricks per workgroup (the ring and the exchange carried from brick to brick), for
every brick shape and both fluid schemes; fluid-recovery failures are counted once per point and stage.
Bars as in the parity tests (1e-11 of the oracle) and, between the kernel variants, round-off: each
right-hand side sums a few hundred terms of at most the field's size, so 1e-13 of it."""
import numpy as np
import pytest
import torch

from tests.inputs import fuzz_state
from tests.test_gpu_parity import err_fields, mk, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2606_02053_amd as P
    return P


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("n", [(8, 8, 8), (16, 4 + 4, 9), (18, 9, 8), (34, 8, 13), (48, 17, 22)])
def test_edges_against_oracle(P, orc, n, scheme):
    L = tuple(0.25 * m for m in n)
    s, sol = mk(P, orc, n, L, fluid_scheme=scheme)
    u = fuzz_state(n, seed=31)
    dt = 0.25 * min(s.h)
    rhs, _ = orc.rhs(s, u, t=0.2)
    one, _ = orc.rk4(s, u, 0.2, dt, 1)
    for tile in ((16, 4, 4), (16, 8, 2), (8, 8, 4), (8, 4, 8)):
        sol.params.tile_x, sol.params.tile_y, sol.params.tile_z = tile
        sol.set_state(to_dev(u), t=0.2)
        assert err_fields(sol.rhs().cpu().numpy(), rhs)[0] < 1e-11, tile
        sol.step(dt)
        assert err_fields(sol.u.cpu().numpy(), one)[0] < 1e-11, tile


@pytest.mark.parametrize("n,order", [((80, 60, 66), 1), ((80, 60, 66), 0), ((64, 64, 64), 2)])
def test_many_bricks_per_workgroup_and_failure_counts(P, orc, n, order):
    L = tuple(0.1 * m for m in n)
    _, sol = mk(P, orc, n, L)
    u = fuzz_state(n, seed=32)
    bad = np.random.default_rng(3).choice(np.prod(n), size=37, replace=False)
    u[21].reshape(-1)[bad] *= -1.0  # negative energy density: the recovery fails there
    sol.set_state(to_dev(u))
    out, count = {}, {}
    for variant in (0, 1):
        sol.params.variant, sol.params.tile_order = variant, order
        P.cosmos_status_reset(sol.ws)
        out[variant] = sol.rhs(t=0.1).cpu().numpy()
        count[variant] = sol.status()["prim_fail"]
    assert err_fields(out[0], out[1])[0] < 1e-13
    assert count[0] == count[1] == 37


@pytest.mark.parametrize("n", [(19, 9, 8), (21, 8, 9), (33, 9, 8), (35, 10, 11), (49, 8, 8)])
def test_odd_widths(P, orc, n):
    """Odd n0: the narrowest LDS-staged width (21) and the widest direct one (19), and widths whose last
    brick holds 1, 3 and 5 columns, so that the upper face cuts the halo boxes of two bricks; state
    arrays at either 8-byte alignment give the same bits."""
    L = tuple(0.25 * m for m in n)
    s, sol = mk(P, orc, n, L)
    u = fuzz_state(n, seed=33)
    sol.set_state(to_dev(u), t=0.2)
    ref, _ = orc.rhs(s, u, t=0.2)
    got = sol.rhs()
    assert err_fields(got.cpu().numpy(), ref)[0] < 1e-11
    buf = torch.empty(u.size + 1, dtype=torch.float64, device="cuda")
    for k in (0, 1):
        view = buf[k:k + u.size]
        view.copy_(sol.u.reshape(-1))
        out = torch.empty_like(sol.u)
        P.cosmos_rhs(sol.grid, sol.params, 0.2, view, out, sol.ws)
        assert torch.equal(out, got), k
    fields = {}
    for variant in (0, 1):
        sol.params.variant = variant
        _, H, M = sol.constraints(want_fields=True)
        fields[variant] = torch.cat([H.reshape(-1), M.reshape(-1)])
    assert torch.equal(fields[0], fields[1])
    kb = fuzz_state(n, seed=34)
    ws = torch.empty(P.cosmos_adjoint_workspace_bytes(sol.grid), dtype=torch.uint8, device="cuda")
    vjp = torch.empty_like(sol.u)
    P.cosmos_rhs_vjp(sol.grid, sol.params, 0.2, sol.u, to_dev(kb), vjp, ws)
    tape = orc.vjp(s, u, kb, "rhs", t=0.2).reshape(25, -1)
    d = np.abs(vjp.cpu().numpy().reshape(25, -1) - tape).max(axis=1)
    assert (d / np.maximum(np.abs(tape).max(axis=1), 1e-8 * np.abs(tape).max())).max() < 1e-11
