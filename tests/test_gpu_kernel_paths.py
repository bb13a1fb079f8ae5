"""Paths of the kernels that the parity suites do not reach by their inputs:
states far from one in binary32 (the range test of the face states)."""
import numpy as np
import pytest

import oracle
from paper_2210_06437_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2210_06437_amd import binding as hb
    return torch, hb


@pytest.mark.parametrize("recon", [0, 1])
@pytest.mark.parametrize("rho_exp,p_exp", [(0, 0), (-100, -100), (-30, 70), (30, -70), (-97, -1),
                                           (95, 0)])
def test_fp32_states_far_from_one(env, rho_exp, p_exp, recon):
    """One binary32 substep of a state at rest whose density or squared sound
    speed is inside, at and outside the range that the fast reciprocal and
    root serve, against the oracle.  Tolerance: at CFL 0.4 each of a cell's
    six faces adds at most 0.4 times its flux's rounding, a few binary32
    roundings (6e-8) of the field's natural scale."""
    torch, hb = env
    print(f"case rho 2^{rho_exp} p 2^{p_exp} recon {recon}", flush=True)
    base, rng = 2, np.random.default_rng(7)
    coord = inputs.uniform_leaves(base)
    X, Y, Z = inputs.cell_centres(coord, base)
    wave = 0.1 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y)
    rho = 2.0 ** rho_exp * (1.0 + wave + 1e-2 * rng.uniform(-1, 1, X.shape))
    p = 2.0 ** p_exp * (1.0 + 0.1 * np.cos(2 * np.pi * Z) + 1e-2 * rng.uniform(-1, 1, X.shape))
    zero = np.zeros_like(rho)
    U32 = inputs.conserved(rho, zero, zero, zero, p).astype(np.float32)
    U = U32.astype(np.float64)
    grid = hb.Grid(coord, base, 6, hb.HYDRO_F32, reconstruction=recon)
    T = oracle.Table(coord, base)
    dt_o = oracle.cfl_dt(T, U, 0.4)
    dt = torch.tensor([dt_o], dtype=torch.float64, device="cuda")
    out = grid.empty_state()
    hb.hydro_step(grid, None, torch.from_numpy(U32).to("cuda"), out, dt, 1.0)
    oracle.set_recon(recon)
    try:
        ref, bad = oracle.step(T, U, dt_o)
    finally:
        oracle.set_recon(0)
    assert bad == 0
    assert hb.hydro_check_status(grid) == hb.HYDRO_OK
    got = out.double().cpu().numpy()
    c = np.sqrt(2.0 ** (p_exp - rho_exp) * 5 / 3)
    scale = [2.0 ** rho_exp] + [2.0 ** rho_exp * c] * 3 + [1.5 * 2.0 ** p_exp, U[5].max()]
    for f in range(6):
        err = np.abs(got[f] - ref[f]).max() / scale[f]
        print(f"  field {f}: {err:.2e}")
        assert err <= 2e-6, (f, err)
