"""Paths of the kernels that the parity suites do not reach by their inputs:
states far from one in binary32 and binary64 (the range test of the face states), and both sides of
the batch size below which a leaf gets a workgroup of its own."""
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


@pytest.mark.parametrize("recon", [0, 1])
@pytest.mark.parametrize("rho_exp,p_exp", [(0, 0), (-510, -510), (0, 510), (0, -510), (495, 10),
                                           (-498, 0)])
def test_fp64_states_far_from_one(env, rho_exp, p_exp, recon):
    """The same in binary64, whose refined reciprocal and root are correctly
    rounded inside the range they serve and IEEE outside it: the oracle's
    bits."""
    torch, hb = env
    print(f"case rho 2^{rho_exp} p 2^{p_exp} recon {recon}", flush=True)
    base, rng = 2, np.random.default_rng(8)
    coord = inputs.uniform_leaves(base)
    X, Y, Z = inputs.cell_centres(coord, base)
    wave = 0.1 * np.sin(2 * np.pi * X) * np.cos(2 * np.pi * Y)
    rho = 2.0 ** rho_exp * (1.0 + wave + 1e-2 * rng.uniform(-1, 1, X.shape))
    p = 2.0 ** p_exp * (1.0 + 0.1 * np.cos(2 * np.pi * Z) + 1e-2 * rng.uniform(-1, 1, X.shape))
    zero = np.zeros_like(rho)
    U = inputs.conserved(rho, zero, zero, zero, p)
    grid = hb.Grid(coord, base, 6, hb.HYDRO_F64, reconstruction=recon)
    T = oracle.Table(coord, base)
    dt_o = oracle.cfl_dt(T, U, 0.4)
    dt = torch.tensor([dt_o], dtype=torch.float64, device="cuda")
    out = grid.empty_state()
    hb.hydro_step(grid, None, torch.from_numpy(U).to("cuda"), out, dt, 1.0)
    oracle.set_recon(recon)
    try:
        ref, bad = oracle.step(T, U, dt_o)
    finally:
        oracle.set_recon(0)
    assert bad == 0 and hb.hydro_check_status(grid) == hb.HYDRO_OK
    assert np.array_equal(out.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("what", ["rho<0", "rho=0", "p<0", "nan"])
def test_unphysical_states_are_reported(env, what, dtype):
    """A state that meets rho <= 0, p <= 0 or NaN at a face sets the status,
    from whichever field holds it."""
    torch, hb = env
    coord = inputs.uniform_leaves(2)
    w = inputs.uniform_state(2)
    U = w.U.copy()
    if what == "rho<0":
        U[0, 3] *= -1.0
    elif what == "rho=0":
        U[0, 3] = 0.0
    elif what == "p<0":
        U[4, 3] = -1.0
        U[5, 3] = -1.0
    else:
        U[2, 3, 4, 4, 4] = np.nan
    tdt = torch.float64 if dtype == 0 else torch.float32
    grid = hb.Grid(coord, 2, 6, dtype)
    dt = torch.tensor([1e-4], dtype=torch.float64, device="cuda")
    out = grid.empty_state()
    hb.hydro_step(grid, None, torch.from_numpy(U).to("cuda").to(tdt).contiguous(), out, dt, 1.0)
    assert hb.hydro_check_status(grid) == hb.HYDRO_E_UNPHYSICAL


def _species(w, nf, seed):
    rng = np.random.default_rng(seed)
    extra = [w.U[0] * rng.uniform(0.1, 0.3, size=w.U[0].shape) for _ in range(nf - 6)]
    return np.ascontiguousarray(np.concatenate([w.U[:6]] + [e[None] for e in extra]))


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("nf,leaf_waves,waves", [(6, 1, 1), (6, 1, 2), (7, 2, 1), (8, 1, 2),
                                                 (11, 1, 1), (11, 2, 2), (16, 1, 2), (16, 2, 1),
                                                 (16, 2, 2)])
def test_launch_shapes_on_a_large_batch(env, nf, leaf_waves, waves, dtype):
    """Register budgets and wavefronts per leaf on a batch above every size
    that gives a leaf its own workgroup (4404 leaves, coarser and refined
    neighbours): binary64 the oracle's bits, binary32 within its rounding."""
    torch, hb = env
    print(f"case nf {nf} waves/leaf {leaf_waves} waves/SIMD {waves} dtype {dtype}", flush=True)
    w = inputs.blobs(base=4, max_level=3)
    U = _species(w, nf, nf)
    tdt = torch.float64 if dtype == 0 else torch.float32
    grid = hb.Grid(w.leaf_coord, w.base, nf, dtype)
    T = oracle.Table(w.leaf_coord, w.base)
    keys = (hb.HYDRO_OPT_WAVES_PER_SIMD, hb.HYDRO_OPT_WAVES_PER_LEAF)
    old = [hb.hydro_get_option(dtype, nf, k) for k in keys]
    for k, v in zip(keys, (waves, leaf_waves)):
        hb.hydro_set_option(dtype, nf, k, v)
    try:
        dt_o = oracle.cfl_dt(T, U, 0.4)
        dt = torch.tensor([dt_o], dtype=torch.float64, device="cuda")
        out = grid.empty_state()
        hb.hydro_step(grid, None, torch.from_numpy(U).to("cuda").to(tdt).contiguous(), out, dt, 1.0)
        ref, bad = oracle.step(T, U, dt_o)
        assert bad == 0
        got = out.double().cpu().numpy()
        if dtype == 0:
            assert np.array_equal(got, ref)
        else:
            top = np.abs(ref).reshape(nf, -1).max(1)
            assert np.all(np.abs(got - ref).reshape(nf, -1).max(1) < 1e-5 * top)
    finally:
        for k, v in zip(keys, old):
            hb.hydro_set_option(dtype, nf, k, v)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("nf", [6, 8, 11, 12, 13, 16])
@pytest.mark.parametrize("n_leaves", [1, 8, 216, 729, 1000])
def test_rk3_step_on_both_sides_of_the_whole_leaf_limit(env, n_leaves, nf, dtype):
    """One chained RK3 step with rotation on uniform boxes from one leaf to
    past the largest batch that gives each leaf a workgroup: binary64 within
    1e-12 of the oracle (its bits expected), binary32 within its rounding, and
    the time step it leaves is the minimum of the state it leaves."""
    torch, hb = env
    print(f"case {n_leaves} leaves nf {nf} dtype {dtype}", flush=True)
    base = round(n_leaves ** (1 / 3))
    coord = inputs.uniform_leaves(base)
    w = inputs.random_smooth(coord, base, nf=6, seed=nf)
    U = _species(w, nf, nf)
    tdt = torch.float64 if dtype == 0 else torch.float32
    grid = hb.Grid(coord, base, nf, dtype, omega=0.3, cfl_epilogue=True)
    T = oracle.Table(coord, base)
    Un = torch.from_numpy(U).to("cuda").to(tdt).contiguous()
    W1, W2, out = (grid.empty_state() for _ in range(3))
    dt = torch.zeros(2, dtype=torch.float64, device="cuda")
    hb.hydro_cfl_dt(grid, Un, 0.0, dt[1:])
    hb.hydro_rk3_step(grid, Un, W1, W2, out, 0.4, dt)
    assert hb.hydro_check_status(grid) == hb.HYDRO_OK
    got = out.double().cpu().numpy()
    oracle.set_omega(0.3)
    try:
        ref, dt_o, bad = oracle.rk3_step(T, U.astype(got.dtype) if dtype == 0 else
                                         U.astype(np.float32).astype(np.float64), 0.4)
    finally:
        oracle.set_omega(0.0)
    assert bad == 0
    top = np.abs(ref).reshape(nf, -1).max(1)
    err = np.abs(got - ref).reshape(nf, -1).max(1) / top
    assert np.all(err < (1e-12 if dtype == 0 else 1e-5)), err
    assert dt[1].item() == oracle.cfl_dt(T, got, 1.0)
    if dtype == 0:
        assert dt[0].item() == dt_o


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("coarse", [[(1, 1, 1)], [(1, 1, 1), (2, 1, 1), (0, 0, 0)]])
def test_flux_correction_of_cells_on_several_refined_faces(env, coarse, dtype):
    """Coarse leaves all but surrounded by refined blocks: their edge and corner
    cells lie on two and three refined faces and take the corrections in the
    order x, y, z, low before high.  Binary64 the oracle's bits, binary32
    within its rounding (a stored value and up to three corrections of it)."""
    torch, hb = env
    print(f"case coarse leaves {coarse} dtype {dtype}", flush=True)
    base = 3
    rows = []
    for z, y, x in np.ndindex(base, base, base):
        if (x, y, z) in coarse:
            rows.append((0, x, y, z))
        else:
            rows += [(1, 2 * x + (q & 1), 2 * y + (q >> 1 & 1), 2 * z + (q >> 2)) for q in range(8)]
    coord = np.array(rows, np.int32)
    coord = np.ascontiguousarray(coord[inputs.morton_order(coord)])
    w = inputs.random_smooth(coord, base, nf=8, seed=3)
    tdt = torch.float64 if dtype == 0 else torch.float32
    grid = hb.Grid(coord, base, 8, dtype, reflux=True)
    assert grid.n_slots
    T = oracle.Table(coord, base)
    U = torch.from_numpy(w.U).to("cuda").to(tdt).contiguous()
    W1, W2, out = (grid.empty_state() for _ in range(3))
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    hb.hydro_rk3_step(grid, U, W1, W2, out, 0.4, dt)
    ref, dt_o, bad = oracle.rk3_step(T, U.double().cpu().numpy(), 0.4, reflux=True)
    assert bad == 0 and dt.item() == dt_o
    got = out.double().cpu().numpy()
    if dtype == 0:
        assert np.array_equal(got, ref)
    else:
        top = np.abs(ref).reshape(8, -1).max(1)
        assert np.all(np.abs(got - ref).reshape(8, -1).max(1) < 5e-6 * top)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n_leaves,nf", [(1, 6), (8, 16), (1000, 7), (1331, 6), (4913, 6)])
def test_totals_over_batches(env, n_leaves, nf, dtype):
    """Totals over batches below, at and past the number of workgroups per
    field and the four leaves a workgroup loads at a time, against sums in
    extended precision: double-double sums leave one rounding of the total,
    plus one of each product, of random sign."""
    torch, hb = env
    base = round(n_leaves ** (1 / 3))
    print(f"case {n_leaves} leaves nf {nf} dtype {dtype}", flush=True)
    rng = np.random.default_rng(n_leaves)
    tdt = np.float64 if dtype == 0 else np.float32
    U = rng.normal(size=(nf, base ** 3, 8, 8, 8)).astype(tdt)
    grid = hb.Grid(inputs.uniform_leaves(base), base, nf, dtype)
    tot = torch.zeros(nf, dtype=torch.float64, device="cuda")
    also = torch.zeros(nf, dtype=torch.float64, device="cuda")
    Ud = torch.from_numpy(U).to("cuda")
    hb.hydro_totals(grid, Ud, tot)
    hb.hydro_totals_noalloc(grid, Ud, also)
    dv = (1.0 / (8 * base)) ** 3
    want = U.astype(np.longdouble).reshape(nf, -1).sum(1) * np.longdouble(dv)
    scale = np.abs(U.astype(np.float64)).reshape(nf, -1).sum(1) * dv
    assert np.all(np.abs(tot.cpu().numpy() - want.astype(np.float64)) <= 1e-15 * scale)
    assert torch.equal(tot, also)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("nf", [6, 11, 16])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_ghost_fill_at_any_alignment(env, shift, nf, dtype):
    """Tiles written to buffers that are not 16-byte aligned, and input states
    that are not, on a tree with coarser and refined neighbours: binary64 the
    oracle's bits, binary32 the bits of its own aligned call and within a
    rounding of each mean."""
    torch, hb = env
    print(f"case shift {shift} nf {nf} dtype {dtype}", flush=True)
    w = inputs.blobs(base=2, max_level=2, threshold=0.5)
    U = _species(w, nf, nf)
    tdt = torch.float64 if dtype == 0 else torch.float32
    grid = hb.Grid(w.leaf_coord, w.base, nf, dtype)
    src = torch.from_numpy(U).to("cuda").to(tdt).contiguous()
    shape = (nf, w.n_leaves, 14, 14, 14)
    n = int(np.prod(shape))
    buf = torch.full((n + 4,), -7.0, dtype=tdt, device="cuda")
    inb = torch.zeros(src.numel() + 4, dtype=tdt, device="cuda")
    inb[shift:shift + src.numel()] = src.reshape(-1)
    G = buf[shift:shift + n].view(shape)
    hb.hydro_fill_ghosts(grid, inb[shift:shift + src.numel()].view(src.shape), G)
    want = oracle.fill_ghosts(oracle.Table(w.leaf_coord, w.base), src.double().cpu().numpy())
    got = G.double().cpu().numpy()
    if dtype == 0:
        assert np.array_equal(got, want)
    else:
        assert np.all(np.abs(got - want) <= 3e-7 * np.abs(want).reshape(nf, -1).max(1)
                      .reshape(nf, 1, 1, 1, 1))
        plain = torch.empty(shape, dtype=tdt, device="cuda")
        hb.hydro_fill_ghosts(grid, src, plain)
        assert torch.equal(plain, G)
    rest = torch.cat([buf[:shift], buf[shift + n:]])
    assert torch.all(rest == -7.0)


@pytest.mark.parametrize("dtype,nf", [(0, 7), (0, 8), (0, 9), (0, 10), (1, 6), (1, 8), (1, 12)])
def test_3d_forms_at_every_register_layout(env, dtype, nf):
    """The workgroup form of the 3D step that shares line reconstructions (8
    wavefronts in binary64, 4 in binary32) at the field counts between the
    smallest and the largest it takes: the bits of the one-wavefront form,
    with the flux correction and rotation on."""
    torch, hb = env
    print(f"case 3D forms dtype {dtype} nf {nf}", flush=True)
    w = inputs.blobs(base=2, max_level=2, threshold=0.5)
    tdt = torch.float64 if dtype == 0 else torch.float32
    U = torch.from_numpy(_species(w, nf, nf)).to("cuda").to(tdt).contiguous()
    grid = hb.Grid(w.leaf_coord, w.base, nf, dtype, omega=0.7, reflux=True,
                   reconstruction=hb.HYDRO_RECON_3D)
    old = hb.hydro_get_option(dtype, nf, hb.HYDRO_OPT_3D_WORKGROUP)
    outs = []
    try:
        for form in (2, 0):
            hb.hydro_set_option(dtype, nf, hb.HYDRO_OPT_3D_WORKGROUP, form)
            W1, W2, Un = (grid.empty_state() for _ in range(3))
            dt = torch.zeros(1, dtype=torch.float64, device="cuda")
            hb.hydro_rk3_step(grid, U, W1, W2, Un, 0.4, dt)
            assert hb.hydro_check_status(grid) == hb.HYDRO_OK
            outs.append(Un.cpu().numpy())
    finally:
        hb.hydro_set_option(dtype, nf, hb.HYDRO_OPT_3D_WORKGROUP, old)
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype,rho_exp,p_exp", [
    (0, 0, 0), (0, -510, -510), (0, 0, -510), (0, 495, 10), (0, 0, -1030), (1, 0, 0),
    (1, -30, 70), (1, 95, 0)])
@pytest.mark.parametrize("n_leaves,nf", [(8, 6), (1000, 6), (1000, 11)])
def test_cfl_minimum_left_by_the_step_is_that_of_a_pass(env, n_leaves, nf, dtype, rho_exp, p_exp):
    """The minimum that the step kernel leaves beside its output, with the
    refined reciprocal and root and one division per wavefront, has the bits
    of the time-step pass over that output (IEEE operations, one division per
    cell): densities and squared sound speeds inside and outside the refined
    range, a quarter of the cells under the dual-energy switch."""
    torch, hb = env
    print(f"case {n_leaves} leaves nf {nf} dtype {dtype} rho 2^{rho_exp} p 2^{p_exp}", flush=True)
    base, rng = round(n_leaves ** (1 / 3)), np.random.default_rng(9)
    coord = inputs.uniform_leaves(base)
    X, Y, Z = inputs.cell_centres(coord, base)
    rho = 2.0 ** rho_exp * (1.0 + 0.1 * np.sin(2 * np.pi * X) + 1e-2 * rng.uniform(-1, 1, X.shape))
    p = 2.0 ** p_exp * (1.0 + 0.1 * np.cos(2 * np.pi * Z) + 1e-2 * rng.uniform(-1, 1, X.shape))
    zero = np.zeros_like(rho)
    # a fast quarter of the box, whose kinetic energy hides the internal one
    fast = np.where((X < 0.5) & (Y < 0.5), 100.0 * 2.0 ** (0.5 * (p_exp - rho_exp)), 0.0)
    w = inputs.random_smooth(coord, base, nf=6, seed=nf)
    w.U = inputs.conserved(rho, zero, zero, zero + fast, p)
    U = _species(w, nf, nf) if nf > 6 else w.U
    tdt = torch.float64 if dtype == 0 else torch.float32
    Ud = torch.from_numpy(U).to("cuda").to(tdt).contiguous()
    grid = hb.Grid(coord, base, nf, dtype, cfl_epilogue=True)
    W1, W2, out = (grid.empty_state() for _ in range(3))
    dt, ref = (torch.zeros(2, dtype=torch.float64, device="cuda") for _ in range(2))
    hb.hydro_cfl_dt(grid, Ud, 0.0, dt[1:])
    hb.hydro_rk3_step(grid, Ud, W1, W2, out, 0.1, dt)
    hb.hydro_cfl_dt(grid, out, 0.0, ref[1:])
    got, want = dt[1].item(), ref[1].item()
    assert got == want and got > 0.0, (got, want)


@pytest.mark.parametrize("nf", [6, 9, 10, 11, 13, 16])
def test_3d_one_wavefront_form_matches_the_oracle(env, nf):
    """The 3D form with one wavefront a leaf on both sides of the field count
    from which it forms the points' states ahead, a later stage with rotation:
    the oracle's bits."""
    torch, hb = env
    print(f"case 3D one wavefront nf {nf}", flush=True)
    w = inputs.blobs(base=2, max_level=2, threshold=0.5)
    U = _species(w, nf, nf)
    grid = hb.Grid(w.leaf_coord, w.base, nf, hb.HYDRO_F64, omega=0.7,
                   reconstruction=hb.HYDRO_RECON_3D)
    T = oracle.Table(w.leaf_coord, w.base)
    U0 = U * 1.01
    old = hb.hydro_get_option(0, nf, hb.HYDRO_OPT_3D_WORKGROUP)
    hb.hydro_set_option(0, nf, hb.HYDRO_OPT_3D_WORKGROUP, 0)
    try:
        dt = torch.tensor([1e-4], dtype=torch.float64, device="cuda")
        out = grid.empty_state()
        hb.hydro_step(grid, torch.from_numpy(U0).to("cuda"), torch.from_numpy(U).to("cuda"), out,
                      dt, 0.25)
        got = out.cpu().numpy()
    finally:
        hb.hydro_set_option(0, nf, hb.HYDRO_OPT_3D_WORKGROUP, old)
    oracle.set_recon(1)
    oracle.set_omega(0.7)
    try:
        ref, bad = oracle.step(T, U, 1e-4, beta=0.25, U0=U0)
    finally:
        oracle.set_recon(0)
        oracle.set_omega(0.0)
    assert bad == 0 and np.array_equal(got, ref)


def _box_refined_at(base, n_refined):
    """A box of base^3 sub-grids, its first n_refined in Morton order refined."""
    coord = inputs.uniform_leaves(base)
    rows = []
    for i, (_, x, y, z) in enumerate(coord[inputs.morton_order(coord)]):
        if i < n_refined:
            rows += [(1, 2 * x + (q & 1), 2 * y + (q >> 1 & 1), 2 * z + (q >> 2)) for q in range(8)]
        else:
            rows.append((0, x, y, z))
    coord = np.array(rows, np.int32)
    return np.ascontiguousarray(coord[inputs.morton_order(coord)])


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("nf", range(6, 17))
@pytest.mark.parametrize("base,n_refined", [(3, 1), (5, 2), (6, 2), (8, 1), (8, 18), (10, 1),
                                            (10, 15)])
def test_default_shapes_in_every_mode(env, base, n_refined, nf, dtype):
    """A chained, rotating RK3 step on octrees of 34, 139, 230, 519, 638, 1007
    and 1105 leaves, on both sides of every batch size at which the launch
    shape changes, for every field count: the first two substeps leave the
    node copies, the last the CFL minimum, as the options of an untouched
    process have it.  Binary64 the oracle's bits; binary32 within its rounding
    over the three stages, and the minimum is that of the state it leaves."""
    torch, hb = env
    coord = _box_refined_at(base, n_refined)
    print(f"case {len(coord)} leaves nf {nf} dtype {dtype}", flush=True)
    w = inputs.random_smooth(coord, base, nf=6, seed=nf)
    U = _species(w, nf, nf)
    tdt = torch.float64 if dtype == 0 else torch.float32
    Un = torch.from_numpy(U).to("cuda").to(tdt).contiguous()
    grid = hb.Grid(coord, base, nf, dtype, omega=0.3, cfl_epilogue=True)
    assert grid.c.n_nodes
    W1, W2, out = (grid.empty_state() for _ in range(3))
    dt = torch.zeros(2, dtype=torch.float64, device="cuda")
    hb.hydro_cfl_dt(grid, Un, 0.0, dt[1:])
    hb.hydro_rk3_step(grid, Un, W1, W2, out, 0.4, dt)
    assert hb.hydro_check_status(grid) == hb.HYDRO_OK
    got = out.double().cpu().numpy()
    T = oracle.Table(coord, base)
    oracle.set_omega(0.3)
    try:
        ref, dt_o, bad = oracle.rk3_step(T, Un.double().cpu().numpy(), 0.4)
    finally:
        oracle.set_omega(0.0)
    assert bad == 0 and dt[0].item() == dt_o
    if dtype == 0:
        assert np.array_equal(got, ref)
    else:
        top = np.abs(ref).reshape(nf, -1).max(1)
        assert np.all(np.abs(got - ref).reshape(nf, -1).max(1) < 1e-5 * top)
    assert dt[1].item() == oracle.cfl_dt(T, got, 1.0)


@pytest.mark.parametrize("nf,waves,leaf_waves", [(8, 1, 1), (9, 1, 1), (9, 2, 2)])
def test_another_shape_than_the_default_below_1024_leaves(env, nf, waves, leaf_waves):
    """A shape other than the default's, set at 8 and 9 binary64 fields, takes
    the place of the batch's own: the options read back, and the result is the
    oracle's."""
    torch, hb = env
    print(f"case nf {nf} waves {waves} {leaf_waves}", flush=True)
    coord = _box_refined_at(10, 1)
    w = inputs.random_smooth(coord, 10, nf=6, seed=nf)
    U = _species(w, nf, nf)
    grid = hb.Grid(coord, 10, nf, hb.HYDRO_F64)
    keys = (hb.HYDRO_OPT_WAVES_PER_SIMD, hb.HYDRO_OPT_WAVES_PER_LEAF)
    old = [hb.hydro_get_option(0, nf, k) for k in keys]
    try:
        for k, v in zip(keys, (waves, leaf_waves)):
            hb.hydro_set_option(0, nf, k, v)
            assert hb.hydro_get_option(0, nf, k) == v
        dt = torch.tensor([1e-4], dtype=torch.float64, device="cuda")
        out = grid.empty_state()
        hb.hydro_step(grid, None, torch.from_numpy(U).to("cuda"), out, dt, 1.0)
        ref, bad = oracle.step(oracle.Table(coord, 10), U, 1e-4)
        assert bad == 0 and np.array_equal(out.cpu().numpy(), ref)
    finally:
        for k, v in zip(keys, old):
            hb.hydro_set_option(0, nf, k, v)


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("nf", [6, 7, 16])
@pytest.mark.parametrize("base,n_refined", [(1, 0), (7, 5), (7, 7), (16, 0), (16, 1)])
def test_ghost_fill_on_both_sides_of_its_batch_sizes(env, base, n_refined, nf, dtype):
    """Tiles of 1, 378, 392, 4,096 and 4,103 leaves: fields in two groups, an odd
    count among them, 512 and 256 threads a leaf.  Binary64 the oracle's bits;
    binary32 within a rounding of each mean, whose operands are within a few
    per cent of each other, and of one addition in its sum."""
    torch, hb = env
    coord = _box_refined_at(base, n_refined)
    print(f"case {len(coord)} leaves nf {nf} dtype {dtype}", flush=True)
    tdt = torch.float64 if dtype == 0 else torch.float32
    rng = np.random.default_rng(nf)
    U = torch.from_numpy(rng.uniform(1.0, 1.1, size=(nf, len(coord), 8, 8, 8))).to("cuda").to(tdt)
    grid = hb.Grid(coord, base, nf, dtype)
    G = torch.full((nf, len(coord), 14, 14, 14), -7.0, dtype=tdt, device="cuda")
    hb.hydro_fill_ghosts(grid, U.contiguous(), G)
    want = oracle.fill_ghosts(oracle.Table(coord, base), U.double().cpu().numpy())
    got = G.double().cpu().numpy()
    if dtype == 0:
        assert np.array_equal(got, want)
    else:
        assert np.abs(got - want).max() <= 3e-7 * 1.1
