"""Values at the ends of the number range in the step kernels."""
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


def _state(base, nf, what):
    """Smooth core fields, species of order one, and in the last species (or
    the field named) values at the end of the range."""
    rng = np.random.default_rng(nf)
    w = inputs.random_smooth(inputs.uniform_leaves(base), base, nf=6, seed=nf)
    extra = [w.U[0] * rng.uniform(0.1, 0.3, size=w.U[0].shape) for _ in range(nf - 6)]
    U = np.ascontiguousarray(np.concatenate([w.U[:6]] + [e[None] for e in extra]))
    if what == "tail":  # differences of 2^-600 .. 2^-480: products up to 2^-960
        U[-1] = 2.0 ** rng.uniform(-600, -480, size=U[-1].shape)
    elif what == "front":  # a front that falls by many orders of magnitude a cell
        U[-1] = 2.0 ** rng.uniform(-1000, 0, size=U[-1].shape)
    elif what != "none":
        field, value = {"nan": (nf - 1, np.nan), "inf": (nf - 1, np.inf), "nan E": (4, np.nan)}[what]
        hit = rng.random(U[field].shape) < 0.002
        hit[0, 4, 4, 4] = True
        U[field][hit] = value
    return w.leaf_coord, U


@pytest.mark.parametrize("recon", [0, 1])
@pytest.mark.parametrize("what", ["tail", "front", "nan", "inf", "nan E"])
@pytest.mark.parametrize("base,nf", [(2, 7), (2, 11), (10, 7), (10, 11)])
def test_fp64_limiter_at_the_ends_of_the_range(env, base, nf, what, recon):
    """The slope is zero wherever the product of the two one-sided differences
    is not positive: where it underflows to zero, as in the tail of a species'
    front, and where a neighbour is NaN or both differences are infinite.
    Batches for each kernel (8 and 1000 leaves), both reconstructions: the
    oracle's bits, not-a-number where it has one."""
    torch, hb = env
    print(f"case base {base} nf {nf} {what} recon {recon}", flush=True)
    coord, U = _state(base, nf, what)
    grid = hb.Grid(coord, base, nf, hb.HYDRO_F64, reconstruction=recon)
    dt = torch.tensor([1e-4], dtype=torch.float64, device="cuda")
    out = grid.empty_state()
    hb.hydro_step(grid, None, torch.from_numpy(U).to("cuda"), out, dt, 1.0)
    oracle.set_recon(recon)
    try:
        ref, _ = oracle.step(oracle.Table(coord, base), U, 1e-4)
    finally:
        oracle.set_recon(0)
    got = out.cpu().numpy()
    assert np.array_equal(got, ref, equal_nan=True), [
        int((~((g == r) | (np.isnan(g) & np.isnan(r)))).sum()) for g, r in zip(got, ref)]


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("dtype", [0, 1])
def test_3d_face_flux_that_overflows(env, dtype, form):
    """A species whose flux overflows the element type leaves infinities where
    one face of a cell is infinite and the other is not, and NaN where both
    are, as the quotient of an infinite Simpson sum by 36 is infinite: in all
    three forms of the 3D step, binary64 the oracle's result, binary32 the
    same classes of values (the state is binary64's with the species' scale
    moved to the end of the binary32 range) around the edge where the species
    falls.  At the other edge binary64's NaN is the difference of two products
    that overflow, of which binary32 forms one inside an FMA."""
    torch, hb = env
    print(f"case overflow dtype {dtype} form {form}", flush=True)
    base, nf = 4, 7
    coord = inputs.uniform_leaves(base)
    X, _, _ = inputs.cell_centres(coord, base)
    one, zero = np.ones_like(X), np.zeros_like(X)
    core = inputs.conserved(one, 1e4 * one, zero, zero, 1e6 * one)
    species = np.where(X < 0.5, 1.0, 0.0)
    U64 = np.ascontiguousarray(np.concatenate([core[:6], 1e305 * species[None]]))
    oracle.set_recon(1)
    try:
        ref, _ = oracle.step(oracle.Table(coord, base), U64, 1e-8)
    finally:
        oracle.set_recon(0)
    assert np.isinf(ref[6]).any() and np.isnan(ref[6]).any() and np.isfinite(ref[6]).any()
    U = U64.copy()
    if dtype == 1:
        U[6] = 1e36 * species
    grid = hb.Grid(coord, base, nf, dtype, reconstruction=hb.HYDRO_RECON_3D)
    old = hb.hydro_get_option(dtype, nf, hb.HYDRO_OPT_3D_WORKGROUP)
    hb.hydro_set_option(dtype, nf, hb.HYDRO_OPT_3D_WORKGROUP, form)
    try:
        dt = torch.tensor([1e-8], dtype=torch.float64, device="cuda")
        out = grid.empty_state()
        Ud = torch.from_numpy(U).to("cuda").to(grid.torch_dtype).contiguous()
        hb.hydro_step(grid, None, Ud, out, dt, 1.0)
        got = out.double().cpu().numpy()
    finally:
        hb.hydro_set_option(dtype, nf, hb.HYDRO_OPT_3D_WORKGROUP, old)
    if dtype == 0:
        assert np.array_equal(got, ref, equal_nan=True)
    else:
        falls = (X > 0.25) & (X < 0.75)
        for what in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(what(got[6][falls]), what(ref[6][falls])), what


@pytest.mark.parametrize("recon", [0, 1])
@pytest.mark.parametrize("field", [0, 1, 3, 4, 6])
@pytest.mark.parametrize("base", [2, 10])
def test_fp32_not_a_number_reaches_the_fluxes_of_its_cell(env, base, field, recon):
    """NaN in one field of a cell: every field whose flux depends on it is NaN
    in the cell and in its six face neighbours (a core field reaches all
    fields, a species itself), and where that is all of the reconstruction's
    reach, in no other cell, as in binary64; a core field's sets the status."""
    torch, hb = env
    print(f"case base {base} field {field} recon {recon}", flush=True)
    nf = 7
    coord, U = _state(base, nf, "none")
    leaf = np.flatnonzero((coord[:, 1:] == 1).all(1))[0]
    U[field, leaf, 4, 3, 5] = np.nan
    grid = hb.Grid(coord, base, nf, hb.HYDRO_F32, reconstruction=recon)
    dt = torch.tensor([1e-4], dtype=torch.float64, device="cuda")
    out = grid.empty_state()
    hb.hydro_step(grid, None, torch.from_numpy(U).to("cuda").float(), out, dt, 1.0)
    want = np.zeros(U.shape, bool)
    for z, y, x in ((4, 3, 5), (3, 3, 5), (5, 3, 5), (4, 2, 5), (4, 4, 5), (4, 3, 4), (4, 3, 6)):
        want[slice(None) if field < 5 else field, leaf, z, y, x] = True
    got = torch.isnan(out).cpu().numpy()
    assert got[want].all(), [int((want & ~got)[f].sum()) for f in range(nf)]
    if recon == 0:
        assert np.array_equal(got, want)
    status = hb.HYDRO_E_UNPHYSICAL if field < 5 else hb.HYDRO_OK
    assert hb.hydro_check_status(grid) == status
