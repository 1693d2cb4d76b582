"""The 3D face and CT kernels at the sizes where their columns (32 x 8 and 31 x 7
cells), the faces solved above them and their runs along z can go wrong, against the oracle:
FP64 to the repository's 1e-12 per field, mixed precision to the mixed path's
stated 2e-5."""
import numpy as np
import pytest

import oracle as O
from paper_2511_20337_amd import workloads as W
from tests.test_gpu_parity import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# one column; a column and one cell, or one row, more; a cell and a row less;
# the smallest grid; more than one plane per run, the last run shorter
GRIDS = [(32, 8, 4), (33, 9, 5), (31, 7, 6), (4, 4, 4), (64, 16, 9), (5, 40, 4), (65, 17, 709)]


@pytest.mark.parametrize("grid", GRIDS + [(65, 33, 707)])
@pytest.mark.parametrize("scheme", ["hlld", "hll_uct_hlld", "hlld_uct_hlld_rk3", "mixed_rk3",
                                    "hll_wenoz_uct_hlld_rk3", "hlld_wenoz"])
def test_columns_and_runs(grid, scheme):
    from paper_2511_20337_amd import mhd
    nx, ny, nz = grid
    lim = "wenoz" if "wenoz" in scheme else ("minmod" if scheme == "hlld" else "vanleer")
    s, U0 = W.generic_state(3, nx, ny, nz, lim, "hll" if scheme.startswith("hll_") else "hlld",
                            seed=nx + nz)
    s = dict(s, emf="uct_hlld" if "uct_hlld" in scheme else "uct_hll",
             integrator="rk3" if "rk3" in scheme else "rk2",
             precision="mixed" if "mixed" in scheme else "fp64")
    tol = 2e-5 if "mixed" in scheme else 1e-12
    print("columns and runs", grid, scheme, flush=True)
    ctx = mhd.Context(s, "cuda:0")
    U = torch.from_numpy(U0).cuda()
    c = O.cfg_from(s)
    err = rel_err(ctx.rhs(U).cpu().numpy(), O.rhs(c, U0))
    assert (err <= tol).all(), err
    # dt inside the step and beforehand: the same bits
    Ub, dts = U.clone(), []
    for _ in range(2):
        ctx.step_cfl(U)
        ctx.step_device_dt(Ub, ctx.dt_dev)
        dts.append(ctx.dt_dev.item())
        assert torch.equal(U, Ub)
    ctx.check()
    got = U.cpu().numpy()
    err = rel_err(got, O.run_dts(c, U0, np.array(dts)))
    assert (err <= tol).all(), err
    # the two sides of a column's edge take the same flux
    for q in range(5):
        mag = np.abs(U0[q]).sum() + np.abs(U0[1:4]).sum() * (1 <= q <= 3)
        assert abs(got[q].sum() - U0[q].sum()) <= 1e-12 * mag, q


@pytest.mark.parametrize("grid", GRIDS + [(65, 33, 707)])
@pytest.mark.parametrize("scheme", ["hlld", "hll_rk3", "mixed", "wenoz"])
def test_columns_and_runs_glm(grid, scheme):
    """The same kernel on the nine cell-centred fields of GLM cleaning."""
    from paper_2511_20337_amd import mhd
    from tests.test_gpu_glm import rel_err9
    nx, ny, nz = grid
    lim = {"mixed": "minmod", "wenoz": "wenoz"}.get(scheme, "vanleer")
    s, U = W.generic_state(3, nx, ny, nz, lim, "hll" if scheme == "hll_rk3" else "hlld",
                           seed=nx + nz)
    s, U0 = W.glm_from_ct(s, U)
    U0[8] = 0.02 * np.random.default_rng(17).normal(size=U0[8].shape)
    s = dict(s, integrator="rk3" if scheme == "hll_rk3" else "rk2",
             precision="mixed" if scheme == "mixed" else "fp64")
    print("columns and runs, GLM", grid, scheme, flush=True)
    ctx = mhd.Context(s, "cuda:0")
    Ua = torch.from_numpy(U0).cuda()
    Ub, dts = Ua.clone(), []
    for _ in range(2):
        dts.append(ctx.dt(Ua))
        ctx.step(Ua, dts[-1])
        ctx.step_cfl(Ub)
        assert ctx.dt_dev.item() == dts[-1]
        assert torch.equal(Ua, Ub)
    ctx.check()
    got = Ua.cpu().numpy()
    err = rel_err9(got, O.glm_run_dts(O.cfg_from(s), U0, np.array(dts)))
    assert (err <= (2e-5 if scheme == "mixed" else 1e-12)).all(), err
    for q in range(8):  # the same flux on both sides of a column's edge
        mag = np.abs(U0[q]).sum() + np.abs(U0[1:4]).sum() * (1 <= q <= 3)
        assert abs(got[q].sum() - U0[q].sum()) <= 1e-12 * mag, q


@pytest.mark.parametrize("grid", GRIDS[:-1] + [(40, 20, 12)])
def test_glm_wenoz_with_hll(grid):
    """The cell-by-cell WENO-Z kernel with GLM cleaning and the HLL solver."""
    from paper_2511_20337_amd import mhd
    from tests.test_gpu_glm import rel_err9
    nx, ny, nz = grid
    s, U = W.generic_state(3, nx, ny, nz, "wenoz", "hll", seed=nx + nz)
    s, U0 = W.glm_from_ct(s, U)
    U0[8] = 0.02 * np.random.default_rng(17).normal(size=U0[8].shape)
    print("GLM, WENO-Z, HLL", grid, flush=True)
    ctx = mhd.Context(s, "cuda:0")
    Ua = torch.from_numpy(U0).cuda()
    dts = []
    for _ in range(2):
        dts.append(ctx.dt(Ua))
        ctx.step(Ua, dts[-1])
    ctx.check()
    err = rel_err9(Ua.cpu().numpy(), O.glm_run_dts(O.cfg_from(s), U0, np.array(dts)))
    assert (err <= 1e-12).all(), err


@pytest.mark.parametrize("scheme", ["hll_wenoz_uct_hlld_rk3", "hlld_wenoz"])
def test_columns_and_runs_of_the_wenoz_march(scheme):
    """WENO-Z on a grid that marches (several columns each way, the last ones ragged)."""
    test_columns_and_runs((94, 63, 200), scheme)


def test_columns_and_runs_of_the_wenoz_march_glm():
    test_columns_and_runs_glm((94, 63, 200), "wenoz")
