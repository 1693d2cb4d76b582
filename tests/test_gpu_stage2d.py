"""The 2D PLM stage kernel at the sizes where its tiles (8 x 8 cells on small
grids, 32 x 8 or 28 x 8 on large ones) can go wrong, against the oracle (FP64 to
the repository's 1e-12 per field, mixed precision to the mixed path's stated
2e-5); and mhd_run, whose steps take dt from the stage before and alternate
between two states, against single steps, bit for bit."""
import numpy as np
import pytest

import oracle as O
from paper_2511_20337_amd import workloads as W
from tests.test_gpu_parity import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# small tiles: whole, one cell more and less, the smallest grid; large tiles
# (more than 256 of 32 x 8): ragged both ways, and more than 1024 partials
GRIDS = [(8, 8), (9, 17), (31, 7), (4, 4), (5, 40), (300, 257), (1030, 281)]


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("scheme", ["hlld", "hll_uct_hlld", "hlld_uct_hlld_rk3", "mixed_rk3",
                                    "mixed_uct_hlld"])
def test_tiles_and_run(grid, scheme):
    from paper_2511_20337_amd import mhd
    nx, ny = grid
    s, U0 = W.generic_state(2, nx, ny, 1, "minmod" if scheme == "hlld" else "vanleer",
                            "hll" if scheme.startswith("hll_") else "hlld", seed=nx + ny)
    s = dict(s, emf="uct_hlld" if "uct_hlld" in scheme else "uct_hll",
             integrator="rk3" if "rk3" in scheme else "rk2",
             precision="mixed" if "mixed" in scheme else "fp64")
    tol = 2e-5 if "mixed" in scheme else 1e-12
    print("tiles and run", grid, scheme, flush=True)
    ctx = mhd.Context(s, "cuda:0")
    U = torch.from_numpy(U0).cuda()
    c = O.cfg_from(s)
    err = rel_err(ctx.rhs(U).cpu().numpy(), O.rhs(c, U0))
    assert (err <= tol).all(), err
    # steps with dt from mhd_dt, with dt inside the step, and as one run
    Ua, Ub, dts = U.clone(), U.clone(), []
    for _ in range(3):
        dts.append(ctx.dt(Ua))
        ctx.step(Ua, dts[-1])
        ctx.step_cfl(Ub)
        assert ctx.dt_dev.item() == dts[-1]
        assert torch.equal(Ua, Ub)
    for nsteps in (3, 2):
        Uc = U.clone()
        assert ctx.run(Uc, nsteps) is Uc
        assert ctx.dt_dev.item() == dts[nsteps - 1]
        if nsteps == 3:
            assert torch.equal(Uc, Ua)
    ctx.check()
    got = Ua.cpu().numpy()
    err = rel_err(got, O.run_dts(c, U0, np.array(dts)))
    assert (err <= tol).all(), err
    for q in (0, 1, 2, 3, 4, 7):
        mag = np.abs(U0[q]).sum() + np.abs(U0[1:4]).sum() * (1 <= q <= 3)
        assert abs(got[q].sum() - U0[q].sum()) <= 1e-12 * mag, q


def test_run_reports_unphysical_cells():
    from paper_2511_20337_amd import mhd
    s, U0 = W.generic_state(2, 40, 24, 1, seed=3)
    U0[4, 0, 5, 7] = 0.0  # no energy left for the pressure
    ctx = mhd.Context(s, "cuda:0")
    ctx.run(torch.from_numpy(U0).cuda(), 2)
    with pytest.raises(mhd.Unphysical):
        ctx.check()
