"""What the 3D stages owe to the last bit, with no oracle beside them: equal fluxes
cancel exactly, and a cell's update depends on the values about it alone, not on its
place in the grid (32 x 8 columns for the faces, 31 x 7 for CT, runs along z). Every
comparison is of the bits, so there is no tolerance."""
import numpy as np
import pytest

from paper_2511_20337_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SCHEMES = ["minmod", "hll", "hlld", "hll_uct_hlld", "uct_hlld_rk3", "mixed", "mixed_hll_uct_hlld",
           "glm", "glm_hll_minmod", "glm_mixed", "wenoz_uct_hlld_rk3", "hll_wenoz", "glm_wenoz",
           "glm_hll_wenoz"]


def setup(scheme, nx, ny, nz, box=(0, 1, 0, 1, 0, 1)):
    lim = "wenoz" if "wenoz" in scheme else ("minmod" if "minmod" in scheme else "vanleer")
    s = W.make_setup("exact3d", 3, nx, ny, nz, box, 5.0 / 3.0, 0.3, lim,
                     "hll" if "hll" in scheme.split("_") else "hlld")
    return dict(s, emf="uct_hlld" if "uct_hlld" in scheme else "uct_hll",
                integrator="rk3" if "rk3" in scheme else "rk2",
                precision="mixed" if "mixed" in scheme else "fp64",
                divb="glm" if "glm" in scheme else "ct")


def state(s, seed=3):
    """Random and physical; cells differ by some 20 %, so that every limiter branch
    and region of the solvers occurs."""
    rng = np.random.default_rng(seed)
    sh = (s["nz"], s["ny"], s["nx"])
    w = [b + 0.2 * rng.uniform(-1, 1, sh) for b in (1.0, 0.3, -0.2, 0.1, 0.8, 0.4, 0.25, -0.15)]
    U = W.assemble(s, *w)
    if s["divb"] == "glm":
        s9, U = W.glm_from_ct(s, U)
        U[8] = 0.02 * rng.uniform(-1, 1, sh)
    return U


def advance(s, U0):
    """One step of U0 (with CT also L(U0)), on the device."""
    from paper_2511_20337_amd import mhd
    ctx = mhd.Context(s, "cuda:0")
    U = torch.from_numpy(np.ascontiguousarray(U0)).cuda()
    out = [ctx.rhs(U)] if s["divb"] == "ct" else []
    dt = ctx.dt(U)
    ctx.step(U, dt)
    ctx.check()
    return out + [U, torch.tensor(dt)]


def assert_same(got, want):
    for a, b in zip(got, want):
        assert torch.equal(a, b), int((a != b).sum())


# more than one column and run each way, ragged; spacings no powers of two
@pytest.mark.parametrize("grid", [(65, 17, 12), (48, 24, 20), (5, 9, 70)])
@pytest.mark.parametrize("scheme", SCHEMES)
def test_uniform_flow_stays(grid, scheme):
    """L of a moving, magnetised uniform state is zero, and a step leaves it as it is."""
    s = setup(scheme, *grid)
    sh = (s["nz"], s["ny"], s["nx"])
    U0 = W.assemble(s, *[np.full(sh, v) for v in (1.3, 0.3, -0.2, 0.1, 0.7, 0.4, -0.25, 0.6)])
    if s["divb"] == "glm":
        _, U0 = W.glm_from_ct(s, U0)
    print("uniform flow", grid, scheme, flush=True)
    got = advance(s, U0)
    if s["divb"] == "ct":
        assert float(got[0].abs().max()) == 0.0
    if s["integrator"] == "rk2":  # (3 u + u) / 4 may round
        assert torch.equal(got[-2], torch.from_numpy(U0).cuda())


@pytest.mark.parametrize("axis", [1, 2, 3])
@pytest.mark.parametrize("scheme", SCHEMES)
def test_what_is_uniform_along_an_axis_stays_so(scheme, axis):
    s = setup(scheme, 65, 17, 21)
    U0 = state(s)
    U0 = np.repeat(U0.take([0], axis=axis), U0.shape[axis], axis=axis)
    print("uniform along", axis, scheme, flush=True)
    for a in advance(s, U0)[:-1]:
        assert torch.equal(a, a.narrow(axis, 0, 1).expand_as(a))


@pytest.mark.parametrize("grid", [(65, 17, 37), (31, 40, 16), (4, 5, 50)])
@pytest.mark.parametrize("scheme", SCHEMES)
def test_a_shifted_state_gives_the_shifted_result(grid, scheme):
    s = setup(scheme, *grid)
    U0 = state(s)
    shift = (3, 5, 13)
    print("shifted state", grid, scheme, flush=True)
    want = [torch.roll(a, shift, (1, 2, 3)) if a.dim() else a for a in advance(s, U0)]
    assert_same(advance(s, np.roll(U0, shift, (1, 2, 3))), want)


def by_cells(s):
    """Whether the faces of s are solved cell by cell (whose update is a kernel of its
    own) instead of in columns."""
    from paper_2511_20337_amd import mhd
    ctx = mhd.Context(s, "cuda:0")
    U = torch.empty(ctx.shape, dtype=torch.float64, device="cuda:0")
    for q, v in enumerate((1.0, 0.3, -0.2, 0.1, 2.0, 0.4, 0.25, -0.15, 0.0)[:ctx.shape[0]]):
        U[q] = v
    mhd.mhd_timing(ctx.ctx, True)
    ctx.step(U, 1e-6)
    return mhd.mhd_timing_read(ctx.ctx)["update"][1] > 0


# more than one column each way, ragged, and many runs along z: WENO-Z marches here, and
# solves the faces between two runs once in either
@pytest.mark.parametrize("scheme", [c for c in SCHEMES if "wenoz" in c])
def test_shifted_state_where_wenoz_marches(scheme):
    grid = (62, 15, 2000)
    assert not by_cells(setup(scheme, *grid))
    test_a_shifted_state_gives_the_shifted_result(grid, scheme)


# a periodic state held once and twice along z: on these grids one is taken cell by cell
# and the other marches. PLM on grids narrower than a column (32 x 8), with indices that
# take one remainder more (under 18, under 6) and that do not; just under and over a column
PLM = [(4, 4, 80), (17, 5, 100), (33, 9, 20), (31, 7, 500), (32, 5, 1500), (96, 5, 500),
       (40, 40, 150)]
WENOZ = {"ct": [(31, 7, 7000), (30, 8, 3000), (62, 15, 1000), (64, 64, 150)],
         "glm": [(31, 7, 3000), (28, 8, 2000), (62, 15, 400)]}


@pytest.mark.parametrize("scheme,grid", [
    (c, g) for c in SCHEMES if "wenoz" in c or "glm" in c
    for g in (PLM if "wenoz" not in c else WENOZ["glm" if "glm" in c else "ct"])])
def test_columns_against_single_cells(scheme, grid):
    """The same bits with PLM. With WENO-Z the two form a z-face's values with other
    roundings: the repository's 1e-12 of each field's maximum."""
    nx, ny, nz = grid
    s1 = setup(scheme, nx, ny, nz, (0, 1, 0, 1, 0, nz / 16))
    s2 = setup(scheme, nx, ny, 2 * nz, (0, 1, 0, 1, 0, nz / 8))
    assert by_cells(s1) != by_cells(s2)
    U0 = state(s1)
    print("columns against cells", grid, scheme, flush=True)
    once = advance(s1, U0)
    twice = advance(s2, np.concatenate([U0, U0], axis=1))
    assert twice[-1] == once[-1]  # the time step
    for a, b in zip(twice[:-1], once[:-1]):
        tol = 1e-12 * b.abs().amax(dim=(1, 2, 3), keepdim=True) if "wenoz" in scheme else 0.0
        for half in (a[:, :nz], a[:, nz:]):
            assert bool(((half - b).abs() <= tol).all())


@pytest.mark.parametrize("scheme", ["glm", "glm_mixed", "glm_wenoz", "wenoz"])
def test_a_narrow_grid_is_not_padded(scheme):
    """A step of 16 x 16 x 1000 cells and one of the same cells in a bar of 4 x 4, which a
    column of 32 x 8 would pad sixteen times: less than three times as long."""
    import time
    from paper_2511_20337_amd import mhd
    took = []
    for grid in ((16, 16, 1000), (4, 4, 16000)):
        s = setup(scheme, *grid)
        ctx = mhd.Context(s, "cuda:0")
        U = torch.from_numpy(state(s)).cuda()
        dt = 1e-3 * ctx.dt(U)
        best = 1.0
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(5):
                ctx.step(U, dt)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best)
    print("narrow grid", scheme, took, flush=True)
    assert took[1] < 3 * took[0], took


def test_a_long_grid_costs_the_host_nothing():
    """The launches of a grid of a million planes are chosen in a bounded number of
    steps: the call returns within a millisecond (a search over all numbers of
    runs took the host several)."""
    import time
    from paper_2511_20337_amd import mhd
    s = setup("hll", 4, 4, 1000000, (0, 1, 0, 1, 0, 250000))
    ctx = mhd.Context(s, "cuda:0")
    w = [1.0, 0.3, -0.2, 0.1, 2.0, 0.4, 0.25, -0.15]
    U = torch.empty(ctx.shape, dtype=torch.float64, device="cuda:0")
    for q, v in enumerate(w):
        U[q] = v
    out = torch.empty_like(U)
    best = 1.0
    for _ in range(4):
        ctx.rhs(U, out)
        torch.cuda.synchronize()
        t = time.perf_counter()
        ctx.rhs(U, out)
        best = min(best, time.perf_counter() - t)
        torch.cuda.synchronize()
    ctx.check()
    assert float(out.abs().max()) == 0.0
    assert best < 1e-3, best
