"""The transport in two kernels (blocking solves) against the one-kernel form
(recorded solves): the same results bit for bit, over the options that either
form treats apart, with launches whose records run out, and on a grid with a
latitude edge within rounding of the equator."""
import numpy as np
import pytest

from paper_2110_15640_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _cloudy(grid, thick):
    k = np.repeat(np.arange(grid.nlay), grid.nlon * grid.nlat) / grid.nlay
    grid.cld_ksca = ((30.0 if thick else 2e-2) * np.exp(-3.0 * k)).astype(np.float32)
    grid.cld_kabs = (1e-3 * np.exp(-3.0 * k)).astype(np.float32)
    grid.cld_g = np.full(grid.nlon * grid.nlat * grid.nlay, 0.6, np.float32)


@pytest.mark.parametrize("mode,shape,n,kw", [
    ("emission", (16, 8, 10), 1, dict()),
    ("emission", (44, 22, 7), 3000, dict(obs_phase=[0.1, 0.5, 0.9])),  # sin of its middle edge is 1e-16
    ("emission", (16, 8, 10), 100000, dict()),
    ("albedo", (16, 8, 10), 20000, dict(thick=True)),                  # hundreds of events a packet: records run out
    ("albedo", (16, 8, 10), 3000, dict(surface_albedo=0.4, cloud_phase=1)),
    ("albedo", (16, 8, 10), 3000, dict(cloud_phase=2, forced=3)),
    ("albedo", (16, 8, 10), 3000, dict(absorption=1)),
    ("emission", (16, 8, 10), 3000, dict(forced=1, forced_first=1)),
    ("emission", (16, 8, 10), 3000, dict(g_sampling=1)),
    ("transmission", (16, 8, 10), 3000, dict(ms_transmission=1, a_orbit=7e11, r_star=I.R_SUN, ld_law=2, ld_c1=0.4,
                                             ld_c2=0.2)),
])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_two_kernels_equal_one(torch_dev, mode, shape, n, kw, precision):
    print(f"split against one kernel: {mode} {shape}, {n} packets, {precision}, {sorted(kw)}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table, phases = I.make_emission_3d(*shape, nband=2, ng=2)
    kw = dict(kw)
    thick = kw.pop("thick", False)
    _cloudy(grid, thick)
    args = dict(n_packets=n, seed=9, precision=M.MCRT_MIXED if precision == "mixed" else M.MCRT_FP64, **kw)
    if mode != "transmission" and "obs_phase" not in args:
        args["obs_phase"] = [0.25, 0.5]
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        solve = getattr(ctx, "solve_" + mode)
        two = solve(gid, oid, table, **args)
        one = solve(gid, oid, table, graph=1, **args)
    if thick:
        assert two["counters"][..., 6].sum() > 16 * 4 * n  # more events than records
    assert np.array_equal(two["sums"], one["sums"])
    assert np.array_equal(two["counters"], one["counters"])
