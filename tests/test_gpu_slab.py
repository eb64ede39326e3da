"""Scattered light of slabs by tabulated optical depths, against the FP64 oracle,
which walks them layer by layer: edge sizes, empty layers, observers in and
below the horizon, rays beyond tau_peel_max, and each place of the tables."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_15640_amd import inputs as I

pytestmark = pytest.mark.gpu

# A packet's depth after n events is good to n times the rounding of a sum of
# nlay terms: 1e3 x 150 x 1.1e-16 = 2e-11, and a contribution e^-t with t <= 50
# to 50 times that.
RTOL = 1e-9


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _dirs(mus):
    return np.array([[np.sqrt(1.0 - m * m), 0.0, m] for m in mus])


@pytest.mark.parametrize("nlay,nlam,n,k_abs,kw", [
    (1, 1, 1, 1e-2, dict()),                                                      # one packet, one layer
    (2, 3, 65, 1e-3, dict(mu0=0.7)),                                              # one over a wave
    (50, 2, 3000, 1e-5, dict(tau_peel_max=2.0)),                                  # dark rays, many events
    (64, 8, 300, 1e-3, dict(obs_dir=_dirs([1.0, 0.3, 1e-3, 0.0, -0.5]))),         # 512 entries: every table in LDS
    (73, 8, 300, 1e-3, dict(cloud_phase=1, obs_dir=_dirs([0.9, 0.2]))),           # 584: depths alone
    (150, 14, 200, 1e-3, dict(mu0=0.5)),                                          # 2100: none
])
@pytest.mark.parametrize("clouds", [False, True])
def test_slab_against_walk(torch_dev, nlay, nlam, n, k_abs, kw, clouds):
    print(f"slab: {nlay} layers, {nlam} wavelengths x {n} packets, clouds {clouds}, {sorted(kw)}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table = I.make_albedo_slab(nlay=nlay, nlam=nlam, k_abs=k_abs)
    if nlay > 2:  # empty layers: at the top, in the middle and at the bottom
        grid.rho[[0, nlay // 2, nlay - 1]] = 0.0
    if clouds:
        k = np.arange(nlay) / nlay
        grid.cld_ksca = (2e-2 * np.exp(-3.0 * k)).astype(np.float32)
        grid.cld_kabs = (1e-3 * np.exp(-3.0 * k)).astype(np.float32)
        grid.cld_g = np.linspace(0.1, 0.8, nlay).astype(np.float32)
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        got = ctx.solve_albedo(gid, oid, table, n_packets=n, seed=7, **kw)
        rec = ctx.solve_albedo(gid, oid, table, n_packets=n, seed=7, graph=1, **kw)
        srv = ctx.wait(ctx.submit("albedo", gid, oid, table, n_packets=n, seed=7, **kw))
        mix = ctx.solve_albedo(gid, oid, table, n_packets=n, seed=7, precision=M.MCRT_MIXED, **kw)
    ref = O.solve_albedo(grid, table, O.Params(n_packets=n, seed=7, **kw))
    np.testing.assert_allclose(got["sums"], ref.sums, rtol=RTOL, atol=1e-300)
    np.testing.assert_allclose(got["counters"], ref.counters, rtol=RTOL, atol=1e-12 * n)
    # events, crossings, capped and lost packets are counts
    assert np.array_equal(got["counters"][..., 6:10], ref.counters[..., 6:10])
    for other in (rec, srv):
        assert np.array_equal(other["sums"], got["sums"]) and np.array_equal(other["counters"], got["counters"])
    if n > 1:  # (one packet has no standard error)
        assert np.all(np.abs(mix["value"] - got["value"]) <= 5.0 * np.hypot(mix["stderr"], got["stderr"]) + 1e-12)
