"""Transmission by groups of 8 x 2 chords and blocks of 64 spectral rows, where
those divide nothing evenly, against the FP64 oracle; and in batches."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_15640_amd import inputs as I

pytestmark = pytest.mark.gpu

# An optical depth sums at most a few hundred products, each good to some 60
# units in the last place (the exponential of an interpolated ln kappa of
# magnitude 60): 1e-14, and ten times that for the sums of squares.
RTOL = 1e-12


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("nlon,nlat,nlay,n_b,n_alpha,nrow", [
    (8, 4, 5, 1, 1, 1),       # one chord of a group
    (10, 6, 7, 8, 2, 16),     # one whole group; a cell across the terminator; 16 rows
    (16, 8, 9, 9, 3, 17),     # one impact parameter and one angle over; 17 rows
    (8, 4, 100, 17, 5, 33),   # chords of more steps than are grouped at a time; 33 rows
    (24, 12, 10, 70, 9, 65),  # more than one chunk of the tallies; one row in a second block
])
@pytest.mark.parametrize("kind", ["ck", "hires"])
def test_ragged_groups_and_rows(torch_dev, kind, nlon, nlat, nlay, n_b, n_alpha, nrow):
    print(f"transmission groups: {kind} {nlon}x{nlat}x{nlay}, {n_b} x {n_alpha} chords, {nrow} rows", flush=True)
    from paper_2110_15640_amd import mcrt as M
    if kind == "ck":
        grid, table, _ = I.make_emission_3d(nlon, nlat, nlay, nband=nrow, ng=1)
    else:
        grid, table = I.make_transmission_hires(nlon, nlat, nlay, nlam=nrow, nT=5, nP=6)
    kw = dict(n_b=n_b, n_alpha=n_alpha, seed=5, r_star=I.R_SUN)
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        got = ctx.solve_transmission(gid, oid, table, **kw)
        mix = ctx.solve_transmission(gid, oid, table, precision=M.MCRT_MIXED, **kw)
    ref = O.solve_transmission(grid, table, O.Params(**kw))
    np.testing.assert_allclose(got["sums"], ref.sums, rtol=RTOL)
    # FP32 tables, extinction and lengths: ln kappa of magnitude 60 rounds to
    # 4e-6, and so does kappa
    np.testing.assert_allclose(mix["sums"][..., 0], ref.sums[..., 0], rtol=2e-5)
    assert got["n_segments"] == mix["n_segments"] > 0


@pytest.mark.parametrize("kind", ["ck", "hires"])
def test_batches_of_groups_change_nothing(torch_dev, kind):
    """A budget that the scratch of all groups does not fit in."""
    print(f"transmission groups in batches: {kind}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    if kind == "ck":
        grid, table, _ = I.make_emission_3d(16, 8, 10, nband=35, ng=2)
    else:
        grid, table = I.make_transmission_hires(16, 8, 10, nlam=70, nT=5, nP=6)
    kw = dict(n_b=64, n_alpha=80, seed=6, r_star=I.R_SUN)
    res = []
    for budget in (0, 24 << 20):
        with M.Context(0, hbm_budget_bytes=budget) as ctx:
            gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
            res.append((ctx.solve_transmission(gid, oid, table, **kw), ctx.memory_in_use))
    (ref, held), (got, held_small) = res
    assert held_small < held  # fewer groups at a time
    assert np.array_equal(got["sums"], ref["sums"]) and got["n_segments"] == ref["n_segments"]
