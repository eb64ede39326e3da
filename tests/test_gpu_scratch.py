"""Scratch under a tight budget: what one solve keeps for the next one does not make
another fail that the budget has room for."""
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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_chords_after_packets(torch_dev, precision):
    """One chunk of chord groups after a solve that kept packet records: the
    records give way wherever the chords' arrays stop fitting beside them."""
    from paper_2110_15640_amd import mcrt as M
    grid, table, _ = I.make_emission_3d(32, 16, 20, nband=3, ng=4)
    kw = dict(n_b=32, n_alpha=32, seed=1, r_star=I.R_SUN, precision=M.MCRT_MIXED if precision == "mixed" else M.MCRT_FP64)

    def packets(ctx, gid, oid):
        ctx.solve_emission(gid, oid, table, n_packets=2000, obs_phase=[0.3, 0.6], seed=1)

    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        ref = ctx.solve_transmission(gid, oid, table, **kw)
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        packets(ctx, gid, oid)
        held = ctx.memory_in_use
    for extra in range(0, 6 << 20, 1 << 18):
        print(f"chords after packets: {precision}, {extra} bytes beside the records", flush=True)
        with M.Context(0, hbm_budget_bytes=held + extra) as ctx:
            gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
            packets(ctx, gid, oid)
            got = ctx.solve_transmission(gid, oid, table, **kw)
        assert np.array_equal(got["sums"], ref["sums"]), extra
