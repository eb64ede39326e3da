"""The face table of a one-grid launch lies in LDS where it has at most 1024 entries
(layers + rows + columns + 1): grids on either side of that, as two kernels and as
one, and against the FP64 oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2110_15640_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("shape", [(8, 4, 1011), (8, 4, 1012)])  # 1024 and 1025 entries
@pytest.mark.parametrize("mode,kw", [("emission", dict()), ("albedo", dict()), ("albedo", dict(surface_albedo=0.5))])
def test_face_table_in_lds_and_in_memory(torch_dev, mode, kw, shape):
    print(f"face table: {shape}, {mode} {sorted(kw)}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table, _ = I.make_emission_3d(*shape, nband=1, ng=1)
    args = dict(n_packets=300, seed=4, obs_phase=[0.2, 0.5], **kw)
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        solve = getattr(ctx, "solve_" + mode)
        two, one = solve(gid, oid, table, **args), solve(gid, oid, table, graph=1, **args)
        mixed = [solve(gid, oid, table, precision=M.MCRT_MIXED, graph=g, **args) for g in (0, 1)]
    for a, b in ((two, one), mixed):
        assert np.array_equal(a["sums"], b["sums"]) and np.array_equal(a["counters"], b["counters"])
    p = O.Params(n_packets=300, seed=4, obs_phase=(0.2, 0.5), **kw)
    ref = (O.solve_emission if mode == "emission" else O.solve_albedo)(grid, table, p)
    # paths of thousands of crossings, each good to a few units in the last place
    np.testing.assert_allclose(two["sums"], ref.sums, rtol=1e-9)
    assert np.array_equal(two["counters"][..., 6:10], ref.counters[..., 6:10])
