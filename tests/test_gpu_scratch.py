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


@pytest.mark.parametrize("kind,shape,nrow,n_b,n_alpha", [
    ("ck", (32, 16, 20), 12, 1, 1),        # one group
    ("ck", (32, 16, 20), 12, 7, 31),       # 16 groups, less than a chunk of the tallies
    ("ck", (32, 16, 20), 12, 32, 32),      # one chunk
    ("ck", (16, 8, 10), 130, 33, 41),      # two chunks; three blocks of rows on two streams
    ("hires", (16, 8, 10), 70, 33, 41),
    ("ck", (128, 64, 40), 2, 32, 32),      # most of it the segments
])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_chords_in_little_scratch(torch_dev, kind, shape, nrow, n_b, n_alpha, precision):
    """Raytrace transmission in as much scratch as the extinction of all cells for
    up to 64 rows (for two streams where there are more) and 12 bytes a segment
    take, and in less as long as it fits: the same sums bit for bit."""
    from paper_2110_15640_amd import mcrt as M
    if kind == "ck":
        grid, table, _ = I.make_emission_3d(*shape, nband=nrow, ng=1)
    else:
        grid, table = I.make_transmission_hires(*shape, nlam=nrow, nT=5, nP=6)
    kw = dict(n_b=n_b, n_alpha=n_alpha, seed=3, r_star=I.R_SUN, precision=M.MCRT_MIXED if precision == "mixed" else M.MCRT_FP64)
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        resident = ctx.memory_in_use
        ref = ctx.solve_transmission(gid, oid, table, **kw)
    most = shape[0] * shape[1] * shape[2] * min(nrow, 64) * (2 if nrow > 64 else 1) * 8 + 12 * ref["n_segments"] + \
        24 * n_b * n_alpha + (1 << 16)
    for q in range(8):
        extra = int(most * 0.7 ** q)
        print(f"chords in little scratch: {kind} {shape}, {nrow} rows, {n_b} x {n_alpha}, {precision}, {extra} bytes", flush=True)
        with M.Context(0, hbm_budget_bytes=resident + extra) as ctx:
            gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
            try:
                got = ctx.solve_transmission(gid, oid, table, **kw)
            except M.McrtError as e:
                assert e.name == "EBUDGET" and q > 0, (e, extra)
                break
            assert ctx.memory_in_use <= resident + extra
        assert np.array_equal(got["sums"], ref["sums"]) and got["n_segments"] == ref["n_segments"], extra


def _needs(grid, table, mode="transmission", **kw):
    """What a served request says it needs, where the budget has nothing left."""
    from paper_2110_15640_amd import mcrt as M
    with M.Context(0) as ctx:
        ctx.upload_grid(grid), ctx.upload_opacity(table)
        resident = ctx.memory_in_use
    with M.Context(0, hbm_budget_bytes=resident) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        with pytest.raises(M.McrtError) as e:
            ctx.submit(mode, gid, oid, table, **kw)
    assert e.value.name == "EBUDGET"
    return resident, int(str(e.value).split("needs ")[1].split()[0])


@pytest.mark.parametrize("kind,shape,nrow,n_b,n_alpha", [
    ("hires", (16, 8, 10), 20000, 64, 80),  # 3 MB of chunk sums if all rows are taken at once
    ("ck", (32, 16, 20), 12, 100, 90),
    ("ck", (128, 64, 40), 2, 3, 5),
])
def test_served_chords_stay_in_what_they_were_admitted_with(torch_dev, kind, shape, nrow, n_b, n_alpha):
    print(f"served chords and their scratch: {kind} {shape}, {nrow} rows, {n_b} x {n_alpha}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    if kind == "ck":
        grid, table, _ = I.make_emission_3d(*shape, nband=nrow, ng=1)
    else:
        grid, table = I.make_transmission_hires(*shape, nlam=nrow, nT=5, nP=6)
    kw = dict(n_b=n_b, n_alpha=n_alpha, seed=3, r_star=I.R_SUN)
    resident, est = _needs(grid, table, **kw)
    ncell, nch, nslot = int(np.prod(shape)), n_b * n_alpha, min(nrow, 64)
    # extinction of the cells, their places in the table, the most segments that
    # chords can have, sums and chunks, 1 MB of small arrays
    assert est <= ncell * (8 * nslot + 40) + nch * (24 + 12 * (2 * shape[2] + 2 * shape[1] + shape[0] + 8)) + \
        (nch + 31) // 32 * 16 * nslot + 20 * nrow + (1 << 20) + 8
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        ref = ctx.solve_transmission(gid, oid, table, **kw)
    with M.Context(0, hbm_budget_bytes=resident + est) as ctx:
        ctx.serve_config(1)
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        ticket = ctx.submit("transmission", gid, oid, table, **kw)
        peak = 0
        while not ctx.poll(ticket):
            peak = max(peak, ctx.memory_in_use)
        got = ctx.wait(ticket)
    assert peak <= resident + est
    assert np.array_equal(got["sums"], ref["sums"]) and got["n_segments"] == ref["n_segments"]


def test_served_chords_take_one_batch_where_there_is_room(torch_dev):
    """Launches of the optical depths of a served transmission: with the whole
    device for it one per block of 64 rows, as in a blocking solve; admitted with
    no more than it must have, more, and the same sums."""
    print("served chords in one batch", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table = I.make_transmission_hires(16, 8, 10, nlam=20000, nT=5, nP=6)
    kw = dict(n_b=64, n_alpha=80, seed=3, r_star=I.R_SUN, profile=1)
    resident, est = _needs(grid, table, **kw)
    res = []
    for budget in (0, resident + est):
        with M.Context(0, hbm_budget_bytes=budget) as ctx:
            ctx.serve_config(1)
            gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
            res.append(ctx.wait(ctx.submit("transmission", gid, oid, table, **kw)))
            if budget == 0:
                res.append(ctx.solve_transmission(gid, oid, table, **kw))
    served, blocking, tight = res
    assert served["kernel_launches"] == blocking["kernel_launches"] == 313
    assert tight["kernel_launches"] > 313
    assert np.array_equal(served["sums"], blocking["sums"]) and np.array_equal(tight["sums"], blocking["sums"])


def test_batch_launches_do_not_depend_on_kept_records(torch_dev):
    """A batch that one launch holds in half of the budget's room, in a fresh
    context and after a solve that kept packet records."""
    print("batch after packets: launches", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table, _ = I.make_emission_3d(16, 8, 10, nband=30, ng=1)
    args = dict(obs_phase=[0.3, 0.6], seed=1)
    res = []
    with M.Context(0) as ctx:
        ctx.upload_grid(grid), ctx.upload_opacity(table)
        resident = ctx.memory_in_use
    for packets_first in (False, True):
        with M.Context(0, hbm_budget_bytes=resident + (400 << 20)) as ctx:
            gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
            if packets_first:
                ctx.solve_emission(gid, oid, table, n_packets=2000, spec_idx=[0, 1], **args)
                assert ctx.memory_in_use > resident + (50 << 20)
            item = dict(mode="emission", gid=gid, oid=oid, table=table, n_packets=20000)
            res.append(ctx.solve_batch([item] * 3, profile=1, **args))  # 90 solves of 2.15 MB
    assert res[0][0]["kernel_launches"] == res[1][0]["kernel_launches"] == 1
    for a, b in zip(*res):
        assert np.array_equal(a["sums"], b["sums"])


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("room_mb,n", [(120, 4000), (800, 30000)])  # records of 91 MB and 480 MB
def test_packet_solves_leave_half_of_the_room(torch_dev, batched, room_mb, n):
    """Packet solves hold at most half of what the budget leaves (and their
    tallies), records included, so that uploads and served requests find room
    while one runs; the sums do not depend on it."""
    print(f"packets in half of {room_mb} MB, batched {batched}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table, _ = I.make_emission_3d(16, 8, 10, nband=8, ng=1)
    args = dict(obs_phase=[0.3, 0.6], seed=1)

    def solve(ctx):
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        held = ctx.memory_in_use
        if batched:
            out = ctx.solve_batch([dict(mode="emission", gid=gid, oid=oid, table=table, n_packets=n)], **args)[0]
        else:
            out = ctx.solve_emission(gid, oid, table, n_packets=n, **args)
        return held, ctx.memory_in_use - held, out

    with M.Context(0) as ctx:
        resident, _, ref = solve(ctx)
    with M.Context(0, hbm_budget_bytes=resident + (room_mb << 20)) as ctx:
        _, kept, out = solve(ctx)
    tallies = 8 * 20 * 8 * (2 + n // 4096) + (1 << 20)
    assert kept <= (room_mb << 19) + tallies
    assert np.array_equal(out["sums"], ref["sums"])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_served_packets_need_what_they_did(torch_dev, precision):
    """Admission of a served emission request: optics (and their FP32 copies),
    sources, packet rows, tallies, solve tables, scan scratch, and 1 MB in which
    the small arrays lie; what it then holds is no more."""
    print(f"served packets and their scratch: {precision}", flush=True)
    from paper_2110_15640_amd import mcrt as M
    grid, table, _ = I.make_emission_3d(16, 8, 10, nband=3, ng=2)
    n, ncell, ns, no = 5000, 1280, 6, 1
    mixed = precision == "mixed"
    kw = dict(n_packets=n, obs_phase=[0.3], seed=2, max_batch=1, precision=M.MCRT_MIXED if mixed else M.MCRT_FP64)
    resident, est = _needs(grid, table, mode="emission", **kw)
    arrays = ncell * (40 + (20 if mixed else 0) + 16) + n * (no + 11) * 8 + ns * (2 * no + 13) * 8 + \
        -(-n // 4096) * (2 * no + 11) * 8
    tables = 256 + 64  # 160 and 72 bytes a solve
    scan = 8 * (2 * -(-ncell // 256) + -(-ncell // 2048) + 16)
    assert arrays < est <= arrays + tables + scan + (1 << 20)
    with M.Context(0) as ctx:
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        ref = ctx.solve_emission(gid, oid, table, **kw)
    with M.Context(0, hbm_budget_bytes=resident + est) as ctx:
        ctx.serve_config(1)
        gid, oid = ctx.upload_grid(grid), ctx.upload_opacity(table)
        ticket, peak = ctx.submit("emission", gid, oid, table, **kw), 0
        while not ctx.poll(ticket):
            peak = max(peak, ctx.memory_in_use)
        assert np.array_equal(ctx.wait(ticket)["sums"], ref["sums"])
    assert peak <= resident + est
