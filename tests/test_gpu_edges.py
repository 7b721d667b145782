"""GPU parity at the edges of what single kernels and host paths hold: values
that outgrow a narrower type, buffers that change under a queued copy, knobs
and numbers out of the usual range."""
import ctypes

import numpy as np
import pytest

import oracle
import tpcgen
from tests import _parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


@pytest.fixture(scope="module")
def tpcca(torch_cuda):
    from paper_1709_00618_amd import tpcca as m
    m.lib()
    return m


# all at one z and the default bins; any z, bins of 400 hits, and the short rows'
# hits at both ends
@pytest.mark.parametrize("per_bin, z0, z1", [(1, 99.5, 100.5), (400, 0.0, 250.0)])
def test_a_crowded_row_in_a_run_of_sparse_rows(tpcca, row_x, per_bin, z0, z1):
    """The neighbour search by waves is taken by the run's mean row: one row of
    70000 hits, few bins long, beside rows of 50 and 40 (its bins' starts do not
    fit 16 bits), in a run of eight units whose mean row stays sparse."""
    rng = np.random.default_rng(7)
    counts = {0: 2, 10: 50, 11: 40, 12: 70000}
    parts, rows = [], []
    for r, k in counts.items():
        z = np.array([0.0, 250.0]) if r == 0 else rng.uniform(z0 if r == 12 else 0.05 * z0 + 0.95 * z1, z1, k)
        z[0] = z0 if r else 0.0
        parts.append(np.stack([np.full(k, row_x[r]), rng.uniform(-3.0, 3.0, k), z, np.ones(k)], axis=1))
        rows.append(np.full(k, r, np.uint8))
    cl, row = np.concatenate(parts).astype(np.float32), np.concatenate(rows)
    o = rng.permutation(cl.shape[0])
    cl, row = np.ascontiguousarray(cl[o]), np.ascontiguousarray(row[o])
    units = [(cl, row)] + [(cl[k:k + 1], row[k:k + 1]) for k in range(7)]
    assert sum(c.shape[0] for c, _ in units) < 96 * len(units) * (len(row_x) + 1)
    with tpcca.Context(row_x, params=tpcca.params_default(grid_hits_per_bin=per_bin)) as ctx:
        for s, (c, r) in enumerate(units):
            ctx.load_sector(0, s, c, r)
        ctx.run_all(0, -1)
        ctx.sync()
        for s, (c, r) in enumerate(units):
            ref = oracle.run_sector(c, r, row_x)
            assert s or (ref.up_raw >= 0).sum() > 10
            _parity.compare_unit_stagewise(ctx, 0, s, c, r, ref)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("pinned", [False, True])
def test_host_input_may_be_overwritten_after_run_batch(tpcca, torch_cuda, row_x, pinned, graph):
    """A batch's host input has been copied when the call returns, also from pinned
    memory, where the copy itself does not wait: the buffers (17 MB, 0.3 ms of
    copying) are overwritten at once, the row numbers, copied last, first."""
    torch = torch_cuda
    b = tpcgen.central_event(seed=3, keep_truth=False)
    hold = [torch.from_numpy(np.ascontiguousarray(a)) for a in (b.cl, b.row)]
    hold = [torch.empty(t.shape, dtype=t.dtype, pin_memory=pinned) for t in hold]
    cl, row = (t.numpy() for t in hold)
    with tpcca.Context(row_x) as ctx:
        ctx.run_batch(b.cl, b.row, b.units, graph=graph)
        want = [a.tobytes() for a in ctx.get_batch_results()]
        for _ in range(3):
            cl[:], row[:] = b.cl, b.row
            ctx.run_batch(cl, row, b.units, graph=graph)
            row[:] = 255
            cl[:] = np.nan
            assert [a.tobytes() for a in ctx.get_batch_results()] == want


# cluster variances whose determinant leaves 2^-120 .. 2^120 (its reciprocal, too),
# a field of 1e-36, directions of 1e-37, rows 1e-18 apart (no second phase: it
# tells rows by their x)
FAR = [
    dict(err2_y=6e-20, err2_z=6e-20, seed_c22=6e-22, seed_c33=6e-22, seed_c44=6e-19, pick_nsig=1e12, pick_chi2=1e22,
         refit_inflate=1.0),
    dict(err2_y=5e17, err2_z=1e20, seed_c22=1e16, seed_c33=1e17, seed_c44=1e18, pick_nsig=1e-8, pick_chi2=1e-10,
         refit_inflate=1.0),
    dict(err2_y=1e18, err2_z=1e20, seed_c22=1e16, seed_c33=1e17, seed_c44=1e18, pick_nsig=1e-8, pick_chi2=1e-10,
         refit_inflate=1.0),
    dict(kB=1e-36), dict(y=1e-36), dict(y=1e-34, kB=0.0), dict(x=1e-18),
]


@pytest.mark.parametrize("far", FAR)
def test_fits_outside_the_range_of_the_short_quotients(tpcca, row_x, far):
    """Every fit form and the compression where quotients and roots leave the range
    in which their short forms are exact, against the oracle."""
    b = tpcgen.one_sector(seed=21)
    cl, row, slot, sec, _ = b.unit(0)
    over = {k: v for k, v in far.items() if k not in "xy"}
    rx = (row_x * np.float32(far.get("x", 1.0))).astype(np.float32)
    cl = cl.copy()
    cl[:, 1] *= np.float32(far.get("y", 1.0))
    cl[:, 1:3] *= np.float32(far.get("x", 1.0))
    cl[:, 0] = rx[row]
    params = oracle.default_params(**over)
    ref = oracle.run_sector(cl, row, rx, params)
    assert ref.n_tracks >= 20
    seg, hb, hits = oracle.segments_of([ref])
    rec, res = oracle.compress(cl, row, rx, seg, hb, hits, params=params)
    for knobs in ({}, {"fit_xcd_slices": 1}, {"fit_rows": 256}):
        with tpcca.Context(rx, params=tpcca.params_default(**over)) as ctx:
            ctx.set_tuning(**knobs)
            ctx.load_sector(slot, sec, cl, row)
            ctx.run_all()
            ctx.sync()
            _parity.compare_unit_stagewise(ctx, slot, sec, cl, row, ref)
            if "x" in far:
                continue
            ctx.phase2()
            grec, gres = ctx.get_compressed(slot, sec)
        assert np.array_equal(grec, rec) and np.array_equal(gres, res)


class KernelNode(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("args", ctypes.POINTER(ctypes.c_void_p)), ("shared", ctypes.c_uint32)]


def _launches(tpcca, stream, call, look=None):
    """The kernels that `call` queues on the stream, captured in a graph and not run:
    (function, grid) each, or what `look` makes of their nodes."""
    hip = tpcca.lib()  # the runtime that the library is linked to
    vp = ctypes.c_void_p
    graph = vp()
    assert hip.hipStreamBeginCapture(vp(stream), 2) == 0  # relaxed: the test is the only user
    try:
        call()
    finally:
        assert hip.hipStreamEndCapture(vp(stream), ctypes.byref(graph)) == 0
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (vp * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        k = KernelNode()
        assert hip.hipGraphKernelNodeGetParams(vp(node), ctypes.byref(k)) == 0
        out.append(look(k) if look else (k.func, tuple(k.grid)))
    assert hip.hipGraphDestroy(graph) == 0
    return out


@pytest.mark.parametrize("per_cu, grid", [(0, 1456), (1, 256), (3, 768), (32, 1456)])
def test_link_blocks_per_cu_holds_for_sparse_rows(tpcca, torch_cuda, row_x, per_cu, grid):
    """The resident blocks per CU that were asked for, also in the neighbour search by
    waves: 36 short units (161 tile slots each, four to a block of the default)."""
    stream = torch_cuda.cuda.Stream().cuda_stream
    b = tpcgen.one_sector(seed=2)
    with tpcca.Context(row_x, stream=stream) as ctx:
        ctx.set_tuning(link_blocks_per_cu=per_cu)
        for slot in (0, 1):
            for s in range(36):
                ctx.load_sector(slot, s, b.cl[:100], b.row[:100])
        ctx.find_links(0)
        ctx.sync()
        assert _launches(tpcca, stream, lambda: ctx.find_links(1))[-1][1] == (grid, 1, 1)


@pytest.mark.parametrize("knobs", [dict(fit_long_first=60), dict(fit_row_bands=4), dict(fit_rows=256)])
def test_order_knobs_clean_once(tpcca, torch_cuda, row_x, knobs):
    """With a knob that orders the fit otherwise, short units' chains go by the lists of
    the cleaning: these are made there, and the chains do not clean again."""
    stream = torch_cuda.cuda.Stream().cuda_stream
    b = tpcgen.one_sector(seed=2)
    with tpcca.Context(row_x, stream=stream) as ctx:
        ctx.load_sector(0, 0, b.cl, b.row)
        ctx.find_links()
        ctx.sync()
        ctx.set_tuning(**knobs)
        clean = _launches(tpcca, stream, ctx.clean_links)[0][0]
        assert clean not in [f for f, _ in _launches(tpcca, stream, ctx.build_tracklets)]


def test_buffers_that_grow_between_the_cleaning_and_the_chains(tpcca, row_x):
    """A unit cleaned by lists (more than 40960 hits) keeps them when the next load
    makes the work buffers grow before its chains are built."""
    big = tpcgen.central_event(seed=8, n_tracks=12500, keep_truth=False)
    units = [big.unit(u)[:2] for u in (4, 5, 6)]
    assert units[0][0].shape[0] > 40960
    with tpcca.Context(row_x) as ctx:
        ctx.load_sector(0, 0, *units[0])
        ctx.find_links()
        ctx.clean_links()
        for slot in (1, 2):
            ctx.load_sector(slot, 0, *units[slot])
        for slot in (1, 2):
            ctx.find_links(slot)
        ctx.build_tracklets(0)
        for slot in (1, 2):
            ctx.clean_links(slot)
            ctx.build_tracklets(slot)
        ctx.select_tracks()
        ctx.sync()
        for slot, (cl, row) in enumerate(units):
            _parity.compare_unit_stagewise(ctx, slot, 0, cl, row, oracle.run_sector(cl, row, row_x))


@pytest.mark.parametrize("n_seg, waves, per", [(1, 1, 1), (65537, 1024, 65), (2 ** 31 - 4096, 4096, 1024),
                                               (2 ** 31 - 1, 4096, 1024)])
def test_decompression_split_up_to_the_largest_count(tpcca, torch_cuda, row_x, n_seg, waves, per):
    """Waves and segments of a set, from the captured launch (nothing is run)."""
    stream = torch_cuda.cuda.Stream().cuda_stream
    with tpcca.Context(row_x, stream=stream) as ctx:
        got = _launches(tpcca, stream, lambda: ctx.decompress(n_seg, *[4096] * 7),
                        lambda k: (k.grid[0], ctypes.cast(k.args[5], ctypes.POINTER(ctypes.c_int32))[0]))
    assert got == [(waves, per)]
