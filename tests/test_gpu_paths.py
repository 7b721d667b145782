"""GPU parity of single paths of the host runtime and of kernel variants, at
the sizes where they switch."""
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


def _first(b, n):
    """The first n clusters of a one-unit batch."""
    return np.ascontiguousarray(b.cl[:n]), np.ascontiguousarray(b.row[:n])


def test_host_loads_whose_row_buffer_grows_alone(tpcca, row_x):
    """Host units loaded one by one: the staging buffers of clusters (16 B each)
    and of rows (1 B) grow at different totals (buffers grow by a quarter,
    in steps of 256 B), and with these sizes the fourth load moves the rows
    alone; the earlier units then have to read the moved rows."""
    b = tpcgen.one_sector(seed=11)
    sizes = (1000, 100, 170, 30)
    cap_cl, cap_row, tot, alone = 0, 0, 0, []
    for n in sizes:  # the buffers' growth as the library does it
        tot += n
        moved = [16 * tot > cap_cl, tot > cap_row]
        if moved[0]:
            cap_cl = (max(16 * tot, cap_cl + cap_cl // 4) + 255) & ~255
        if moved[1]:
            cap_row = (max(tot, cap_row + cap_row // 4) + 255) & ~255
        alone.append(moved == [False, True])
    assert alone[-1]
    with tpcca.Context(row_x) as ctx:
        for s, n in enumerate(sizes):
            ctx.load_sector(0, s, *_first(b, n))
        ctx.run_all(0, -1)
        ctx.sync()
        for s, n in enumerate(sizes):
            cl, row = _first(b, n)
            _parity.compare_unit_stagewise(ctx, 0, s, cl, row, oracle.run_sector(cl, row, row_x))


FIT_FORMS = [
    dict(),                                     # the loops: one tracklet per wave up to 2048, then several lanes
    dict(fit_xcd_slices=1),                     # the state machine (never the loops), claims from eight counters
    dict(fit_block=64, fit_blocks_per_cu=1),    # 256 waves: a wave's share exceeds its 64 lanes
    dict(fit_block=256, fit_min_waves=5),       # the largest block
    dict(fit_pool=200, fit_xcd_slices=1),       # claims longer than the tracklets read ahead
    dict(fit_claims=0),                         # claims in a kernel of their own
]


@pytest.mark.parametrize("tracks, sectors", [(12, 1), (700, 3), (8000, 4), (8000, 36)])
def test_fit_forms_against_the_oracle(tpcca, torch_cuda, row_x, tracks, sectors):
    """Both forms of the fit kernel (loops for few tracklets, state machine for
    many) at tracklet counts below and above a wave each, with every block size,
    against the oracle: tracklets, tracks, assignment."""
    torch = torch_cuda
    ev = tpcgen.central_event(seed=5, n_tracks=tracks, keep_truth=False)
    parts = [ev.unit(u) for u in range(sectors)]
    off = np.cumsum([0] + [p[0].shape[0] for p in parts])
    units = np.array([(off[i], parts[i][0].shape[0], parts[i][2], parts[i][3]) for i in range(sectors)], np.int64)
    b = tpcgen.Batch(np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts]), units)
    refs = _parity.oracle_units(b, row_x)
    print(f"{tracks} tracks, {sectors} sectors: {b.n_clusters} clusters, "
          f"{sum(r.tracklets.shape[0] for r in refs)} tracklets", flush=True)
    dcl, drow = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (b.cl, b.row))
    torch.cuda.synchronize()
    for knobs in FIT_FORMS:
        with tpcca.Context(row_x) as ctx:
            ctx.set_tuning(**knobs)
            ctx.run_batch(dcl, drow, units, device=True)
            ctx.sync()
            for u in range(sectors):
                cl, row, slot, sec, _ = b.unit(u)
                _parity.compare_unit_stagewise(ctx, slot, sec, cl, row, refs[u])
            w = ctx.work_stats()
            assert w["fit_steps"] == sum(r.work["propagations"] for r in refs)
            assert w["fit_tests"] == sum(r.work["tests"] for r in refs)
            assert w["fit_updates"] == sum(r.work["updates"] for r in refs)


def _unit_of_rows(row_x, counts, seed, z_of=None):
    """A unit with counts[r] hits in row r, at random y and z (z_of: rows whose
    hits lie at almost one z, so that a lot of 64 hits has them all as neighbours)."""
    rng = np.random.default_rng(seed)
    parts, rows = [], []
    for r, k in enumerate(counts):
        z = 10.0 + rng.uniform(-0.05, 0.05, k) if z_of and r in z_of else rng.uniform(0.0, 250.0, k)
        parts.append(np.stack([np.full(k, row_x[r]), rng.uniform(-0.13, 0.13, k) * row_x[r], z, np.ones(k)], axis=1))
        rows.append(np.full(k, r, np.uint8))
    cl, row = np.concatenate(parts).astype(np.float32), np.concatenate(rows)
    o = rng.permutation(cl.shape[0])
    return np.ascontiguousarray(cl[o]), np.ascontiguousarray(row[o])


# hits in every row: the classes of mean row length (lines at 96, 300 and 1024), then
# single rows around a wave's lanes, a tile and the longest row that a wave sorts
@pytest.mark.parametrize("base", [2, 94, 97, 298, 303])
def test_rows_around_the_wave_and_block_forms(tpcca, row_x, base):
    """Row sort and neighbour search, by waves and by blocks, at row lengths around
    their edges, two units in one run."""
    R = len(row_x)
    counts = np.full(R, base)
    if base == 2:
        special = [0, 1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 700]
        counts[10:10 + 2 * len(special):2] = special
        counts[11:11 + 2 * len(special):2] = special[::-1]
        counts[60:63], counts[70:73], counts[80:83] = (255, 300, 256), (257, 20, 258), (600, 64, 40)
    units = [_unit_of_rows(row_x, counts, 1, {60, 61, 62, 70, 71, 72, 80, 81, 82}),
             _unit_of_rows(row_x, np.full(R, base), 2)]
    with tpcca.Context(row_x) as ctx:
        for s, (cl, row) in enumerate(units):
            ctx.load_sector(0, s, cl, row)
        ctx.run_all(0, -1)
        ctx.sync()
        for s, (cl, row) in enumerate(units):
            print(f"base {base}: unit {s}, {cl.shape[0]} hits", flush=True)
            _parity.compare_unit_stagewise(ctx, 0, s, cl, row, oracle.run_sector(cl, row, row_x))


def test_results_of_units_in_any_order(tpcca, torch_cuda, row_x):
    """Copies of units that lie one after the other are joined: units loaded in
    another order (reversed, two slots in turn, one left out, one empty) give the
    same results per unit and per slot, from the batch, the finals and a server."""
    from paper_1709_00618_amd import serving
    b = tpcgen.minbias_batch(seed=9, n_events=2)
    some = [u for u in range(72) if u % 36 < 12 and u != 5]
    turn = [u for s in range(12) for u in (s, 36 + s) if u != 5]

    def run(order):
        units = np.array([b.units[u] for u in order], np.int64)
        units[order.index(7), 1] = 0
        with tpcca.Context(row_x) as ctx:
            ctx.run_batch(b.cl, b.row, units, device=False)
            res, tracks, hits, asg = ctx.get_batch_results()
            per, off = {}, 0
            for k, u in enumerate(order):
                t0, h0, nt, nh = (int(res[k][f]) for f in ("track_begin", "hit_begin", "n_tracks", "n_track_hits"))
                n = int(units[k, 1])
                per[u] = (tracks[t0:t0 + nt].tobytes(), hits[h0:h0 + nh].tobytes(), asg[off:off + n].tobytes())
                off += n
            ctx.phase2()
            finals = [tuple(a.tobytes() for a in ctx.get_finals(slot)) for slot in (0, 1)]
        frame = [k for k, u in enumerate(order) if u < 36]
        f = serving.Frame(b.cl, b.row, units[frame])
        o = serving.Outputs(f.n_clusters, f.n_units)
        with serving.Server(row_x, n_streams=1, budget_bytes=2 << 30) as srv:
            rid = srv.submit(f, o)
            assert srv.wait(rid, 100).status == tpcca.OK
            served = {}
            for k, (t, h, a) in zip(frame, serving.unit_results(f, o)):
                served[order[k]] = (t.tobytes(), h.tobytes(), a.tobytes())
            srv.release(rid)
        return per, finals, served

    per, finals, served = run(some)
    assert sum(len(p[0]) > 0 for p in per.values()) > 15 and len(finals[0][0]) and len(finals[1][0])
    for u, p in served.items():
        assert p == per[u]
    for order in (some[::-1], turn, turn[::-1]):
        p2, f2, s2 = run(order)
        assert p2 == per and s2 == served
        if order is turn:
            assert f2 == finals


# hits of the largest unit: chains in LDS (up to 8192, up to 40960 hits), else by lists
@pytest.mark.parametrize("n", [1, 2, 31, 33, 8191, 8192, 8193, 40959, 40960, 40961])
def test_chains_around_the_lds_unit_sizes(tpcca, torch_cuda, row_x, n):
    """Tracklet numbers, fit order and results with units at the sizes where the
    chain kernels change, beside an empty unit, one cluster and a short unit; then
    with an order knob set between the cleaning and the chains."""
    big = tpcgen.central_event(seed=8, n_tracks=12500, keep_truth=False)
    cl, row, _, _, _ = big.unit(4)
    assert cl.shape[0] > 40961
    parts = [(np.ascontiguousarray(cl[:k]), np.ascontiguousarray(row[:k])) for k in (700, n, 0, 1)]
    refs = [oracle.run_sector(c, r, row_x) for c, r in parts]
    for knobs in ({}, {"fit_long_first": 60}):
        with tpcca.Context(row_x) as ctx:
            for s, (c, r) in enumerate(parts):
                ctx.load_sector(0, s, c, r)
            ctx.find_links()
            ctx.clean_links()
            ctx.set_tuning(**knobs)
            ctx.build_tracklets()
            ctx.select_tracks()
            ctx.sync()
            for s, (c, r) in enumerate(parts):
                _parity.compare_unit_stagewise(ctx, 0, s, c, r, refs[s])



@pytest.fixture(scope="module")
def stored(tpcca, row_x):
    """Compressed segments of a sector, cut to lengths from 0 hits on, and what the
    oracle reads back of them."""
    b = tpcgen.one_sector(seed=12)
    cl, row, slot, sec, _ = b.unit(0)
    with tpcca.Context(row_x) as ctx:
        ctx.load_sector(slot, sec, cl, row)
        ctx.run_all()
        nh = ctx.get_tracks(slot, sec)[0]["n_hits"].astype(np.int32)
        ctx.phase2()
        rec, res = ctx.get_compressed(slot, sec)
    begin = np.cumsum(nh) - nh
    return rec, [res[o:o + k] for o, k in zip(begin, nh)], oracle.decompress(row_x, nh, rec, res)


# the sets of a wave: 64 segments and fewer, then up to a wave per SIMD, to four, and beyond a set's room
@pytest.mark.parametrize("n_seg", [1, 63, 65, 65536, 65537, 524288, 4194304 + 7])
def test_decompression_of_any_number_of_segments(tpcca, torch_cuda, row_x, stored, n_seg):
    """Segments of 0 to 159 hits in any order, with gaps between their hits; one
    of them turns to a row that is not there and ends before it."""
    torch = torch_cuda
    rec, res, (y, z, r) = stored
    first = np.cumsum([0] + [len(x) for x in res])
    rng = np.random.default_rng(n_seg)
    cut = [(u, k) for u in range(len(res)) for k in ((0, 1, 2, len(res[u])) if n_seg < 100000 else (0, 1, 2, 9))]
    pick = rng.integers(0, len(cut), n_seg)
    unit, n = np.array(cut, np.int32).T[:, pick]
    begin = np.cumsum(np.maximum(n, 1) + rng.integers(0, 2, n_seg)) - np.maximum(n, 1)  # the first is written of 0, too
    total = int(begin[-1] + max(1, n[-1]) + 1)
    at = np.repeat(begin - (np.cumsum(np.maximum(n, 1)) - np.maximum(n, 1)), np.maximum(n, 1)) + np.arange(
        np.maximum(n, 1).sum())
    src = np.repeat(first[unit] - (np.cumsum(np.maximum(n, 1)) - np.maximum(n, 1)), np.maximum(n, 1)) + np.arange(
        np.maximum(n, 1).sum())
    all_res = np.zeros((total, 4), np.int32)
    all_res[at, :3] = np.concatenate(res)[src]
    want = [np.full(total, -5, np.int32), np.full(total, -6, np.int32), np.full(total, 255, np.uint8)]
    for w, v in zip(want, (y, z, r)):
        w[at] = v[src]
    bad = int(np.argmax(n))
    if n[bad] > 2:
        all_res[begin[bad] + 2, 0] = 1000
        for w, v in zip(want, (-5, -6, 255)):
            w[begin[bad] + 2:begin[bad] + n[bad]] = v
    print(f"{n_seg} segments, {len(at)} hits", flush=True)
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (n, begin.astype(np.int64), rec[unit], all_res)]
    out = [torch.full((total,), v, dtype=t, device="cuda")
           for v, t in ((-5, torch.int32), (-6, torch.int32), (255, torch.uint8))]
    torch.cuda.synchronize()
    with tpcca.Context(row_x) as ctx:
        ctx.decompress(n_seg, *d, *out)
        ctx.sync()
    for o, w in zip(out, want):
        assert np.array_equal(o.cpu().numpy(), w)


@pytest.mark.parametrize("qy, qz", [(0.01, 0.01), (0.037, 2.0 ** -60), (2.0 ** 60, 0.3), (1e-20, 0.01), (0.01, 1e22)])
def test_compression_steps_inside_and_outside_the_shared_reciprocals(tpcca, row_x, qy, qz):
    """Quantisation steps where the quotients share a reciprocal and where they are
    divisions; segments of every length, the last wave partly filled."""
    b = tpcgen.one_sector(seed=13)
    cl, row, slot, sec, _ = b.unit(0)
    seg, hb, hits = oracle.segments_of([oracle.run_sector(cl, row, row_x)])
    rec, res = oracle.compress(cl, row, row_x, seg, hb, hits, p2=oracle.default_p2params(cmp_qy=qy, cmp_qz=qz))
    assert seg.shape[0] % 64
    with tpcca.Context(row_x) as ctx:
        ctx.load_sector(slot, sec, cl, row)
        ctx.run_all()
        ctx.set_phase2_params(cmp_qy=qy, cmp_qz=qz)
        ctx.phase2()
        grec, gres = ctx.get_compressed(slot, sec)
    assert np.array_equal(grec, rec) and np.array_equal(gres, res)


@pytest.mark.parametrize("units, largest", [(255, 8192), (256, 8192), (256, 8193), (300, 40960), (256, 40961)])
def test_runs_of_many_units(tpcca, row_x, units, largest):
    """From 256 units on the units' chains and assignments go by two sizes of
    blocks: units around the limits among short, empty and one-cluster ones."""
    big = tpcgen.central_event(seed=8, n_tracks=12500, keep_truth=False)
    sizes = [largest, 8191, 8192, min(largest, 8193), 0, 1, largest] + [300 + 7 * (u % 40) for u in range(units - 7)]
    parts = [(u, tuple(a[:k] for a in big.unit(u % 36)[:2])) for u, k in enumerate(sizes)]
    off = np.cumsum([0] + sizes)
    table = np.array([(off[u], sizes[u], u // 36, u % 36) for u in range(units)], np.int64)
    b = tpcgen.Batch(np.concatenate([p[0] for _, p in parts]), np.concatenate([p[1] for _, p in parts]), table)
    refs = _parity.oracle_units(b, row_x)
    with tpcca.Context(row_x) as ctx:
        for graph in (False, True, True):
            ctx.run_batch(b.cl, b.row, table, graph=graph)
            _parity.compare_batch(*ctx.get_batch_results(), b, refs)
