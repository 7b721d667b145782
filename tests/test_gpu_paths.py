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
    dict(fit_block=256, fit_min_waves=5),       # the 5-wave register budget
    dict(fit_claims=0),                         # claims in a kernel of their own
]


@pytest.mark.parametrize("tracks, sectors", [(12, 1), (700, 3), (8000, 4)])
def test_fit_forms_against_the_oracle(tpcca, torch_cuda, row_x, tracks, sectors):
    """Both forms of the fit kernel (loops for few tracklets, state machine for
    many) at tracklet counts below and above a wave each, with every register
    budget and block size, against the oracle: tracklets, tracks, assignment."""
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
