"""GPU parity at the edges of what single kernels and host paths hold: values
that outgrow a narrower type, buffers that change under a queued copy, knobs
and numbers out of the usual range."""
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
