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
