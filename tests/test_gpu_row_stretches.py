"""Row pointers of sorted keys and rows back to coordinates: stretches of a thousand rows that are empty, short, full or hold more
entries than are read in order, sizes at the edges of the kernels' tiles."""
import numpy as np
import pytest
import torch

from paper_2404_04541_amd import binding as sg

pytestmark = pytest.mark.gpu


def entries(rows, kind, seed):
    """Sorted rows of the entries."""
    rng = np.random.default_rng(seed)
    if kind == "one":          # a single entry, everything else empty
        return np.array([rows - 1])
    if kind == "full":
        return np.repeat(np.arange(rows), 3)
    if kind == "heavy":        # one row of more entries than a stretch is read with, few elsewhere
        return np.sort(np.concatenate([np.full(70001, rows // 2), rng.integers(rows, size=500)]))
    return np.sort(rng.integers(rows, size=rows // 3 + 4095))


@pytest.mark.parametrize("kind", ["one", "full", "heavy", "sparse"])
@pytest.mark.parametrize("i, j", [(1, 1), (1, 1023), (32, 32), (25, 41), (1, 4096), (64, 1600), (7, 100003)])
def test_unfold_and_fold(i, j, kind):
    r = entries(i * j, kind, i + j)
    k = np.arange(r.size) % 5
    order = np.random.default_rng(1).permutation(r.size)
    dev = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(t).cuda()  # noqa: E731
    h = sg.Handle()
    u = sg.sptensor_unfold(h, 3, (i, j, 5), *(dev(c[order], torch.int32) for c in (r // j, r % j, k)), dev(np.ones(r.size), torch.float64))
    torch.cuda.synchronize()
    rowptr = np.searchsorted(r, np.arange(i * j + 1))
    assert np.array_equal(u.rowptr.cpu().numpy(), rowptr)
    yi, yj, yk = sg.sptensor_fold(h, 3, (i, j, 5), u)
    torch.cuda.synchronize()
    assert np.array_equal(yi.cpu().numpy(), r // j)
    assert np.array_equal(yj.cpu().numpy(), r % j)
    assert torch.equal(yk, u.colidx)
