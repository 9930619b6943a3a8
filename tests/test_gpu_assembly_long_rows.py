"""Assembly of lists with rows beyond the pool of a workgroup (448 blocks)
against the oracle's, bit for bit: the ends of the pool, of a piece (2,048)
and of the rows that are grouped at all (8,192), runs of one column that are
longer than a tile, long rows next to one another and among empty ones."""

import numpy as np
import pytest

import oracle
from test_gpu_assembly_rows import _lengths, _list

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LISTS = [
    (_lengths(40, 3, [444, 445, 447, 448, 449, 450, 0, 511, 512, 513]), 9),
    (_lengths(1100, 2, [448, 449, 0, 2047, 2048, 2049, 4095, 4096, 4097]), 10**6),  # hardly a column twice
    (_lengths(40, 2, [2047, 0, 2048, 2049, 4097]), 2),  # long runs of a column
    (_lengths(17, 0, [8192]), 17),
    (_lengths(9000, 2, [0] * 70 + [8192, 8191, 6145]), 10**6),
    (_lengths(9000, 2, [5, 8193]), 300),  # too long: sorted as a whole
    (_lengths(3000, 4, [3] * 1000 + [600, 1250, 470] * 60), 500),
    (_lengths(9, 450, []), 9),
    (_lengths(9, 400, []), 9),  # the longest rows on average
    (_lengths(6000, 3, ([2] * 20 + [300, 3, 0, 10]) * 40), 50),  # a long row in rows that hold no more than the pool
    (_lengths(6000, 3, [180, 224, 225, 0, 226] * 200), 50),  # batches and long rows in turn
]


@pytest.mark.parametrize("order", ["shuffled", "runs"])
@pytest.mark.parametrize("i", range(len(LISTS)))
def test_assemble_long_rows(i, order):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2411_06224_amd as mp

    lengths, spread = LISTS[i]
    n = lengths.size
    rows, cols, blocks = _list(lengths, spread, order)
    print("[case]", n, rows.size, order, flush=True)
    dev = torch.device("cuda:0")
    r, c = (torch.as_tensor(a.astype(np.int32), device=dev) for a in (rows, cols))
    b = torch.as_tensor(blocks, device=dev)
    want = oracle.assemble(n, rows, cols, blocks)
    H = mp.bcsr_assemble(n, r, c, b)
    got = [t.cpu().numpy() for t in (H.row_ptr, H.col_idx, H.val)]
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert np.array_equal(got[2].reshape(-1).view(np.int64), want[2].reshape(-1).view(np.int64))
    long_ = int(np.flatnonzero(rows == int(np.argmax(lengths)))[0])  # a bad index in the longest row
    for bad in (-1, n, 0x7FFFFFFF, -0x80000000):
        for t in (r, c):
            u = t.clone()
            u[long_] = bad
            with pytest.raises(mp.MasError):
                mp.bcsr_assemble(n, u if t is r else r, u if t is c else c, b)
