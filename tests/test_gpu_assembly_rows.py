"""Assembly of lists of short rows against the oracle's, bit for bit (both sum
equal blocks in list order): row lengths around one wave, one wave's rows and
a workgroup's, uneven rows, the ends of the rules that take the list to this
path, the scan's limit, and an index out of range."""

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lengths(n_rows, fill, special):
    k = np.full(n_rows, fill)
    k[: len(special)] = special
    return k


LISTS = [
    (_lengths(1, 2, []), 1),
    (_lengths(1, 512, []), 3),  # the longest rows on average; at 513, one block more
    (_lengths(1, 513, []), 3),
    (_lengths(40, 3, [0, 1, 2, 63, 64, 65, 127, 128, 129, 0, 255, 256, 257, 600]), 9),
    (_lengths(63, 5, [4] * 20 + [0, 141]), 9),  # one workgroup's rows, as many as its pool holds
    (_lengths(64, 5, [4] * 20 + [0, 145]), 9),
    (_lengths(40, 3, [0, 64, 128, 129]), 10**6),  # hardly a column twice
    (_lengths(30, 2, [130, 2047]), 200),
    (_lengths(30, 2, [5, 2048]), 200),
    (_lengths(30, 2, [5, 2049]), 200),  # too long: sorted as a whole
    (_lengths(4095, 1, [2]), 4),  # one block more than rows; the most rows of the small scan
    (_lengths(4096, 1, [2]), 4),
    (_lengths(4096, 1, []), 4),  # as many blocks as rows: not this path
    (_lengths(70001, 1, [0] * 500 + [90] * 300), 40),
    (_lengths(3000, 0, [115] * 1000), 30),  # three rows to a batch, eight to a workgroup
    (_lengths(70000, 4, [1990] * 1000), 200),  # sampled, and sorted as a whole
]


def _list(lengths, spread, order):
    rng = np.random.default_rng(lengths.size + spread)
    rows = np.repeat(np.arange(lengths.size), lengths)
    cols = rng.integers(0, min(spread, lengths.size), rows.size) + rows // 7
    cols %= lengths.size
    if order == "shuffled":
        p = rng.permutation(rows.size)
    else:  # runs of four equal rows, as elements list them, in mixed order
        p = np.arange(rows.size)
        head = p[: p.size // 4 * 4].reshape(-1, 4)
        p = np.concatenate([head[rng.permutation(len(head))].reshape(-1), p[p.size // 4 * 4:]])
    blocks = rng.standard_normal((rows.size, 3, 3)) * 10.0 ** rng.integers(-6, 7, (rows.size, 1, 1))
    return rows[p], cols[p], blocks


@pytest.mark.parametrize("order", ["shuffled", "runs"])
@pytest.mark.parametrize("i", range(len(LISTS)))
def test_assemble_short_rows(i, order):
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
    for capacity in (None, max(1, want[1].size - 1)):  # too small at first: sized and assembled again
        H = mp.bcsr_assemble(n, r, c, b, capacity=capacity)
        got = [t.cpu().numpy() for t in (H.row_ptr, H.col_idx, H.val)]
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        assert np.array_equal(got[2].reshape(-1).view(np.int64), want[2].reshape(-1).view(np.int64))
    for bad in (-1, n):
        for at in (0, rows.size - 1):
            for t in (r, c):
                u = t.clone()
                u[at] = bad
                with pytest.raises(mp.MasError):
                    mp.bcsr_assemble(n, u if t is r else r, u if t is c else c, b)
