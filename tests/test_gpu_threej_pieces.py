"""Rows of 3j symbols are written in pieces of 2048 entries, each thread on one parity
of l1 + l2 + l3: row lengths and strides at the edges of a piece and of the 256-thread
block, even and odd, against the oracle's long-double rows.

The bounds are those of the symbols elsewhere: 1e-13 of a row's largest value (the
recursion's own error at these degrees is below 1e-14), and exact zeros past the row.
Each output row is followed by a guard column that no kernel may touch.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (l1, l2): rows of 2 min(l1, l2) + 1 entries, L = l1 + l2 + |l1 - l2| = 2 max even at entry 0
PAIRS = [(0, 0), (0, 5), (1, 1), (1, 900), (2, 3), (3, 2), (127, 128), (128, 127), (255, 300), (1023, 1023),
         (1024, 1023), (1024, 1024), (1025, 1300), (2047, 2048), (2048, 2100)]
STRIDES = [1, 2, 255, 256, 2047, 2048, 2049, 4096, 4097, 6001]


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    c = couple.couple_init(2100)
    yield c
    couple.couple_free(c)


@pytest.mark.parametrize("ms", [(0,), (1,), (2,), (1, 1), (2, 2), (-2, -1), (2, -1), (-1, 0)])
def test_rows_in_pieces(ctx, oracle_bulk, ms):
    import torch
    from paper_2602_15605_amd import couple
    l1, l2 = (torch.tensor([p[k] for p in PAIRS], dtype=torch.int32, device="cuda") for k in range(2))
    refs = [oracle_bulk.threej_row(a, b, -ms[0]) if len(ms) == 1 else oracle_bulk.threej_row_m(a, b, *ms) for a, b in PAIRS]
    for stride in STRIDES:
        buf = torch.full((len(PAIRS) * stride + 2,), 7.0, dtype=torch.float64, device="cuda")
        out = buf[1:-1].view(len(PAIRS), stride)
        if len(ms) == 1:
            couple.couple_threej_rows(ctx, l1, l2, ms[0], stride=stride, out=out)
        else:
            couple.couple_threej_rows_m(ctx, l1, l2, *ms, stride=stride, out=out)
        assert buf[0].item() == 7.0 and buf[-1].item() == 7.0, (ms, stride)
        got = out.cpu().numpy()
        for row, ref, pair in zip(got, refs, PAIRS):
            n = min(len(ref), stride)
            big = np.max(np.abs(ref))
            assert np.max(np.abs(row[:n] - ref[:n])) <= 1e-13 * big, (ms, stride, pair)
            assert np.all(row[n:] == 0.0), (ms, stride, pair)
