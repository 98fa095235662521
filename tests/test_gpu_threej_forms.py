"""Rows of 3j symbols by the form that a call takes: short rows (up to 512 entries, 64
threads each), pieces of 2048 entries, and the longer pieces and whole rows of results
beyond the memory-side cache (more than 256 MB).  A symbol does not depend on the form, so
a large call of a few pairs over and over has the rows of a small call, bitwise; the small
calls are checked against the oracle's long-double rows.

A short row costs its setup once: 20000 rows of (2 2 -4) at lmax 10 stay within 2.5 times
the rows of (0 0 0), whose setup is next to nothing (3.2 with four waves for 21 entries).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PAIRS = [(0, 0), (0, 5), (1, 1), (3, 2), (127, 128), (128, 127), (255, 255), (255, 256), (256, 300), (700, 900),
         (1023, 1024), (1300, 1299), (2048, 2047), (2049, 2600), (4096, 4100)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_15605_amd import couple
    c = couple.couple_init(4200)
    yield c
    couple.couple_free(c)


def _rows(ctx, pairs, ms, stride):
    import torch
    from paper_2602_15605_amd import couple
    l1, l2 = (torch.tensor([p[k] for p in pairs], dtype=torch.int32, device="cuda") for k in range(2))
    if len(ms) == 1:
        return couple.couple_threej_rows(ctx, l1, l2, ms[0], stride=stride)
    return couple.couple_threej_rows_m(ctx, l1, l2, *ms, stride=stride)


@pytest.mark.parametrize("ms", [(0,), (1,), (2,), (1, 1), (2, 2), (-2, 1), (-2, 4), (0, 2)])
def test_short_rows_and_pieces(ctx, oracle_bulk, ms):
    refs = [oracle_bulk.threej_row(a, b, -ms[0]) if len(ms) == 1 else oracle_bulk.threej_row_m(a, b, *ms) for a, b in PAIRS]
    for stride in (1, 63, 64, 65, 128, 129, 511, 512, 513, 2048, 8200):
        got = _rows(ctx, PAIRS, ms, stride).cpu().numpy()
        for row, ref, pair in zip(got, refs, PAIRS):
            n = min(len(ref), stride)
            assert np.max(np.abs(row[:n] - ref[:n])) <= 1e-13 * np.max(np.abs(ref)), (ms, stride, pair)
            assert np.all(row[n:] == 0.0), (ms, stride, pair)


@pytest.mark.parametrize("stride", [400, 512, 513, 1399, 1400, 2047, 2600, 2601, 4096, 4097, 8193])
@pytest.mark.parametrize("ms", [(0,), (1,), (2, 2), (-2, 1)])
def test_results_beyond_the_cache(ctx, ms, stride):
    import torch
    small = _rows(ctx, PAIRS + [(-1, 3), (2, 4201)], ms, stride)
    k = len(small)
    times = int(256e6 / (8 * k * stride)) + 1
    large = _rows(ctx, (PAIRS + [(-1, 3), (2, 4201)]) * times, ms, stride).view(times, k, stride)
    assert torch.equal(large.nan_to_num(7.0), small.nan_to_num(7.0).expand(times, k, stride))
    assert torch.isnan(small[-2:]).all() and not torch.isnan(small[:-2]).any()


def test_short_rows_cost_their_setup_once(ctx):
    import torch
    from paper_2602_15605_amd import couple
    rng = np.random.default_rng(1)
    l1, l2 = (torch.as_tensor(rng.integers(0, 11, 20000).astype(np.int32)).cuda() for _ in range(2))
    out = torch.empty((20000, 21), dtype=torch.float64, device="cuda")
    best = {}
    for ms in ((0, 0), (2, 2)):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for _ in range(10):
            e0.record()
            for _ in range(20):
                if ms == (0, 0):
                    couple.couple_threej_rows(ctx, l1, l2, 0, stride=21, out=out)
                else:
                    couple.couple_threej_rows_m(ctx, l1, l2, *ms, stride=21, out=out)
            e1.record()
            torch.cuda.synchronize()
            best[ms] = min(best.get(ms, 1e9), e0.elapsed_time(e1))
    assert best[2, 2] <= 2.5 * best[0, 0], best
