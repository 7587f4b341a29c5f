"""The one-workgroup bucketing (a request of up to 1024 rows alone, jobs of up to
8192 rows in a batch of several): a request's counts equal the same rows' counts
inside a larger request, which is bucketed by the many-workgroup kernels -- at
the edges of its waves, of its passes over the rows and of its range; rows as
given, translated by dot products (prime q) or by the step table (prime powers);
int8 and int16; few and many patterns.  Single requests of 1025 rows and more
take the many-workgroup kernels: the edge of the rule."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 64, 65, 1023, 1024, 1025, 4097, 8191, 8192]


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_11991_amd import hwcount
    c = hwcount.Context(device=0)
    yield c
    c.close()


def _rows(curvegen_mod, q, g, n, dtype):
    rows = curvegen_mod.sample(q, g, n, seed=31 * q + g, dtype=dtype)
    rng = np.random.default_rng(q)
    for i in range(0, n, 2):                  # every zero pattern, of both degrees
        if i % 3 == 0:
            rows[i, -1] = 0
            rows[i, -2] = max(int(rows[i, -2]), 1)
        top = 2 * g + 2 if rows[i, -1] else 2 * g + 1
        rows[i, :top][rng.random(top) < 0.4] = 0
    return rows


def _count(ctx, q, g, rows, flags=0):
    import torch
    N = torch.full((len(rows), g), -1, dtype=torch.int32, device="cuda")
    ctx.count_curves_dev(q, g, torch.from_numpy(rows).cuda(), N, flags=flags)
    ctx.status()
    return N.cpu().numpy()


@pytest.mark.parametrize("q,g,dtype", [(3, 1, np.int8), (37, 2, np.int8), (31, 2, np.int16), (13, 3, np.int8),
                                       (27, 2, np.int8), (9, 3, np.int16), (25, 2, np.int16), (5, 4, np.int8),
                                       (7, 4, np.int16)])
def test_same_counts_as_the_large_bucketing(ctx, oracle_mod, curvegen_mod, q, g, dtype):
    rows = _rows(curvegen_mod, q, g, 9000, dtype)
    want = _count(ctx, q, g, rows)
    assert np.array_equal(want[:60], oracle_mod.count_curves(q, g, rows[:60]))
    for n in SIZES:
        assert np.array_equal(_count(ctx, q, g, rows[:n]), want[:n]), n
        assert np.array_equal(_count(ctx, q, g, rows[9000 - n:], flags=8), want[9000 - n:]), n


def test_batch_of_small_and_large(ctx, curvegen_mod):
    import torch
    jobs, want = [], []
    for q, g, n, dtype in [(13, 3, 9000, np.int8), (27, 2, 8192, np.int8), (9, 3, 100, np.int16), (5, 4, 1, np.int8),
                           (67, 2, 700, np.int8), (131, 2, 90, np.int16), (7, 1, 1024, np.int8), (29, 2, 8193, np.int8)]:
        rows = _rows(curvegen_mod, q, g, n, dtype)
        want.append(_count(ctx, q, g, rows))
        jobs.append({"q": q, "g": g, "d_coeffs": torch.from_numpy(rows).cuda(),
                     "d_out_N": torch.zeros((n, g), dtype=torch.int32, device="cuda")})
    jobs.append({"q": 13, "g": 3, "d_coeffs": torch.zeros((0, 9), dtype=torch.int8, device="cuda"),
                 "d_out_N": torch.zeros((0, 3), dtype=torch.int32, device="cuda")})
    want.append(np.zeros((0, 3), np.int32))
    for flags in (8, 0, 0):
        for j in jobs:
            j["d_out_N"].zero_()
        torch.cuda.synchronize()
        ctx.count_batch(jobs, flags=flags)
        ctx.status()
        for j, w in zip(jobs, want):
            assert np.array_equal(j["d_out_N"].cpu().numpy(), w), (j["q"], j["g"], flags)


@pytest.mark.parametrize("q,g,dtype", [(13, 3, np.int8), (31, 2, np.int16), (67, 2, np.int16), (27, 2, np.int8),
                                       (9, 3, np.int16), (25, 2, np.int16), (3, 1, np.int8), (7, 4, np.int16)])
def test_large_jobs_together(ctx, oracle_mod, curvegen_mod, q, g, dtype):
    """More rows than one pass of the workgroup: every job of a batch of at least
    three, at the edges of the passes and of the range."""
    import torch
    from paper_1805_11991_amd import hwcount as hw
    rows = _rows(curvegen_mod, q, g, 9000, dtype)
    want = _count(ctx, q, g, rows)                       # many-workgroup kernels
    assert np.array_equal(want[:60], oracle_mod.count_curves(q, g, rows[:60]))
    cuts = [(0, 1025), (500, 2048), (9000 - 4097, 4097), (7, 8191), (808, 8192), (0, 63), (0, 8193)]
    jobs = [{"q": q, "g": g, "d_coeffs": torch.from_numpy(np.ascontiguousarray(rows[a:a + n])).cuda(),
             "d_out_N": torch.full((n, g), -1, dtype=torch.int32, device="cuda")} for a, n in cuts]
    for flags in (hw.HWC_NO_GRAPH, 0, 0):
        for j in jobs:
            j["d_out_N"].fill_(-1)
        torch.cuda.synchronize()
        print(q, g, dtype, flags, flush=True)
        ctx.count_batch(jobs, flags=flags)
        ctx.status()
        for (a, n), j in zip(cuts, jobs):
            assert np.array_equal(j["d_out_N"].cpu().numpy(), want[a:a + n]), (a, n, flags)


@pytest.mark.parametrize("bad,code", [((0, 13), -4), ((0, -1), -4), (None, -5)])
def test_row_errors(ctx, curvegen_mod, bad, code):
    from paper_1805_11991_amd import hwcount
    rows = curvegen_mod.sample(13, 3, 100, seed=3)
    if bad:
        rows[57, bad[0]] = bad[1]
    else:
        rows[57, 7:] = 0
    with pytest.raises(hwcount.HwcError) as e:
        _count(ctx, 13, 3, rows)
    assert e.value.code == code
    _count(ctx, 13, 3, curvegen_mod.sample(13, 3, 100, seed=3))
