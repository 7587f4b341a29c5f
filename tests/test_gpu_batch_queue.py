"""How the workgroups of a batch take the jobs' entries: chunks of a job's queue,
shared out by waves.  Every row is counted once whatever the sizes -- jobs of no
rows, of less and of more entries than waves, one job and many -- and a batch of
one mid-size job of a small field does not wait for its queue."""
from __future__ import annotations

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_11991_amd import hwcount
    c = hwcount.Context(device=0)
    yield c
    c.close()


def _job(curvegen_mod, q, g, n):
    import torch
    rows = curvegen_mod.sample(q, g, max(n, 1), seed=7 * q + g)[:n]
    return {"q": q, "g": g, "d_coeffs": torch.from_numpy(np.ascontiguousarray(rows)).cuda(),
            "d_out_N": torch.full((n, g), -1, dtype=torch.int32, device="cuda")}


def _best(ctx, call):
    call()
    ctx.status()
    t = []
    for _ in range(10):
        t0 = time.perf_counter()
        call()
        ctx.status()
        t.append(time.perf_counter() - t0)
    return min(t)


@pytest.mark.parametrize("sizes", [(1,), (65,), (70_001,), (0, 1, 64, 5000), (40_000, 3, 0, 9000, 20_000)])
def test_every_entry_once(ctx, curvegen_mod, sizes):
    import torch
    from paper_1805_11991_amd import hwcount as hw
    fields = [(13, 3), (101, 2), (5, 4), (49, 2), (9, 3)]
    jobs = [_job(curvegen_mod, *fields[i], n) for i, n in enumerate(sizes)]
    want = []
    for j in jobs:
        N = torch.full_like(j["d_out_N"], -1)
        ctx.count_curves_dev(j["q"], j["g"], j["d_coeffs"], N, flags=hw.HWC_PLAIN)
        want.append(N)
    ctx.status()
    for flags in (hw.HWC_NO_GRAPH, 0, 0):
        print(sizes, flags, flush=True)
        for j in jobs:
            j["d_out_N"].fill_(-1)
        torch.cuda.synchronize()
        ctx.count_batch(jobs, flags=flags)
        ctx.status()
        for j, w in zip(jobs, want):
            assert torch.equal(j["d_out_N"], w), (j["q"], j["g"], len(w), flags)


def test_one_job_is_not_bound_by_its_queue(ctx, curvegen_mod):
    """2^18 curves at g = 3, q = 13: about 110 us of counting in some 32 768 entries,
    which popped one by one from one address take 530 us."""
    import torch
    j = _job(curvegen_mod, 13, 3, 1 << 18)

    alone = _best(ctx, lambda: ctx.count_curves_dev(13, 3, j["d_coeffs"], j["d_out_N"]))
    batch = _best(ctx, lambda: ctx.count_batch([j]))
    assert batch < alone + 300e-6, (batch, alone)


def test_late_workgroups_take_their_share(ctx, curvegen_mod):
    """Two large jobs take about the sum of their times alone: a workgroup that comes
    to the second one when little of it is left takes little (with a chunk by the
    whole job's size the end cost an eighth)."""
    import torch
    jobs = []
    for q in (11, 13):
        j = _job(curvegen_mod, q, 4, 1 << 20)
        jobs.append({**j, "d_coeffs": j["d_coeffs"].repeat(4, 1),
                     "d_out_N": torch.empty((1 << 22, 4), dtype=torch.int32, device="cuda")})
    alone = [_best(ctx, lambda j=j: ctx.count_batch([j])) for j in jobs]
    both = _best(ctx, lambda: ctx.count_batch(jobs))
    assert both < 1.06 * sum(alone), (both, alone)
