"""Genus 2, level 2 counted by norms in F_q (the persistent forms of
primes q >= 37 and prime powers q >= 81):
equal to the oracle and, on more rows, to the plain form, which counts the same
level through its Zech table in F_{q^2}.  Fields on both sides of each choice:
3M or 2M Zech rows (243 / 251), prime (integer translates) or prime power (log
translates), q = 1 or 3 mod 4, every remainder of the (q - 1) / 2 nonsquares by
the inner loop's 8; rows of both degrees with zero coefficients anywhere and
with roots in F_{q^2}."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FIELDS = [37, 41, 43, 61, 67, 71, 79, 81, 101, 121, 127, 131, 169, 191, 239, 241, 243, 251, 283, 289, 293]


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_11991_amd import hwcount
    c = hwcount.Context(device=0)
    yield c
    c.close()


def _rows(curvegen_mod, q, n):
    """Seeded rows, a third with one to five zero coefficients below the
    leading one, a third of degree 5; int16."""
    c = curvegen_mod.sample(q, 2, n, seed=4100 + q, dtype=np.int16)
    rng = np.random.default_rng(q)
    for i in range(n):
        if i % 3 == 1:
            c[i, 6] = 0
            c[i, 5] = max(int(c[i, 5]), 1)
        top = 6 if c[i, 6] else 5
        if i % 3 != 2:
            c[i, rng.permutation(top)[: i % 6]] = 0
    return c


def _run(ctx, q, rows, flags):
    import torch
    n = len(rows)
    d = torch.from_numpy(rows).cuda()
    N = torch.full((n, 2), -1, dtype=torch.int32, device="cuda")
    ctx.count_curves_dev(q, 2, d, N, flags=flags)
    ctx.status()
    return N.cpu().numpy()


@pytest.mark.parametrize("q", FIELDS + [307])     # 307: the largest folded image
def test_norm_count(ctx, oracle_mod, curvegen_mod, q):
    from paper_1805_11991_amd import hwcount as hw
    rows = _rows(curvegen_mod, q, 2000)
    plain = _run(ctx, q, rows, hw.HWC_PLAIN)
    few = 40 if q < 150 else 12
    assert np.array_equal(plain[:few], oracle_mod.count_curves(q, 2, rows[:few]))
    for n in (1, 64, 65, 2000):
        assert np.array_equal(_run(ctx, q, rows[:n], hw.HWC_NO_GRAPH), plain[:n]), (q, n)
    if q <= 127:
        assert np.array_equal(_run(ctx, q, rows.astype(np.int8), 0), plain)


def test_norm_count_in_a_batch(ctx, curvegen_mod):
    """Jobs with and without norm tables in one launch, the image restaged
    between them."""
    import torch
    from paper_1805_11991_amd import hwcount as hw
    jobs, want = [], []
    for q in (13, 49, 37, 121, 251, 293, 29):
        rows = _rows(curvegen_mod, q, 300 + q)
        jobs.append({"q": q, "g": 2, "d_coeffs": torch.from_numpy(rows).cuda(),
                     "d_out_N": torch.zeros((len(rows), 2), dtype=torch.int32, device="cuda")})
        want.append(_run(ctx, q, rows, hw.HWC_PLAIN))
    for flags in (0, hw.HWC_NO_GRAPH):
        for j in jobs:
            j["d_out_N"].zero_()
        torch.cuda.synchronize()
        ctx.count_batch(jobs, flags=flags)
        ctx.status()
        for j, w in zip(jobs, want):
            assert np.array_equal(j["d_out_N"].cpu().numpy(), w), (j["q"], flags)


@pytest.mark.parametrize("q", [67, 169, 251])
def test_norm_root_counts(ctx, curvegen_mod, q):
    """The partition reads level 2's root counts: the same codes as from the
    plain form."""
    import torch
    from paper_1805_11991_amd import hwcount as hw
    rows = curvegen_mod.sample(q, 2, 3000, seed=77, dtype=np.int16)
    d = torch.from_numpy(rows).cuda()
    got = []
    for flags in (hw.HWC_PLAIN, 0):
        N = torch.zeros((len(rows), 2), dtype=torch.int32, device="cuda")
        lam = torch.zeros(len(rows), dtype=torch.int32, device="cuda")
        ctx.count_lambda_dev(q, 2, d, N, lam, flags=flags)
        ctx.status()
        got.append((N.cpu().numpy(), lam.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


def test_small_budget_keeps_the_level_tables(curvegen_mod):
    """A table budget that holds the level tables alone still counts."""
    from paper_1805_11991_amd import hwcount
    rows = _rows(curvegen_mod, 101, 100)
    with hwcount.Context(device=0, autotune_db=None) as c:
        want, _ = c.count_curves(101, 2, rows)
        full = c.stats()["table_bytes"]
    with hwcount.Context(device=0, autotune_db=None, hbm_budget_bytes=full - 1) as c:
        got, _ = c.count_curves(101, 2, rows)
        assert c.stats()["table_bytes"] < full - 1
    assert np.array_equal(got, want)


def test_budget_of_several_plans(ctx, curvegen_mod):
    """A budget that holds the level tables of several plans, and not all of their
    norm tables: a batch over them runs (its plans cannot be evicted), and calls in
    turn evict none of them."""
    import torch
    from paper_1805_11991_amd import hwcount as hw
    fields = (101, 121, 199)
    rows = {q: _rows(curvegen_mod, q, 200) for q in fields}
    want = {q: _run(ctx, q, rows[q], hw.HWC_PLAIN) for q in fields}
    with hw.Context(device=0, autotune_db=None) as c:
        for q in fields:
            c.plan_info(q, 2)
        full = c.stats()["table_bytes"]
    with hw.Context(device=0, autotune_db=None, hbm_budget_bytes=full - 1) as c:
        for rep in range(2):
            for q in fields:
                assert np.array_equal(_run(c, q, rows[q], 0), want[q]), q
        st = c.stats()
        assert st["evictions"] == 0 and st["table_bytes"] + st["pending_free_bytes"] < full
    with hw.Context(device=0, autotune_db=None, hbm_budget_bytes=full - 1) as c:
        jobs = [{"q": q, "g": 2, "d_coeffs": torch.from_numpy(rows[q]).cuda(),
                 "d_out_N": torch.zeros((len(rows[q]), 2), dtype=torch.int32, device="cuda")} for q in fields]
        torch.cuda.synchronize()
        for flags in (hw.HWC_NO_GRAPH, 0, 0):
            c.count_batch(jobs, flags=flags)
            c.status()
            for j in jobs:
                assert np.array_equal(j["d_out_N"].cpu().numpy(), want[j["q"]]), (j["q"], flags)
                j["d_out_N"].zero_()
            torch.cuda.synchronize()
