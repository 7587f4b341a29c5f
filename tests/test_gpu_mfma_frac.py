"""The matrix-product path's fractional form (primes p <= 13): equal to the
oracle on rows with zero and extreme coefficients, with padding rows in every
level's last block, partial tiles, both code widths, the full sweep and the
top level in one or several images."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (q, g): every degree with each size of word table; (13, 4), (11, 4) and (7, 4)
# spread their top level over several images; (13, 1) and (5, 4) stay on the
# other side of the rule
CASES = [(13, 1), (3, 2), (11, 2), (13, 2), (3, 3), (5, 3), (7, 3), (11, 3), (13, 3),
         (5, 4), (7, 4), (11, 4), (13, 4)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_11991_amd import hwcount
    c = hwcount.Context(device=0, mfma=True)
    yield c
    c.close()


def _run(ctx, q, g, rows, flags=0):
    import torch
    N = torch.full((len(rows), g), -1, dtype=torch.int32, device="cuda")
    ctx.count_curves_dev(q, g, torch.from_numpy(rows).cuda(), N, flags=flags)
    ctx.status()
    return N.cpu().numpy()


@pytest.mark.parametrize("q,g", CASES)
def test_fractional_form(ctx, oracle_mod, q, g):
    from paper_1805_11991_amd import hwcount as hw
    print(q, g, flush=True)
    frac = g >= 2 and (g < 4 or q >= 7)          # the rule: below, residues are faster
    for flags in (0, hw.HWC_FULL_SWEEP):
        assert [level["mfma"] for level in ctx.plan_info(q, g, flags)] == [2 if frac else 1] * g
    n = 97 if g < 4 or q < 7 else 33
    rng = np.random.default_rng(100 * q + g)
    rows = rng.integers(0, q, (n, 2 * g + 3)).astype(np.int8)
    h = (q - 1) // 2
    # the largest sums: every code at either end of the balanced range
    rows[0] = h
    rows[1] = h + 1
    rows[2] = np.where(np.arange(2 * g + 3) % 2, h, h + 1)
    rows[3:40] = np.where(rng.integers(0, 2, (min(n, 40) - 3, 2 * g + 3)), h, h + 1)
    rows[-20:, 1: 2 * g + 2] *= rng.integers(0, 2, (20, 2 * g + 1)).astype(np.int8)   # sparse
    rows[-10:, -1] = 0
    rows[-9:, 0] = 0
    rows[:, -2] = np.where(rows[:, -1] == 0, np.maximum(rows[:, -2], 1), rows[:, -2])
    want = oracle_mod.count_curves(q, g, rows)
    for m in (n, 1, 31, 32):
        assert np.array_equal(_run(ctx, q, g, rows[:m]), want[:m]), (q, g, m)
    assert np.array_equal(_run(ctx, q, g, rows.astype(np.int16), hw.HWC_NO_GRAPH), want)
    assert np.array_equal(_run(ctx, q, g, rows, hw.HWC_FULL_SWEEP), want)


@pytest.mark.parametrize("q,g", [(11, 4), (7, 4), (11, 3), (13, 3)])
def test_full_sweep_keeps_the_matrix_path(ctx, q, g):
    """Levels whose points do not fit one image are spread over several."""
    from paper_1805_11991_amd import hwcount as hw
    assert all(level["mfma"] for level in ctx.plan_info(q, g, hw.HWC_FULL_SWEEP)), (q, g)


def test_block_option_reaches_the_fractional_form(curvegen_mod):
    """The images of genus 3 over F_13 leave one workgroup to a CU, so four waves of
    256 threads take several times as long as sixteen."""
    import torch
    from paper_1805_11991_amd import hwcount as hw
    rows = torch.from_numpy(curvegen_mod.sample(13, 3, 1 << 19, seed=5)).cuda()
    out, ms = [], {}
    with hw.Context(device=0, mfma=True) as c:
        for block in (256, 1024):
            c.set_plan_option(13, 3, hw.HWC_OPT_BLOCK, block)
            assert c.plan_info(13, 3)[0]["mfma"] == 2
            N = torch.empty((len(rows), 3), dtype=torch.int32, device="cuda")
            c.count_curves_dev(13, 3, rows, N, flags=hw.HWC_NO_GRAPH)
            c.status()
            c.profile(True)
            for _ in range(3):
                c.count_curves_dev(13, 3, rows, N)
            ms[block] = c.profile_read()["count_ms"]
            c.profile(False)
            c.status()
            out.append(N)
    assert torch.equal(out[0], out[1])
    assert ms[256] > 1.5 * ms[1024], ms
