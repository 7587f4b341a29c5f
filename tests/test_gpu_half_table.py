"""The half table (u16 low halves and a plane of 17th bits): equal to the oracle
on its smallest and largest fields, split over mu_4 and mu_2, on dense and sparse
rows, with roots at the level (zero points) and vanishing sub-polynomials."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FORM_F = 4


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1805_11991_amd import hwcount
    c = hwcount.Context(device=0)
    yield c
    c.close()


# (q, g), rows: M = 83 520, 85 848, 130 320 and 117 648 with mu_4 (4 | q - 1), M =
# 103 822 with mu_2; the plain form, as genus 2 otherwise counts by norms
@pytest.mark.parametrize("q,g,n", [(17, 4, 24), (293, 2, 24), (361, 2, 24), (49, 3, 16), (47, 3, 16)])
def test_half_table(ctx, oracle_mod, curvegen_mod, q, g, n):
    import torch
    from paper_1805_11991_amd import hwcount as hw
    print(q, g, flush=True)
    assert ctx.plan_info(q, g)[g - 1]["form"] == FORM_F
    rows = curvegen_mod.sample(q, g, n, seed=77 + q, dtype=np.int16)
    rows[: n // 4, 1] = 0
    rows[: n // 4, 5] = 0                       # odd class of mu_4 without terms
    rows[n // 4: n // 2, 1: 2 * g + 1] = 0      # x^(2g+2) and x^(2g+1) terms and a constant
    if q % 4 == 1:
        rows[n // 2 - 1] = 0
        rows[n // 2 - 1, 0] = 1
        rows[n // 2 - 1, 2 * g + 2] = 1         # binomial: roots of unity of order 2 (2g + 2)
    want = oracle_mod.count_curves(q, g, rows)
    for flags in (hw.HWC_PLAIN, 0, hw.HWC_NO_GRAPH):
        N = torch.full((n, g), -1, dtype=torch.int32, device="cuda")
        ctx.count_curves_dev(q, g, torch.from_numpy(rows).cuda(), N, flags=flags)
        ctx.status()
        assert np.array_equal(N.cpu().numpy(), want), (q, g, flags)
