"""How the waves of a persistent count take its entries: requests of less than one
round of the resident waves, of one to two, of more (a first round of their own
and the rest common) and of more than twelve (all common), whole tiles and parts,
Zech tables and norms.  Equal to the plain form, whose launches share out whole
tiles by workgroup."""
from __future__ import annotations

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


# tiles against about 6144 (genus 3 over F_13) or 8192 (genus 2 over F_37) and 4096
# (genus 3 over F_25: parts) resident waves
@pytest.mark.parametrize("q,g,sizes", [
    (13, 3, (1, 65, 40_000, 300_000, 500_000, 1_000_000, 5_000_000)),
    (37, 2, (1, 129, 10_000, 700_000, 1_200_000)),
    (25, 3, (64, 5_000, 40_000, 140_000)),
])
def test_every_share(ctx, curvegen_mod, q, g, sizes):
    import torch
    from paper_1805_11991_amd import hwcount as hw
    n = max(sizes)
    rows = torch.from_numpy(curvegen_mod.sample(q, g, n, seed=91 + q)).cuda()
    want = torch.full((n, g), -1, dtype=torch.int32, device="cuda")
    ctx.count_curves_dev(q, g, rows, want, flags=hw.HWC_PLAIN)
    ctx.status()
    for m in sizes:
        print(q, g, m, flush=True)
        for flags in (hw.HWC_NO_GRAPH, 0, 0):        # a captured graph and its replay
            N = torch.full((m, g), -1, dtype=torch.int32, device="cuda")
            ctx.count_curves_dev(q, g, rows[:m], N, flags=flags)
            ctx.status()
            assert torch.equal(N, want[:m]), (q, g, m, flags)
    assert np.array_equal(want[:64].cpu().numpy() >= 0, np.ones((64, g), dtype=bool))
