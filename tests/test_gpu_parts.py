"""Small requests over the largest admitted fields, whose top level (millions of
points in device memory) is cut into the most parts: equal to the plain form,
which sweeps whole tiles.  Dense rows take the split sweep, rows with empty
residue classes the unsplit one."""
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


@pytest.mark.parametrize("q,g", [(2063, 2), (4093, 2), (251, 3), (61, 4)])
def test_most_parts(ctx, q, g):
    import torch
    from paper_1805_11991_amd import hwcount as hw
    nc = 2 * g + 3
    rng = np.random.default_rng(q)
    rows = rng.integers(1, q, (200, nc)).astype(np.int16)
    rows[1::4, -1] = 0                                   # odd degree
    rows[2::4, 1:nc - 1:2] = 0                           # even powers only
    rows[3::4, :nc - 2] *= rng.integers(0, 2, (50, nc - 2)).astype(np.int16)
    d = torch.from_numpy(rows).cuda()
    print(q, g, flush=True)
    want = torch.full((len(rows), g), -1, dtype=torch.int32, device="cuda")
    ctx.count_curves_dev(q, g, d, want, flags=hw.HWC_PLAIN)
    ctx.status()
    for n in (1, 3, 65, 200):
        print(q, g, n, flush=True)
        N = torch.full((n, g), -1, dtype=torch.int32, device="cuda")
        ctx.count_curves_dev(q, g, d[:n].contiguous(), N)
        ctx.status()
        assert torch.equal(N, want[:n]), n
