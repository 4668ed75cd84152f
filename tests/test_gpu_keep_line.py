"""Where a serial list goes over from 16 to 4 steps in one order (1.2e8 pairs of
holes, 10,954 of one event): loads on both sides, and a batch at the line, give the
same bits however a run is split, at short and long steps."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LINE = math.isqrt(120000000)


@pytest.mark.parametrize("dt", [10.0, 500.0])
@pytest.mark.parametrize("sizes", [[LINE], [LINE + 1], [7746] * 2], ids=str)
def test_split_run(sizes, dt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    off = [0] + np.cumsum(sizes).tolist()
    p = np.random.default_rng(7800).normal(0.0, 1.2, size=(3, off[-1]))
    p = [torch.as_tensor(v).cuda() for v in p + np.array([[480.0], [480.0], [500.0]])]
    whole, split = (g.gccd_init(g.Params()) for _ in range(2))
    for ctx in (whole, split):
        g.gccd_load_events(ctx, off, *p)
    g.gccd_run(whole, dt, 39)
    for k in (3, 1, 9, 4, 22):
        g.gccd_run(split, dt, k)
    assert torch.equal(g.gccd_positions(whole, off[-1])[0], g.gccd_positions(split, off[-1])[0])
    for ctx in (whole, split):
        g.gccd_destroy(ctx)
