"""Batches of many small events: a step that keeps the list's order takes one source
tile per turn of at most 512 workgroups, and a list of fewer than 16 holes per
tile is sorted every step.  Fewer and more tiles than workgroups, at, below and
above 16 holes per tile, and small events beside a large one: every event has to
move as the oracle moves it alone, and a run has to give the same bits and counts
however it is split."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LOADS = [[20] * 30, [16] * 513, [15] * 600, [33] * 1100, [1] * 700, [3000] + [16] * 600 + [257] * 5]


@pytest.mark.parametrize("sizes", LOADS, ids=lambda s: f"{len(s)}x{s[-1]}")
def test_small_events(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W
    r = np.random.default_rng(7700)
    off = [0] + np.cumsum(sizes).tolist()
    n = off[-1]
    p = r.normal(0.0, 0.8, size=(3, n)) + np.array([[480.0], [480.0], [300.0]])
    dev = [torch.as_tensor(v).cuda() for v in p]
    whole, split, fp64 = (g.gccd_init(g.Params.from_device(W.DEVICE)) for _ in range(3))
    g.gccd_set_precision(fp64, "fp64")
    for ctx in (whole, split, fp64):
        g.gccd_load_events(ctx, off, *dev)
    steps = 37
    for ctx in (whole, fp64):
        assert g.gccd_run(ctx, 10.0, steps) == (steps, n)
    for k in (1, 5, 10, 4, steps - 20):
        g.gccd_run(split, 10.0, k)
    a, _ = g.gccd_positions(whole, n)
    b, _ = g.gccd_positions(split, n)
    assert torch.equal(a, b)
    a = g.gccd_positions(fp64, n)[0].cpu().numpy()
    for ctx in (whole, split, fp64):
        s = g.gccd_stats(ctx)
        assert s["carrier_steps"] == steps * n
        assert s["pair_interactions"] == steps * sum(k * k for k in sizes)
        g.gccd_destroy(ctx)
    for e in {0, 1, len(sizes) // 2, 511, 512, len(sizes) - 1}:
        if e >= len(sizes):
            continue
        st = oracle.State(oracle.Device(**dict(W.DEVICE, event=e)), *p[:, off[e]:off[e + 1]])
        st.run(10.0, steps)
        # a field good to 1e-14, amplified by close encounters by 1e4 or so
        assert np.max(np.abs(a[:, off[e]:off[e + 1]] - np.array([st.x, st.y, st.z]))) <= 1e-6
