"""A context keeps its load buffers from load to load.  Loads of changing size
and shape on one context have to run exactly as on a fresh one: larger, smaller and
equal loads, several events, the far smaller load that lets the large buffers go,
and loads whose partial sums or closure buffers grew in between.  The kernel that
takes a load in reads the caller's arrays directly only where it may; a
misaligned or host-pinned source is copied first and must load the same."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# events of each load in turn, holes per event; 1.6 million holes take more than
# four times 64 MiB, so the small load after them gives the buffers back
LOADS = [[5], [3000], [300], [70001], [255, 1, 513], [1], [1_600_003], [2049], [64] * 40, [20011]]


def cloud(sizes, seed):
    r = np.random.default_rng(seed)
    n = sum(sizes)
    xy = r.normal(480.0, 30.0, size=(2, n))
    z = r.uniform(100.0, 505.0, size=n)
    z[::7] = 0.01  # collected at the load
    return [torch.as_tensor(v).cuda() for v in (xy[0], xy[1], z)]


def state(g, ctx, n, steps):
    g.gccd_run(ctx, 10.0, steps)
    return [v.cpu().numpy() for v in g.gccd_positions(ctx, n)]


@pytest.mark.parametrize("coulomb", [0, 1])
def test_reused_context(coulomb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g

    params = g.Params(coulomb=coulomb, event=3)
    kept = g.gccd_init(params)
    for k, sizes in enumerate(LOADS):
        if coulomb and max(sizes) > 100000:
            steps = 1
        else:
            steps = 5
        p = cloud(sizes, 40 + k)
        off = [0] + np.cumsum(sizes).tolist()
        fresh = g.gccd_init(params)
        for ctx in (kept, fresh):
            g.gccd_load_events(ctx, off, *p)
        a, b = (state(g, ctx, off[-1], steps) for ctx in (kept, fresh))
        for u, v in zip(a, b):
            np.testing.assert_array_equal(u, v)
        # the field allocates what a load without repulsion does not have
        if off[-1] < 10000:
            for u, v in zip(g.gccd_field(kept, off[-1]), g.gccd_field(fresh, off[-1])):
                assert torch.equal(u, v)
        g.gccd_destroy(fresh)
    g.gccd_destroy(kept)


@pytest.mark.parametrize("source", ["misaligned", "pinned"])
def test_copied_source(source):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g

    n = 777
    p = cloud([n], 9)
    if source == "misaligned":
        held = [torch.zeros(8 * n + 8, dtype=torch.uint8, device="cuda") for _ in p]
        for h, v in zip(held, p):
            h[4:4 + 8 * n] = v.view(torch.uint8)
        addr = [h.data_ptr() + 4 for h in held]
    else:
        held = [v.cpu().pin_memory() for v in p]
        addr = [h.data_ptr() for h in held]
    torch.cuda.synchronize()
    a, b = g.gccd_init(g.Params()), g.gccd_init(g.Params())
    g.gccd_load(a, *p)
    assert g.lib.gccd_load(b, n, *[ctypes.c_void_p(v) for v in addr]) == 0
    for u, v in zip(state(g, a, n, 3), state(g, b, n, 3)):
        np.testing.assert_array_equal(u, v)
    g.gccd_destroy(a)
    g.gccd_destroy(b)


@pytest.mark.parametrize("n", [700, 3000])
def test_replays_of_a_later_load(n):
    """Loads of the same shape replay the steps captured for an earlier one: other
    positions, other events of the same total and number of tiles, another
    launch shape and another time step in between, each as on a fresh context."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g

    params = g.Params()
    kept = g.gccd_init(params)
    a, b = n // 2 - 20, n - n // 2 + 20
    for k, (sizes, dt, chunks) in enumerate([([n], 10.0, 0), ([n], 10.0, 0), ([a, b], 10.0, 0),
                                             ([b, a], 10.0, 0), ([n], 10.0, 3), ([n], 5.0, 3),
                                             ([n - 1], 5.0, 3), ([n], 10.0, 0)]):
        p = cloud(sizes, 80 + k)
        off = [0] + np.cumsum(sizes).tolist()
        fresh = g.gccd_init(params)
        out = []
        for ctx in (kept, fresh):
            g.gccd_set_launch(ctx, 0, chunks)
            g.gccd_load_events(ctx, off, *p)
            g.gccd_run(ctx, dt, 70)
            assert g.gccd_stats(ctx)["graph_usable"] == 1
            out.append(g.gccd_positions(ctx, off[-1]))
        for u, v in zip(*out):
            assert torch.equal(u, v)
        g.gccd_destroy(fresh)
    g.gccd_destroy(kept)
