"""A serial list with every hole a source keeps its order for several steps: the
step kernel then writes the new positions in slot order and its source tile's
boxes, and only the steps at the end of such a stretch sort.  A run has to give
the same bits however it is split and whatever is asked in between, the sort
after kept steps has to give the list of a fresh load (holes collected since
then included), and a field between runs is that of the fresh list."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# one hole, one tile, a part tile, the largest load whose step kernel sorts, the
# smallest beyond it, both sides of 4e8 pairs, the long steps of a load above 2e9 (no
# order kept), and events of every kind of size
LOADS = [[1], [256], [700], [2048], [2049], [20000], [20001], [1, 300, 256, 7, 1100],
         [2500, 1, 513, 3000]]
STEPS = 37


def setup(sizes, seed):
    r = np.random.default_rng(seed)
    n = sum(sizes)
    p = r.normal(0.0, 1.0, size=(3, n)) + np.array([480.0, 480.0, 14.0])[:, None]
    return ([torch.as_tensor(v).cuda() for v in p], [0] + np.cumsum(sizes).tolist())


def same(a, b):
    for u, v in zip(a, b):
        assert torch.equal(u, v)


@pytest.mark.parametrize("sizes", LOADS, ids=lambda s: "-".join(map(str, s)))
def test_split_and_field_between(sizes, dt=10.0):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W

    params = g.Params.from_device(W.DEVICE)
    p, off = setup(sizes, 11)
    n = off[-1]
    whole, split, fresh = (g.gccd_init(params) for _ in range(3))
    g.gccd_load_events(whole, off, *p)
    g.gccd_load_events(split, off, *p)
    g.gccd_run(whole, dt, STEPS)
    for steps in (1, 5, 10, 4, STEPS - 20):  # to steps 1, 6, 16, 20 and the end
        g.gccd_run(split, dt, steps)
        field = g.gccd_field(split, n)
        pos, _ = g.gccd_positions(split, n)
        g.gccd_load_events(fresh, off, *[v.contiguous() for v in pos])
        same(field, g.gccd_field(fresh, n))
    same(g.gccd_positions(whole, n), g.gccd_positions(split, n))
    a, b = g.gccd_stats(whole), g.gccd_stats(split)
    assert a["pair_interactions"] == b["pair_interactions"]
    for ctx in (whole, split, fresh):
        g.gccd_destroy(ctx)


def test_long_steps():
    test_split_and_field_between([45001], 41.0)


def test_collected_between_sorts():
    """Holes collected within kept steps: their keys are marked at the next sort, so
    the list at step 32 and the field's targets are those of a fresh load."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W

    r = np.random.default_rng(5)
    for n in (900, 4000):
        p = r.normal(0.0, 2.0, size=(3, n)) + np.array([480.0, 480.0, 9.0])[:, None]
        p = [torch.as_tensor(v).cuda() for v in p]
        run, fresh = (g.gccd_init(g.Params.from_device(W.DEVICE)) for _ in range(2))
        g.gccd_load(run, *p)
        done, left = 0, n
        while left == n or done % 16 or left > 0.9 * n:
            k, left = g.gccd_run(run, 10.0, 1)
            done += k
            assert 0 < left and done < 400
        pos, cstep = g.gccd_positions(run, n)
        g.gccd_load(fresh, *[v.contiguous() for v in pos])
        _, c2 = g.gccd_positions(fresh, n)
        assert torch.equal(cstep >= 0, c2 >= 0)
        same(g.gccd_field(run, n), g.gccd_field(fresh, n))
        g.gccd_destroy(run)
        g.gccd_destroy(fresh)
