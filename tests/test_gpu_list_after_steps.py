"""The list that a run leaves where its order is renewed (a step that is a multiple of
16), after holes were collected in steps that kept it: made from the step kernel's
keys by the counted sort (up to 12288 holes) or from its sorted runs. gccd_field
there sums over this list itself, in its order, with its tile boxes and counts, so it
equals a fresh load's of the same positions bit for bit only if the lists are the
same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def cloud(sizes, depths, spread, seed):
    r = np.random.default_rng(seed)
    parts = [r.normal(0.0, spread, size=(3, k)) + np.array([[480.0], [480.0], [z]])
             for k, z in zip(sizes, depths)]
    return [torch.as_tensor(v).cuda() for v in np.concatenate(parts, axis=1)]


def check(sizes, depths, spread, seed, left_of=(0.05, 0.95)):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    off = [0] + np.cumsum(sizes).tolist()
    n = off[-1]
    run, fresh = (g.gccd_init(g.Params()) for _ in range(2))
    g.gccd_load_events(run, off, *cloud(sizes, depths, spread, seed))
    done, left = 0, n
    while left > left_of[1] * n and done < 960:
        k, left = g.gccd_run(run, 10.0, 16)
        done += k
    pos, cstep = g.gccd_positions(run, n)
    assert done % 16 == 0 and left_of[0] * n < left <= left_of[1] * n
    at = cstep[cstep > 0]
    assert bool((at % 4 != 0).any())  # between sorts, whichever number of steps keeps the order
    E = g.gccd_field(run, n)
    g.gccd_load_events(fresh, off, *[v.contiguous() for v in pos])
    assert torch.equal(cstep >= 0, g.gccd_positions(fresh, n)[1] >= 0)
    assert torch.equal(E, g.gccd_field(fresh, n))
    for ctx in (run, fresh):
        g.gccd_destroy(ctx)


@pytest.mark.parametrize("n", [700, 2000, 2048, 10007, 12288, 12289, 14000])
def test_one_event(n):
    check([n], [12.0], 2.0, 8000 + n)


def test_small_events():
    check([300, 7, 1, 900, 250, 400], [9.0, 300.0, 8.0, 10.0, 400.0, 11.0], 1.5, 8101)


def test_events_above_the_counted_sort():
    check([1500] * 9 + [513, 1, 40], [9.0 + k for k in range(12)], 1.5, 8102)
