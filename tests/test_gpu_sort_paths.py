"""The three ways of sorting a list of keys (counted places, tiles merged in one
launch, tiles merged level by level), at the edges of their ranges and with
part tiles.  A step moves exactly the holes that the list names, so a key lost
or doubled by the sort of the load (unsorted keys) or by a step's (sorted runs
of 256) shows as a hole that stands still in the next step; and the field of the
whole load has to be the oracle's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 512, 513, 12288, 12289, 20480, 61441, 65536, 65537])
def test_every_hole_listed(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W

    p = W.gaussian_cloud(n, W.cloud_sigma(max(n, 100)), (480.0, 480.0, 300.0), 31, stream=n)
    ctx = g.gccd_init(g.Params.from_device(dict(W.DEVICE)))
    try:
        g.gccd_load(ctx, *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
        E = g.gccd_field(ctx, n).cpu().numpy()
        last = g.gccd_positions(ctx, n)[0].cpu().numpy()
        # the load's list, the list after kept steps, and the lists that steps sorted
        for steps in (1, 15, 1, 1, 15):
            g.gccd_run(ctx, 10.0, steps)
            pos = g.gccd_positions(ctx, n)[0].cpu().numpy()
            assert np.all(np.any(pos != last, axis=0))
            last = pos
    finally:
        g.gccd_destroy(ctx)
    idx = np.random.default_rng(2).choice(n, min(n, 200), replace=False)
    Eo, A = oracle.field([v[idx] for v in p], list(p), with_magnitude=True)
    assert np.all(np.linalg.norm(E[:, idx] - Eo, axis=0) <= 1e-5 * A + 1e-9)


@pytest.mark.parametrize("sources", [0, 1])
@pytest.mark.parametrize("n", [1, 64, 65, 128, 129, 192, 256, 257, 511, 512, 513])
def test_small_load_in_one_launch(n, sources):
    """A load of up to 512 holes is taken in and sorted by one workgroup.  Its list
    is compared with the one that a step's separate launches leave, through the
    field, whose rounding depends on slots, counts and boxes: bit for bit.  Part of
    the holes are collected at the load, mirrored, or travel."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W

    r = np.random.default_rng(n)
    p = r.normal(0.0, 1.0, size=(3, n)) + np.array([480.0, 480.0, 300.0])[:, None]
    p[2, 1::3] = -0.01                       # in the well
    p[2, 2::7] = W.DEVICE["thickness_um"] + 0.5   # beyond the back surface
    a, b = (g.gccd_init(g.Params.from_device(dict(W.DEVICE, collected_are_sources=sources)))
            for _ in range(2))
    try:
        g.gccd_load(a, *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
        g.gccd_run(a, 10.0, 1)
        pos, cstep = g.gccd_positions(a, n)
        g.gccd_load(b, *[v.contiguous() for v in pos])
        assert torch.equal(cstep >= 0, g.gccd_positions(b, n)[1] >= 0)
        assert g.gccd_stats(a)["n_active"] == g.gccd_stats(b)["n_active"]
        assert torch.equal(g.gccd_field(a, n), g.gccd_field(b, n))
        g.gccd_run(a, 10.0, 0)
        E = g.gccd_field_noalloc(g.Params.from_device(dict(W.DEVICE, collected_are_sources=sources)),
                                 *[v.contiguous() for v in pos])
        assert torch.equal(E, g.gccd_field(b, n))
    finally:
        g.gccd_destroy(a)
        g.gccd_destroy(b)
