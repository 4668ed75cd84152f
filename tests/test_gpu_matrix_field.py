"""The default Eq. (6) kernel sums blocks of 16 targets and 16 sources, far
ones with r^2 from the matrix cores and near ones from differences.  These
loads put the edges of its blocks, waves and tiles where they can go wrong:
two clusters of m holes each, 12 um apart, so that every target has near blocks
(its own cluster, which straddles a block of 16 whenever m is no multiple of
16) and far ones, with padding lanes and padding sources in both, at each
tile size and for both choices of sources.

Tolerance: 1e-5 of the sum of term magnitudes at every hole and 1e-5 of the
rms field, as for every field test (each FP32 term is within 84 roundings,
5e-6, of its value; pairs within 64 softening lengths are summed in FP64)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd
    return gccd


def clusters(m, seed):
    r = np.random.default_rng(seed)
    p = r.normal(0.0, 0.4, size=(3, 2 * m))
    p[0, m:] += 12.0
    return p + np.array([480.0, 480.0, 300.0])[:, None]


def field(g, d, p, tile):
    ctx = g.gccd_init(g.Params.from_device(d))
    try:
        g.gccd_set_tile(ctx, tile)
        g.gccd_load(ctx, *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
        return g.gccd_field(ctx, p.shape[1]).cpu().numpy()
    finally:
        g.gccd_destroy(ctx)


@pytest.mark.parametrize("tile", [64, 128, 256])
@pytest.mark.parametrize("m", [1, 15, 16, 17, 63, 65, 127, 129, 255, 257, 500])
def test_two_clusters(g, m, tile):
    import oracle
    from paper_2203_11043_amd import workloads as W
    p = clusters(m, 7000 + m)
    E = field(g, dict(W.DEVICE), p, tile)
    Eo, A = oracle.field(list(p), with_magnitude=True)
    dE = np.linalg.norm(E - Eo, axis=0)
    assert np.max(dE / A) <= TOL
    assert np.max(dE) <= TOL * np.sqrt(np.mean(np.sum(Eo * Eo, axis=0)))


@pytest.mark.parametrize("m", [40, 300])
def test_targets_that_are_no_sources(g, m):
    """Collected holes that do not repel: targets outnumber sources, so the
    targets' boxes are reduced from the positions instead of read from the list."""
    import oracle
    from paper_2203_11043_amd import workloads as W
    p = clusters(m, 7100 + m)
    p[2, ::3] = -0.5 - np.arange(p[2, ::3].size) * 1e-3   # collected at load
    E = field(g, dict(W.DEVICE, collected_are_sources=0), p, 0)
    Eo, A = oracle.field(list(p), list(p[:, p[2] > 0.0]), with_magnitude=True)
    dE = np.linalg.norm(E - Eo, axis=0)
    assert np.max(dE / A) <= TOL


def test_more_close_pairs_than_the_lists_hold(g):
    """700 holes within 50 nm: nearly every pair is one to be summed exactly, far
    more than a wave's list holds; the rest keep their FP32 terms."""
    import oracle
    from paper_2203_11043_amd import workloads as W
    r = np.random.default_rng(7200)
    p = r.uniform(0.0, 0.03, size=(3, 700)) + np.array([480.0, 480.0, 300.0])[:, None]
    E = field(g, dict(W.DEVICE), p, 0)
    Eo, A = oracle.field(list(p), with_magnitude=True)
    assert np.max(np.linalg.norm(E - Eo, axis=0) / A) <= TOL
