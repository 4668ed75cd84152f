"""The closure's near sum of loads of at least 65536 holes takes the matrix
kernel: 16-source groups within a of a workgroup's targets are listed and staged
sixteen at a time, far blocks of 16 targets and 16 sources take r^2 from the matrix
cores, near ones differences, and the cutoff is a factor of 0 or 1.  Its near
part is compared with the oracle's windowed sum: a load of exactly the smallest
size, an odd one, and one with a dense clump and a distant cluster (groups of
very different extent, blocks out of reach of all others).

Tolerance: the Eq. (6) tolerance 1e-5 of the sum of term magnitudes, plus the
field of the sources within 1e-5 of the cutoff (their r^2 may round to either
side), as for the smaller loads."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import closure as C

pytestmark = pytest.mark.gpu


def positions(kind):
    r = np.random.default_rng(7300)
    if kind == "clump":
        p = np.concatenate([r.normal(0.0, 2.0, size=(3, 64000)),
                            r.normal(0.0, 0.03, size=(3, 400)) + 1.0,
                            r.normal(0.0, 0.4, size=(3, 1700)) + np.array([[40.0], [0.0], [0.0]])],
                           axis=1)
    else:
        p = r.normal(0.0, 2.0, size=(3, kind))
    return p + np.array([480.0, 480.0, 300.0])[:, None]


@pytest.mark.parametrize("kind", [65536, 70001, "clump"])
def test_near_part(kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W
    p = positions(kind)
    n = p.shape[1]
    ctx = g.gccd_init(g.Params.from_device(dict(W.DEVICE)))
    try:
        g.gccd_load(ctx, *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
        near, _, _, grid = g.gccd_closure_parts(ctx, n)
        near, h = near.cpu().numpy(), float(grid[3])
    finally:
        g.gccd_destroy(ctx)
    a = C.NEAR_CELLS * h
    idx = np.random.default_rng(1).choice(n, 300, replace=False)
    if kind == "clump":
        idx[:60] = 64000 + np.arange(60) * 35   # clump and distant cluster
    t, src = [v[idx] for v in p], list(p)
    Eo = oracle.field_window(t, src, 0.0, a)
    shell = oracle.field_window(t, src, a * (1 - 1e-5), a * (1 + 1e-5))
    _, A = oracle.field(t, src, with_magnitude=True)
    dn = np.linalg.norm(near[:, idx] - Eo, axis=0)
    assert np.all(dn <= 1e-5 * A + np.linalg.norm(shell, axis=0) + 1e-9)
