"""The closure's near sum of loads below 65536 holes: one wave per 64 targets and
chunk of source tiles, whose 16-source groups are listed by boxes and then tested
against each target.  Checked at the edges of a wave, a 256-hole block, the chunks
(7 tiles in one, 9 in two, the largest load) and for a cloud with far outliers,
whose waves span large boxes; and, with holes already collected (fewer targets
than sources), a step against the field of the same positions.

Tolerance: the Eq. (6) tolerance 1e-5 of the sum of term magnitudes, plus the
field of the sources within 1e-5 of the cutoff (their r^2 may round to either
side).  The step takes the same sums as the field but for the origin of a block
whose last slots are no targets: the same tolerance, 1e-5 of the largest field."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import closure as C

pytestmark = pytest.mark.gpu


def positions(kind):
    r = np.random.default_rng(7400)
    if kind == "outliers":
        p = r.normal(0.0, 0.8, size=(3, 9000))
        p[:, :40] *= 30.0
    else:
        p = r.normal(0.0, 0.2 * kind ** (1 / 3) / 5, size=(3, kind))
    return p + np.array([480.0, 480.0, 300.0])[:, None]


@pytest.mark.parametrize("kind", [2, 63, 65, 257, 1792, 2049, 9001, 65535, "outliers"])
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
    idx = np.random.default_rng(1).choice(n, min(n, 300), replace=False)
    if kind == "outliers":
        idx[:40] = np.arange(40)
    t, src = [v[idx] for v in p], list(p)
    Eo = oracle.field_window(t, src, 0.0, a)
    shell = oracle.field_window(t, src, a * (1 - 1e-5), a * (1 + 1e-5))
    _, A = oracle.field(t, src, with_magnitude=True)
    dn = np.linalg.norm(near[:, idx] - Eo, axis=0)
    assert np.all(dn <= 1e-5 * A + np.linalg.norm(shell, axis=0) + 1e-9)


def test_step_with_collected_holes():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import closure_eval
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W
    n, dt = 6000, 1.0
    p = positions(n)
    p[2] -= 299.5       # half of the cloud in the well
    d = dict(W.DEVICE, diffusion=0, mobility_model=1)
    ctx = g.gccd_init(g.Params.from_device(d))
    try:
        g.gccd_set_closure(ctx, closure_eval.load_weights(), 0)
        g.gccd_load(ctx, *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
        E = g.gccd_field(ctx, n).cpu().numpy()
        before, cstep = (v.cpu().numpy() for v in g.gccd_positions(ctx, n))
        g.gccd_run(ctx, dt, 1)
        after = g.gccd_positions(ctx, n)[0].cpu().numpy()
    finally:
        g.gccd_destroy(ctx)
    free = cstep < 0
    assert 500 < np.sum(free) < n - 500
    assert np.array_equal(before[:, ~free], after[:, ~free])
    # x and y move by mu E dt alone: one constant mu (cm^2/(V s)) for all holes
    dx = (after - before)[:2, free]
    Exy = E[:2, free]
    mu = np.sum(dx * Exy) / np.sum(Exy * Exy)
    assert mu > 0
    assert np.max(np.abs(dx / mu - Exy)) <= 1e-5 * np.max(np.linalg.norm(E[:, free], axis=0))
