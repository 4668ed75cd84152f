"""Sums of far blocks of the default Eq. (6) kernel at targets that are no
sources, whose field is a sum of coherent far terms only: neither cancellation
nor near terms hide an error.  u = 2^-24."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
WELL = 300.0


def far_field(p, offsets, launch=(0, 0)):
    """gccd_field of holes above z = WELL at those and at the collected ones below."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    # (no mirror in reach of the sources)
    ctx = g.gccd_init(g.Params(thickness_um=1e7, well_z_um=WELL, collected_are_sources=0))
    try:
        g.gccd_set_launch(ctx, *launch)
        g.gccd_load_events(ctx, offsets,
                           *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
        return g.gccd_field(ctx, offsets[-1]).cpu().numpy()
    finally:
        g.gccd_destroy(ctx)


def test_many_tiles():
    """One chunk of 512 source tiles.  The tiles are added in FP64, so what is left is
    the rounding of each tile's FP32 sums (about 2 u at random, 0.1 u over 512
    tiles), of the result (u / 2) and the mean rounding of r^-3: 4 u in all with a
    margin of several.  (Added in FP32, 512 roundings of a growing sum: about 6 u
    rms, and the largest of 256 targets beyond 10 u.)"""
    import oracle
    r = np.random.default_rng(7400)
    src = r.normal(0.0, 5.0, size=(3, 131072)) + np.array([[480.0], [480.0], [400.0]])
    tgt = r.normal(0.0, 0.5, size=(3, 256)) + np.array([[480.0], [480.0], [WELL - 4.0]])
    E = far_field(np.concatenate([src, tgt], axis=1), [0, 131072 + 256], (1, 1))
    Eo, A = oracle.field(list(tgt), list(src), with_magnitude=True)
    assert np.max(np.linalg.norm(E[:, 131072:] - Eo, axis=0) / A) <= 4 * U


def on_an_axis(gap, m, events, seed):
    """Events of 256 targets along a random axis, their half-diagonal rho, and m sources
    on the same axis beyond its end, at the given gap in units of rho; 256 - m more
    travelling holes fill the sources' block, too far away to matter."""
    r = np.random.default_rng(seed)
    parts, rho = [], 8.0
    for _ in range(events):
        u = r.normal(size=3)
        u[2] = abs(u[2]) + 0.3
        u /= np.linalg.norm(u)
        side = np.linalg.svd(u[None])[2][1:]
        a = r.uniform(-rho, rho, 256)
        a[:2] = -rho, rho
        t = u[:, None] * a + side.T @ r.normal(0.0, 0.004 * rho, size=(2, 256))
        s = (u[:, None] * (rho * (1 + gap) + r.uniform(0.0, 0.02 * rho, m)) +
             side.T @ r.normal(0.0, 0.004 * rho, size=(2, m)))
        fill = u[:, None] * r.uniform(2e5, 4e5, 256 - m)
        c = np.array([480.0, 480.0, WELL])[:, None] - u[:, None] * 1.3 * rho
        t, s, fill = c + t, c + s, c + fill
        t[2] = np.minimum(t[2], WELL - 1e-3)
        s[2] = np.maximum(s[2], WELL + 1e-3)
        parts.append(np.concatenate([s, fill, t], axis=1))
    return parts


@pytest.mark.parametrize("gap", [0.15, 0.21, 0.3, 0.45, 0.58, 0.75, 1.05])
@pytest.mark.parametrize("m", [1, 16])
def test_at_the_limits(gap, m):
    """Gaps below and above rho / 4 and 4 rho / 7, where the form of a block changes, with
    targets at the rim and sources beyond it: the partial results of r^2 are then as
    large, and the coordinates as coarse, against the distance as they get.  The
    bound of a single term is 84 u; the sum of m of them adds m - 1 roundings."""
    import oracle
    events = on_an_axis(gap, m, 120, 7500)
    offsets = [512 * e for e in range(len(events) + 1)]
    E = far_field(np.concatenate(events, axis=1), offsets)
    worst = 0.0
    for e, p in enumerate(events):
        Eo, A = oracle.field(list(p[:, 256:]), list(p[:, :256]), with_magnitude=True)
        dE = E[:, offsets[e] + 256:offsets[e + 1]] - Eo
        worst = max(worst, float(np.max(np.linalg.norm(dE, axis=0) / A)))
    print(f"[far limit] gap {gap} rho, {m} sources: {worst:.2e}", flush=True)
    assert worst <= (84 + m - 1) * U
