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
