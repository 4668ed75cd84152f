"""The field of a load with holes whose position is not finite (one, or whole blocks of
them), at every hole, in every mode: what Eq. (6) gives.  A NaN in any coordinate makes every component of
every hole's field NaN (r of each pair holds it); an infinite coordinate makes that
component NaN (inf times 0)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("holes", [1, 300])
@pytest.mark.parametrize("mode", ["default", "block", "event", "absolute", "compensated", "fp64"])
def test_field(mode, holes, axis, value):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    n = 700
    p = np.random.default_rng(7900).normal(0.0, 0.5, size=(3, n)) + 300.0
    p[axis, 33:33 + holes] = value
    ctx = g.gccd_init(g.Params())
    g.gccd_set_precision(ctx, mode)
    g.gccd_load(ctx, *[torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p])
    E = g.gccd_field(ctx, n).cpu().numpy()
    g.gccd_destroy(ctx)
    assert np.all(np.isnan(E if np.isnan(value) else E[axis]))
