"""Loads on one context with closure runs and closure calls between them, whose
buffers grow past those that captured steps name, and loads of one shape whose list
is pipelined (from 5e9 pairs on): each as on a fresh context."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def cloud(n, seed):
    p = np.random.default_rng(seed).normal(0.0, 1.5, size=(3, n))
    return [torch.as_tensor(v).cuda() for v in p + np.array([[480.0], [480.0], [300.0]])]


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd
    return gccd


def test_closure_between_loads(g):
    from paper_2203_11043_amd import closure_eval
    weights = closure_eval.load_weights()
    kept = g.gccd_init(g.Params())
    # (holes, closure on, closure_parts called after the run)
    for k, (n, on, parts) in enumerate([(3000, 0, 0), (3000, 1, 0), (3000, 0, 1), (3000, 0, 0),
                                        (20000, 1, 1), (3000, 0, 0), (9000, 0, 1), (9000, 0, 0),
                                        (70001, 1, 0), (9000, 0, 0)]):
        p = cloud(n, 8300 + k)
        fresh = g.gccd_init(g.Params())
        out = []
        for ctx in (kept, fresh):
            g.gccd_set_closure(ctx, weights if on else None, 0)
            g.gccd_load(ctx, *p)
            g.gccd_run(ctx, 10.0, 70 if n < 10000 else 3)
            out.append(list(g.gccd_positions(ctx, n)))
            if parts:
                out[-1] += list(g.gccd_closure_parts(ctx, n))
                g.gccd_run(ctx, 10.0, 34)  # past the next capture's start
                out[-1] += list(g.gccd_positions(ctx, n))
        for u, v in zip(*out):
            assert torch.equal(u, v)
        g.gccd_destroy(fresh)
    g.gccd_destroy(kept)


def test_pipelined_loads(g):
    n = 75000
    kept = g.gccd_init(g.Params())
    replays = []
    for k in range(3):
        p = cloud(n, 8400 + k)
        fresh = g.gccd_init(g.Params())
        for ctx in (kept, fresh):
            g.gccd_load(ctx, *p)
            g.gccd_run(ctx, 10.0, 67)
        for u, v in zip(g.gccd_positions(kept, n), g.gccd_positions(fresh, n)):
            assert torch.equal(u, v)
        s = g.gccd_stats(kept)
        assert s["graph_usable"] == 1
        replays.append(s["graph_replays"])
        g.gccd_destroy(fresh)
    assert replays == [2, 4, 6]
    g.gccd_destroy(kept)
