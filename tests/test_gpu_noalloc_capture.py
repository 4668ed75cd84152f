"""gccd_field_noalloc recorded into a HIP graph: the queries it makes about its
source pointers (to read them without a copy) have to be allowed while a stream
captures, and a replay has to read the sources' values at that time.  Replayed
several times with other eager work between, each against the eager call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 12289])
def test_captured_call(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_11043_amd import gccd as g
    from paper_2203_11043_amd import workloads as W

    params = g.Params.from_device(dict(W.DEVICE))

    def cloud(seed):
        p = W.gaussian_cloud(n, W.cloud_sigma(n), (480.0, 480.0, 300.0), seed, stream=n)
        return [torch.as_tensor(np.ascontiguousarray(v)).cuda() for v in p]

    xyz = cloud(1)
    out = torch.empty((3, n), dtype=torch.float64, device="cuda")
    g.gccd_field_noalloc(params, *xyz, out=out)  # the first call loads the code
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.gccd_field_noalloc(params, *xyz, out=out)
    for seed in (2, 3, 2):
        new = cloud(seed)
        for a, b in zip(xyz, new):
            a.copy_(b)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        want = g.gccd_field_noalloc(params, *new, out=torch.empty_like(out))
        torch.cuda.synchronize()
        assert torch.equal(got, want)
