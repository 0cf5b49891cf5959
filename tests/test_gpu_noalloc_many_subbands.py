"""The plan-less call where the subband frequencies take several uploads, eager and captured into a graph:
equal to a plan's call on the same block, bit for bit, also when the caller's frequency array changes right
after the call.
"""

import numpy as np
import pytest

from paper_1801_04834_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("SB", [257, 1000, 2500])
def test_equal_to_plan(SB):
    from paper_1801_04834_amd import binding
    print(f"CASE noalloc subbands SB={SB}", flush=True)
    n_c = 20
    kw = dict(n_stations=1, n_subbands=SB, samples_per_block=64 * n_c, sample_type=binding.CI8, x_mode=binding.X_FP32,
              fir=synth.Workload(name="nm", S=1, SB=1, sample_type=synth.CI8, x_mode=synth.X_FP32, N=64).fir(),
              subband_freqs=np.linspace(110e6, 250e6, SB))
    gen = torch.Generator(device="cuda").manual_seed(SB)
    x = torch.randint(-60, 60, (1, 2, SB, 64 * n_c, 2), generator=gen, dtype=torch.int8, device="cuda")
    d = np.array([[1e-6, 3e-6]])
    with binding.Plan(**kw) as plan:
        want = plan.correlate(x, d)
    out = torch.full_like(want, float("nan"))
    freqs = kw["subband_freqs"] = kw["subband_freqs"].copy()
    binding.correlate_noalloc(x, d, out, **kw)
    keep = freqs.copy()
    freqs[:] = 0.0
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    freqs[:] = keep
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        binding.correlate_noalloc(x, d, out, **kw)
    freqs[:] = 0.0
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
