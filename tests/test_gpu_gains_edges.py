"""Gain adjoint around the wave boundaries of its workgroup (16 stations per wave) and at the largest
station counts, against the oracle: sums of at most 4 S products in FP32, so the gradient is within
2e-6 of its largest magnitude (4 S u with u = 2^-24 is 3e-5 at worst for S = 128; the rounding errors
add up like sqrt(4 S) u = 1.3e-6)."""

import numpy as np
import pytest

from oracle import gains as og
from paper_1801_04834_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,mode", [(15, synth.X_FP16_SPLIT), (16, synth.X_FP16_SPLIT), (17, synth.X_FP16_SPLIT),
                                    (33, synth.X_FP16_SPLIT), (64, synth.X_FP32), (65, synth.X_FP32), (128, synth.X_FP32)])
def test_adjoint_edges(S, mode):
    from paper_1801_04834_amd import binding
    print(f"CASE gains edges S={S}", flush=True)
    rng = np.random.default_rng(S)
    B = S * (S + 1) // 2
    cplx = lambda *shape: (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)  # noqa: E731
    v0, g, G = cplx(1, 64, B, 4), cplx(1, 64, 2 * S), cplx(1, 64, B, 4)
    w = synth.Workload(name="ge", S=S, SB=1, sample_type=synth.CI16, x_mode=mode, N=64 * 16, seed=3,
                       fp16_prescale_log2=-1 if mode == synth.X_FP16_SPLIT else 0)
    with binding.plan_for(w) as plan:
        dev = [torch.from_numpy(a).cuda() for a in (v0, g, G)]
        fwd = plan.apply_gains(dev[0], dev[1])
        adj = plan.apply_gains_adjoint(*dev)
        torch.cuda.synchronize()
        want_f = og.apply_gains(v0, g, S)
        want = og.apply_gains_adjoint(v0, g, G, S)
        assert np.max(np.abs(fwd.cpu().numpy() - want_f)) <= 2e-6 * np.max(np.abs(want_f))
        assert np.max(np.abs(adj.cpu().numpy() - want)) <= 2e-6 * np.max(np.abs(want))
