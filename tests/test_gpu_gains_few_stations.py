"""Gains of small arrays with several subbands, where one workgroup's entries belong to many channels (the
forward) and one wave holds a whole channel (the adjoint), and the sizes next to each size class of the
adjoint's LDS, against the oracle.

Tolerances: a gain-applied entry is two complex products in turn, sqrt(5) u each: 2.7e-7 of its magnitude,
taken as 3e-7; the gradient sums at most 4 S products, within 2e-6 of its largest magnitude (sqrt(4 S) u =
1.3e-6 at 128 stations).
"""

import numpy as np
import pytest

from oracle import gains as og
from paper_1801_04834_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,SB", [(1, 1), (1, 7), (2, 3), (3, 5), (4, 1), (5, 3), (15, 2), (16, 3), (32, 2), (48, 1), (127, 1)])
def test_against_oracle(S, SB):
    from paper_1801_04834_amd import binding
    print(f"CASE gains few S={S} SB={SB}", flush=True)
    rng = np.random.default_rng([S, SB])
    B = S * (S + 1) // 2
    cplx = lambda *shape: (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)  # noqa: E731
    v0, g, G = cplx(SB, 64, B, 4), cplx(SB, 64, 2 * S), cplx(SB, 64, B, 4)
    w = synth.Workload(name="gf", S=S, SB=SB, sample_type=synth.CI16, x_mode=synth.X_FP32, N=64 * 16, seed=3)
    with binding.plan_for(w) as plan:
        dev = [torch.from_numpy(a).cuda() for a in (v0, g, G)]
        fwd = plan.apply_gains(dev[0], dev[1])
        adj = plan.apply_gains_adjoint(*dev)
        torch.cuda.synchronize()
        want_f = og.apply_gains(v0, g, S)
        want = og.apply_gains_adjoint(v0, g, G, S)
        assert (np.abs(fwd.cpu().numpy() - want_f) <= 3e-7 * np.abs(want_f) + 1e-30).all()
        assert np.max(np.abs(adj.cpu().numpy() - want)) <= 2e-6 * np.max(np.abs(want))
