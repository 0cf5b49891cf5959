"""X stage on blocks of one or two LDS chunks, few and many channels: up to 16 stations a channel has one
wave (FP16-split to 32, int8 to 128 channel samples), in FP32 mode up to 64 samples no wave splits the
k-steps.  Against the oracle.

FP32: every sum has at most 128 products per part, coherence error <= 1e-6; FP16-split <= 1e-5, the bound of
the 16-bit mode; int8: exact integers.  Positions past N_c hold NaN (int8: 99): they must not enter the sums.
"""

import numpy as np
import pytest

import oracle
from paper_1801_04834_amd import synth
from tests.layout import block, block_planes
from tests.metrics import coherence_error, vis_complex

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _plan(S, SB, n_c, st, mode):
    from paper_1801_04834_amd import binding
    return binding.plan_for(synth.Workload(name="xshort", S=S, SB=SB, sample_type=st, x_mode=mode, N=64 * n_c, sigma=64.0, seed=5))


def _run(plan, buf):
    V = plan.correlate_channelized(torch.from_numpy(buf.reshape(plan.chan_shape)).cuda())
    torch.cuda.synchronize()
    return V.cpu().numpy()


@pytest.mark.parametrize("S,SB", [(1, 5), (5, 1), (8, 5), (13, 5), (16, 1), (17, 5), (29, 5)])
@pytest.mark.parametrize("n_c", [1, 32, 33, 64, 65])
def test_float_modes(S, SB, n_c):
    print(f"CASE xshort S={S} SB={SB} n_c={n_c}", flush=True)
    Z = synth.float_channelised(seed=S * 19 + n_c, n_chan=64 * SB, M=2 * S, n_c=n_c, sigma=7.7)
    zs = np.stack([Z.real, Z.imag], -1)
    with _plan(S, SB, n_c, synth.CI16, synth.X_FP32) as plan:
        buf = np.full((64 * SB, 2 * S, plan.pitch, 2), np.nan, np.float32)
        buf[:, :, :n_c] = zs
        z32 = buf[:, :, :n_c].astype(np.float64)
        ref = oracle.correlate(z32[..., 0] + 1j * z32[..., 1], S)
        eps = coherence_error(vis_complex(_run(plan, block(buf))).reshape(ref.shape), ref, S)
        assert eps <= 1e-6
    with _plan(S, SB, n_c, synth.CF32, synth.X_FP16_SPLIT) as plan:
        hi = zs.astype(np.float16)
        lo = (zs - hi.astype(np.float64)).astype(np.float16)
        buf = np.full((2, 64 * SB, 2 * S, plan.pitch, 2), np.nan, np.float16)
        buf[0, :, :, :n_c] = hi
        buf[1, :, :, :n_c] = lo
        exact = hi.astype(np.float64) + lo.astype(np.float64)
        ref = oracle.correlate(exact[..., 0] + 1j * exact[..., 1], S)
        eps = coherence_error(vis_complex(_run(plan, block_planes(buf[0], buf[1]))).reshape(ref.shape), ref, S)
        assert eps <= 1e-5


@pytest.mark.parametrize("S,SB", [(1, 5), (5, 1), (8, 5), (13, 5), (16, 1), (17, 5), (29, 5)])
@pytest.mark.parametrize("n_c", [1, 40, 128, 129])
def test_int8(S, SB, n_c):
    print(f"CASE xshort int8 S={S} SB={SB} n_c={n_c}", flush=True)
    with _plan(S, SB, n_c, synth.CI8, synth.X_INT8) as plan:
        q = synth.int8_channelised(seed=S * 23 + n_c, n_chan=64 * SB, M=2 * S, n_c=n_c, pitch=plan.pitch)
        ref = oracle.correlate_int(q[:, :, :n_c, :], S)
        q[:, :, n_c:] = 99
        assert np.array_equal(_run(plan, block(q)).reshape(ref.shape).astype(np.int64), ref)
