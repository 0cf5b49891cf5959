"""X stage at the edges of its work splits: row-block remainders, channel samples around a K
block, a k-step and a fold, one and several workgroups per channel, few and many channels; each
against the oracle.

Tolerances: FP32 mode, coherence error <= 1e-6 (blocked accumulation over 128 channel samples:
u (128 / sqrt(N_c) + sqrt(N_c / 128)) / 6 with u = 2^-24, at most 3e-7 rms for the sizes here).
Positions past N_c hold NaN: they must not enter the sums.
"""

import sys

import numpy as np
import pytest

import oracle
from paper_1801_04834_amd import synth
from tests.layout import block, block_planes
from tests.metrics import coherence_error, vis_complex

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _plan(S, SB, n_c, st, mode):
    from paper_1801_04834_amd import binding
    return binding.plan_for(synth.Workload(name="xsplit", S=S, SB=SB, sample_type=st, x_mode=mode, N=64 * n_c, sigma=64.0,
                                           seed=5, ripple=0.05, fp16_prescale_log2=-1 if mode == synth.X_FP16_SPLIT else 0))


@pytest.mark.parametrize("S,SB,n_c", [(1, 1, 1), (7, 1, 31), (8, 1, 33), (9, 5, 129), (16, 1, 255), (17, 1, 64), (24, 5, 257),
                                      (33, 1, 40), (41, 1, 8), (56, 1, 72), (73, 1, 39), (80, 5, 24), (97, 1, 65), (128, 5, 17)])
def test_fp32_splits(S, SB, n_c):
    _say(f"CASE xsplit fp32 S={S} SB={SB} n_c={n_c}")
    with _plan(S, SB, n_c, synth.CI16, synth.X_FP32) as plan:
        Z = synth.float_channelised(seed=S * 11 + n_c, n_chan=64 * SB, M=2 * S, n_c=n_c)
        buf = np.full((64 * SB, 2 * S, plan.pitch, 2), np.nan, np.float32)
        buf[:, :, :n_c, 0] = Z.real
        buf[:, :, :n_c, 1] = Z.imag
        V = plan.correlate_channelized(torch.from_numpy(block(buf).reshape(plan.chan_shape)).cuda())
        torch.cuda.synchronize()
        ref = oracle.correlate(Z, S)
        eps = coherence_error(vis_complex(V.cpu().numpy()).reshape(ref.shape), ref, S)
        _say(f"  eps={eps:.3e}")
        assert eps <= 1e-6


_EDGES = [(1, 1, 1), (7, 1, 31), (8, 5, 33), (9, 1, 129), (16, 5, 47), (17, 1, 300), (24, 5, 257), (25, 1, 16), (33, 5, 40),
          (40, 1, 8), (41, 5, 130), (56, 1, 72), (57, 5, 33), (64, 1, 200), (65, 5, 39), (73, 1, 300), (80, 5, 24)]


@pytest.mark.parametrize("S,SB,n_c", _EDGES)
def test_fp16_splits(S, SB, n_c):
    """Coherence error <= 1e-5, the bound of the 16-bit mode (every product exact in FP32, sums of at
    most 300 samples: rounding stays near 1e-6)."""
    _say(f"CASE xsplit fp16 S={S} SB={SB} n_c={n_c}")
    with _plan(S, SB, n_c, synth.CI16, synth.X_FP16_SPLIT) as plan:
        Z = synth.float_channelised(seed=S * 13 + n_c, n_chan=64 * SB, M=2 * S, n_c=n_c, sigma=7.7)
        zs = np.stack([Z.real, Z.imag], -1) * 0.5
        hi = zs.astype(np.float16)
        lo = (zs - hi.astype(np.float64)).astype(np.float16)
        buf = np.full((2, 64 * SB, 2 * S, plan.pitch, 2), np.nan, np.float16)
        buf[0, :, :, :n_c] = hi
        buf[1, :, :, :n_c] = lo
        exact = (hi.astype(np.float64) + lo.astype(np.float64)) * 2.0
        V = plan.correlate_channelized(torch.from_numpy(block_planes(buf[0], buf[1]).reshape(plan.chan_shape)).cuda())
        torch.cuda.synchronize()
        ref = oracle.correlate(exact[..., 0] + 1j * exact[..., 1], S)
        eps = coherence_error(vis_complex(V.cpu().numpy()).reshape(ref.shape), ref, S)
        _say(f"  eps={eps:.3e}")
        assert eps <= 1e-5


@pytest.mark.parametrize("S,SB,n_c", _EDGES)
def test_int8_splits(S, SB, n_c):
    """Exact integers."""
    _say(f"CASE xsplit int8 S={S} SB={SB} n_c={n_c}")
    with _plan(S, SB, n_c, synth.CI8, synth.X_INT8) as plan:
        q = synth.int8_channelised(seed=S * 17 + n_c, n_chan=64 * SB, M=2 * S, n_c=n_c, pitch=plan.pitch)
        ref = oracle.correlate_int(q[:, :, :n_c, :], S)
        q[:, :, n_c:] = 99
        V = plan.correlate_channelized(torch.from_numpy(block(q).reshape(plan.chan_shape)).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(V.cpu().numpy().reshape(ref.shape).astype(np.int64), ref)
