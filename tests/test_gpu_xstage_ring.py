"""X stage with many channels (four waves per workgroup) and several LDS chunks where a chunk fills its
share of the LDS: 80 stations and two below (two chunks hold the whole 80 KB), 40 and 39 (four chunks of
which two make a stage).  Whole and ragged last chunks; other data before each call, so that a chunk read
before it has landed holds wrong samples, not the right ones of the call before.

FP16-split: coherence error <= 1e-5, the bound of the 16-bit mode; a chunk missed or read twice is an error
of at least 32 / 512 of an auto-correlation.  Int8: exact integers.
"""

import numpy as np
import pytest

import oracle
from paper_1801_04834_amd import synth
from tests.layout import block, block_planes
from tests.metrics import coherence_error, vis_complex

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

_STATIONS = [39, 40, 78, 79, 80]


def _plan(S, n_c, st, mode):
    from paper_1801_04834_amd import binding
    return binding.plan_for(synth.Workload(name="xring", S=S, SB=5, sample_type=st, x_mode=mode, N=64 * n_c, sigma=64.0,
                                           seed=5, ripple=0.05, fp16_prescale_log2=-1 if mode == synth.X_FP16_SPLIT else 0))


@pytest.mark.parametrize("n_c", [64, 65, 257, 512])
@pytest.mark.parametrize("S", _STATIONS)
def test_fp16_ring(S, n_c):
    print(f"CASE xring fp16 S={S} n_c={n_c}", flush=True)
    with _plan(S, n_c, synth.CI16, synth.X_FP16_SPLIT) as plan:
        for seed in (1, 2):
            Z = synth.float_channelised(seed=1000 * seed + S + n_c, n_chan=320, M=2 * S, n_c=n_c, sigma=7.7)
            zs = np.stack([Z.real, Z.imag], -1) * 0.5
            hi = zs.astype(np.float16)
            lo = (zs - hi.astype(np.float64)).astype(np.float16)
            buf = np.full((2, 320, 2 * S, plan.pitch, 2), np.nan, np.float16)
            buf[0, :, :, :n_c] = hi
            buf[1, :, :, :n_c] = lo
            exact = (hi.astype(np.float64) + lo.astype(np.float64)) * 2.0
            V = plan.correlate_channelized(torch.from_numpy(block_planes(buf[0], buf[1]).reshape(plan.chan_shape)).cuda())
            torch.cuda.synchronize()
            ref = oracle.correlate(exact[..., 0] + 1j * exact[..., 1], S)
            eps = coherence_error(vis_complex(V.cpu().numpy()).reshape(ref.shape), ref, S)
            print(f"  eps={eps:.3e}", flush=True)
            assert eps <= 1e-5


@pytest.mark.parametrize("n_c", [64, 257, 512, 700])
@pytest.mark.parametrize("S", _STATIONS)
def test_int8_ring(S, n_c):
    print(f"CASE xring int8 S={S} n_c={n_c}", flush=True)
    with _plan(S, n_c, synth.CI8, synth.X_INT8) as plan:
        for seed in (1, 2):
            q = synth.int8_channelised(seed=1000 * seed + S + n_c, n_chan=320, M=2 * S, n_c=n_c, pitch=plan.pitch)
            ref = oracle.correlate_int(q[:, :, :n_c, :], S)
            q[:, :, n_c:] = 99
            V = plan.correlate_channelized(torch.from_numpy(block(q).reshape(plan.chan_shape)).cuda())
            torch.cuda.synchronize()
            assert np.array_equal(V.cpu().numpy().reshape(ref.shape).astype(np.int64), ref)
