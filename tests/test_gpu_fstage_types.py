"""The F stage's output for equal samples held in 8-bit, 16-bit and float storage.

FP16-split planes are the same bits for every storage type (one arithmetic, exact conversions).  Requantised
output of long blocks is pinned by digest: a change of one fused product anywhere in the chain flips about
one value in 2e6, too few for the oracle's rounding tolerance to show; the digests are those of
the conversion before packed words too (parity unpinned: no outside reference rounds in FP32 as it does).
"""

import hashlib

import numpy as np
import pytest

from paper_1801_04834_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _channelise(st, mode, C, S, SB, n_c):
    from paper_1801_04834_amd import binding
    v = np.random.default_rng([7, C]).integers(-100, 101, (S, 2, SB, C * n_c, 2), dtype=np.int16)
    w = synth.Workload(name="types", S=S, SB=SB, sample_type=st, x_mode=mode, N=C * n_c, C=C, seed=5, ripple=0.05,
                       delay_spread_s=5e-6, delay_drift_s=25e-9)
    with binding.plan_for(w, fp16_prescale_log2=-1 if mode == synth.X_FP16_SPLIT else 0, requant_gain=3.0) as plan:
        out = plan.channelize(torch.from_numpy(v.astype(synth.storage_dtype(st))).cuda(), w.delays(0))
        torch.cuda.synchronize()
        return out.cpu().numpy()


@pytest.mark.parametrize("C,n_c", [(64, 700), (256, 300)])
def test_fp16_split_is_the_same_for_every_type(C, n_c):
    print(f"CASE fstage types C={C}", flush=True)
    a, b, c = (_channelise(st, synth.X_FP16_SPLIT, C, 4, 4, n_c).view(np.uint16) for st in (synth.CI8, synth.CI16, synth.CF32))
    assert np.array_equal(a, b)
    assert np.array_equal(a, c)


@pytest.mark.parametrize("st,digest", [(synth.CI8, "dce98cadd18e"), (synth.CI16, "5854efd7e4fb")])
def test_requantised_values_stay(st, digest):
    print(f"CASE fstage requantised digest st={st}", flush=True)
    out = _channelise(st, synth.X_INT8, 64, 6, 4, 3072)
    assert hashlib.sha256(out.tobytes()).hexdigest()[:12] == digest
