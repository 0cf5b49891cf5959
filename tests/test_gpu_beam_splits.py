"""Beamformer with a channel's time split over workgroups and with one, two and four waves per
workgroup: parts of whole windows (windows of 3 K blocks, a short last part), ragged last blocks,
all outputs, against the oracle with the tolerances of the beamformer parity test (voltages 2e-5
rms; Stokes 2e-5 I + 1e-6 mean I)."""

import numpy as np
import pytest

from tests.test_gpu_beam import _check, _oracle, _say, _work

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,NB,n_c,n_int,n_stokes", [(5, 16, 480, 96, 1), (3, 1, 300, 4, 4), (8, 32, 129, 1, 1), (13, 40, 300, 2, 4),
                                                     (16, 64, 288, 96, 4), (20, 33, 260, 1, 1), (24, 64, 416, 32, 1),
                                                     (30, 10, 384, 64, 4), (48, 130, 288, 96, 1)])
def test_time_parts_and_waves(S, NB, n_c, n_int, n_stokes):
    from paper_1801_04834_amd import binding
    seed = 5100 + S + NB + n_c
    w = _work(S, 1, n_c, seed)
    dtau = np.random.default_rng(seed).uniform(-4e-6, 4e-6, (NB, S))
    _say(f"CASE beam parts S={S} NB={NB} n_c={n_c} n_int={n_int} n_stokes={n_stokes} seed={seed}")
    blocks = [w.block(0)]
    outs = _oracle(w, blocks, dtau, n_stokes, n_int)
    with binding.plan_for(w) as plan:
        cs, vs, isz = plan.beam_shapes(NB, n_stokes, n_int)
        coh = torch.full(cs, np.nan, dtype=torch.float32, device="cuda")
        volt = torch.full(vs, np.nan, dtype=torch.float32, device="cuda")
        inc = torch.full(isz, np.nan, dtype=torch.float32, device="cuda")
        plan.beamform(torch.from_numpy(blocks[0]).cuda(), w.delays(0), torch.from_numpy(dtau).cuda(), n_stokes, n_int,
                      coherent=coh, voltages=volt, incoherent=inc)
        torch.cuda.synchronize()
        _check("parts", coh.cpu().numpy(), volt.cpu().numpy(), inc.cpu().numpy(), outs[0])
