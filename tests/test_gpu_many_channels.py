"""More channels than one launch holds work-items for (one station, 65537 subbands, one channel
sample): the plain FP32 X stage and the gain application against the definitions on the GPU.

Tolerances (references in 64 bits, u = 2^-24): a visibility here is one complex product on matrix
units that round towards zero, two products and one sum of at most 2 u each: 6 u = 3.6e-7 of
|z_a| |z_b|, taken as 4e-7; a gain-applied entry is two complex products in turn, sqrt(5) u each:
2.7e-7 of its magnitude, taken as 3e-7.
"""

import pytest

from paper_1801_04834_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_fp32_and_gains_past_one_launch():
    from paper_1801_04834_amd import binding
    print("CASE many channels S=1 SB=65537", flush=True)
    w = synth.Workload(name="many", S=1, SB=65537, sample_type=synth.CI8, x_mode=synth.X_FP32, N=64, seed=9)
    n = w.SB * 64
    with binding.plan_for(w) as plan:
        gen = torch.Generator(device="cuda").manual_seed(9)
        chan = plan.empty_chan()
        assert chan.dtype == torch.float32 and chan.numel() == n * 2 * 32 * 2
        chan.fill_(float("nan"))
        rows = chan.view(n, 2, 32, 2)
        rows[:, :, 0] = torch.randn((n, 2, 2), generator=gen, device="cuda")
        z = torch.view_as_complex(rows[:, :, 0].contiguous())
        vis = plan.correlate_channelized(chan)
        torch.cuda.synchronize()
        v = vis if vis.is_complex() else torch.view_as_complex(vis.contiguous())
        v = v.reshape(n, 2, 2)
        z = z.to(torch.complex128)
        want = z[:, :, None] * z[:, None, :].conj()
        size = z.abs()[:, :, None] * z.abs()[:, None, :]
        assert bool(((v - want).abs() <= 4e-7 * size + 1e-30).all())
        g = torch.randn((n, 2, 2), generator=gen, device="cuda")
        g = torch.view_as_complex(g)
        out = plan.apply_gains(v.reshape(w.SB, 64, 1, 4), g.reshape(w.SB, 64, 2))
        torch.cuda.synchronize()
        g = g.to(torch.complex128)
        gw = g[:, :, None] * g[:, None, :].conj() * v
        assert bool(((out.reshape(n, 2, 2) - gw).abs() <= 3e-7 * gw.abs() + 1e-30).all())
