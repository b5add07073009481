"""The time shift in the binary32 mode: k tau / T is thousands of revolutions,
of which only the fraction counts.  The shift per bin is a binary32 number;
its product with the bin number is not rounded before the fraction is taken."""

import numpy as np
import pytest

from oracle import detectors
from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over", [("paper_scale", {}), ("pr1_plain", {}), ("sine_gaussian", dict(t_window=16.0))])
def test_projection_phase(name, over):
    """Projection of h+ = 1, hx = 0: F+ fs exp(-2 pi i k t), t the binary32 value of tau / T, so the ratio of two bins
    does not depend on F+.  Tolerance 1e-6: the fraction's rounding (2^-25 revolutions, 2e-7 rad), the hardware sine's
    1.3e-7 twice, two binary32 roundings."""
    import torch
    cfg = inputs.config(name, precision=0, **over)
    gen = gwgen.Generator(cfg)
    z, B = gen.sizes, 32
    params = torch.empty((gwgen.N_PARAMS, B), dtype=torch.float64, device="cuda")
    offset = torch.empty(B, dtype=torch.int64, device="cuda")
    gen.sample_params(8, 0, B, 1 << 20, params, offset)
    hp = torch.ones((B, z["F"]), dtype=torch.complex64, device="cuda")
    hdet = torch.empty((B, z["D"], z["F"]), dtype=torch.complex64, device="cuda")
    gen.project_detectors(params, hp, torch.zeros_like(hp), hdet)
    torch.cuda.synchronize()
    got, p = hdet.cpu().numpy().astype(np.complex128), params.cpu().numpy()
    k = np.arange(z["F"])
    for d, det in enumerate(cfg["det_ids"]):
        _, vertex = detectors.detector_geometry(det)
        for i in range(B):
            tau = p[10, i] + detectors.time_delays(vertex, p[6, i], p[7, i])
            # (tau / T may lie within 1e-15 of a binary32 rounding boundary in one of 10^8 draws)
            t = float(np.float32(tau * (1.0 / cfg["t_window"])))
            want = np.exp(-2j * np.pi * np.remainder(k * t, 1.0))
            assert np.max(np.abs(got[i, d] / got[i, d, 0].real - want)) < 1e-6


def test_fused_burst_equals_the_steps():
    """The fused window and the six steps take the same fraction: whitened bursts agree to binary32's own rounding (two
    transforms more in the steps, 2e-7 each, and the hardware sines' 1.3e-7 in different sums: 2e-6 of the window)."""
    import torch
    cfg = inputs.config("sine_gaussian", precision=0, hrss=(1e-20, 2e-20))  # loud: most of the window is signal
    gen = gwgen.Generator(cfg)
    z, B = gen.sizes, 16
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 20, cfg["fs"], seed=5)).cuda()
    out = torch.empty((B, z["D"], z["N"]), dtype=torch.float32, device="cuda")
    ws = gen.alloc_workspace(B)
    gen.generate_batch(3, 0, B, bg, out, ws)
    params, offs = (t.clone() for t in gen.workspace_views(ws, B))
    hp = torch.empty((B, z["F"]), dtype=torch.complex64, device="cuda")
    hc = torch.empty_like(hp)
    hdet = torch.empty((B, z["D"], z["F"]), dtype=torch.complex64, device="cuda")
    strain = torch.empty_like(out)
    psd = torch.empty((B, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    steps = torch.empty_like(out)
    gen.gen_fd_waveform(params, hp, hc)
    gen.project_detectors(params, hp, hc, hdet)
    gen.inject(bg, offs, hdet, strain)
    gen.welch_psd(bg, offs, psd)
    gen.whiten(strain, psd, steps)
    torch.cuda.synchronize()
    a, b = out.double(), steps.double()
    assert float(((a - b).norm(dim=2) / b.norm(dim=2)).max()) < 2e-6
