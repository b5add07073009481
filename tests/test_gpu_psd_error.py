"""A binary32 Welch PSD's error against binary64.  A twiddle's rounding is the
same in every segment, so this part of the error does not average out: with
the best rounding of each twiddle it is 4.7e-8 of the PSD's norm (emulated on
the CPU at 4096 points; 4.3e-8 at 2048), and the result's own rounding 3.5e-8,
5.9e-8 together; a fifth more is allowed."""

import numpy as np
import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ("paper_scale", "pr1_plain"))
def test_psd_error(name):
    import torch
    cfg = inputs.config(name)
    gen = gwgen.Generator(cfg)
    z = gen.sizes
    bg = inputs.background(z["D"], 1 << 20, cfg["fs"], seed=6)
    offs = np.arange(8) * 12345
    psd = torch.empty((8, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    gen.welch_psd(torch.from_numpy(bg).cuda(), torch.from_numpy(offs).cuda(), psd)
    torch.cuda.synchronize()
    got = psd.cpu().numpy().astype(np.float64)
    L = z["L"]
    w = np.sin(np.pi * np.arange(L) / L) ** 2
    errors = []
    for i, o in enumerate(offs):
        for d in range(z["D"]):
            seg = np.lib.stride_tricks.sliding_window_view(bg[d, o:o + z["P"]].astype(np.float64), L)[::L // 2][:z["K"]]
            want = (np.abs(np.fft.rfft(seg * w)) ** 2).mean(0) / (cfg["fs"] * (w ** 2).sum())
            want[1:-1] *= 2
            errors.append(np.linalg.norm(got[i, d] - want) / np.linalg.norm(want))
    assert np.sqrt(np.mean(np.square(errors))) < 1.2 * 5.9e-8
