"""Whitening with a given PSD that falls by almost 10^4 between neighbouring bins and
rises again, as at the edges of a spectral line's gap: the gain of the window
bins on both edges against binary64.  The input is one unit impulse, whose
spectrum has modulus 1, so the output's spectrum is the gain.

Tolerance 1e-6.  The interpolated PSD carries two binary32 roundings (half of
their size in its root), the reciprocal root one unit in the last place, the
common factors three roundings: 4e-7 together; the transforms leave less than
half of the rest on these bins, whose gains are the largest (binary32
transforms of the same input on the CPU: 4.4e-7 in all).  Only these bins are
compared: a transform's error scales with its strongest bins."""

import numpy as np
import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,t_window,order,ratio", [("paper_scale", 16.0, 0, 8), ("paper_scale", 16.0, 1, 8),
                                                       ("bns_long", 256.0, 0, 128), ("bns_long", 256.0, 1, 128),
                                                       ("bns_long", 512.0, 1, 256)])
def test_gain_at_steep_edges(name, t_window, order, ratio):
    import torch
    gen = gwgen.Generator(inputs.config(name, t_window=t_window))
    gen.set_tuning(gwgen.TUNE_ORD_WINDOW, order)
    z = gen.sizes
    assert z["N"] // z["L"] == ratio
    psd = np.ones((1, z["D"], z["Fw"]), dtype=np.float32)
    low = [97 + 211 * d for d in range(z["D"])]
    for d, j in enumerate(low):
        psd[0, d, j] = 1.1e-4
    strain = torch.zeros((1, z["D"], z["N"]), dtype=torch.float32, device="cuda")
    strain[:, :, 12345] = 1.0
    out = torch.empty_like(strain)
    gen.whiten(strain, torch.from_numpy(psd).cuda(), out)
    torch.cuda.synchronize()
    got = np.abs(np.fft.rfft(out.cpu().numpy()[0].astype(np.float64)))
    for d, j in enumerate(low):
        k = np.arange((j - 1) * ratio, (j + 1) * ratio)
        i = k // ratio
        t = (k - i * ratio) / ratio
        s = psd[0, d].astype(np.float64)
        want = 1.0 / np.sqrt(gen.cfg["fs"] / 2 * ((1 - t) * s[i] + t * s[i + 1]))
        assert k[0] / t_window >= gen.cfg["f_min"]
        assert np.max(np.abs(got[d][k] / want - 1.0)) < 1e-6
