"""The run PSD with the least workspace that is accepted: the chunks' PSDs,
averaged, as a call without room for a full set of shares makes them; bit for
bit the mean in binary64 of the same PSDs from welch_psd, rounded once.  With
the size that the query names, also for stretches of few pairs, the two agree
to the rounding of binary32 transforms (1e-6)."""

import ctypes

import numpy as np
import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over,chunks", [("paper_scale", {}, 4), ("paper_scale", dict(psd_length=16.0), 9),
                                              ("paper_scale", dict(psd_length=3.0), 3),
                                              ("paper_scale", dict(psd_length=3.0), 4), ("pr1_plain", dict(psd_length=5.0), 40)])
def test_least_workspace_averages_chunks(name, over, chunks):
    import torch
    gen = gwgen.Generator(inputs.config(name, **over))
    z = gen.sizes
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 20, gen.cfg["fs"], seed=4)).cuda()
    offs = torch.arange(chunks, device="cuda") * (z["K"] * z["L"] // 2)
    each = torch.empty((chunks, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    gen.welch_psd(bg, offs, each)
    want = each.double().mean(0).cpu().numpy()
    size = ctypes.c_int64()
    assert gwgen.lib().gw_run_psd_workspace_size(gen._h, chunks, ctypes.byref(size)) == 0
    least = -(-8 * chunks // 256) * 256 + -(-4 * chunks * z["D"] * z["Fw"] // 256) * 256
    got = []
    for nbytes in (least, size.value):
        ws = torch.empty(nbytes // 8, dtype=torch.float64, device="cuda")
        psd = torch.zeros((z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
        assert gwgen.lib().gw_run_psd(gen._h, gwgen._ptr(bg), bg.shape[1], chunks, gwgen._ptr(psd), gwgen._ptr(ws), nbytes,
                                      gwgen._stream()) == 0
        torch.cuda.synchronize()
        got.append(psd.cpu().numpy())
    if size.value > least:  # no room for the shares
        assert np.array_equal(got[0], want.astype(np.float32))
    assert np.max(np.abs(got[1] / want - 1.0)) <= 1e-6
