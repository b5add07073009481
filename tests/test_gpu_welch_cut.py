"""Batches whose Welch stage divides its stretches over the workgroups (few or
unevenly many of them) against the stage that gives each stretch to one
workgroup: one sample, odd and even segment counts, a single pair, both segment
lengths, binary64, and a batch that cuts across many stretches.

Tolerance: the pieces' sums are added in binary64 and rounded once to binary32,
as the whole sum is, so a PSD bin may differ by one binary32 rounding (2^-24
relative) at most."""

import numpy as np
import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu

CASES = [("paper_scale", {}, 1), ("paper_scale", {}, 301), ("paper_scale", dict(psd_length=33.0), 7),
         ("paper_scale", dict(psd_length=3.0), 260), ("paper_scale", dict(precision=2), 40),
         ("paper_scale", dict(t_window=32.0), 5), ("pr1_plain", {}, 64), ("pr1_plain", dict(psd_length=2.0), 3),
         ("pr1_plain", dict(psd_length=20.0, precision=2), 33), ("pr1_short", dict(psd_length=17.0), 901)]


@pytest.mark.parametrize("name,over,B", CASES)
def test_cut_stretches_equal_whole_ones(name, over, B):
    import torch
    cfg = inputs.config(name, **over)
    gen = gwgen.Generator(cfg)
    z = gen.sizes
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 20, cfg["fs"], seed=3)).cuda()
    out = torch.empty((B, z["D"], z["N"]), dtype=torch.float32, device="cuda")
    ws = gen.alloc_workspace(B)
    status = torch.empty(B, dtype=torch.int32, device="cuda")
    gen.generate_batch(11, 2, B, bg, out, ws, status=status)
    _, offs = gen.workspace_views(ws, B)
    # the six-step call has no workspace and never cuts a stretch
    whole = torch.empty((B, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    gen.welch_psd(bg, offs.clone(), whole)
    torch.cuda.synchronize()
    at = -(-96 * B // 256) * 256 + -(-8 * B // 256) * 256
    psd = ws.view(torch.uint8)[at:at + whole.numel() * 4].view(torch.float32).view(whole.shape)
    a, b = psd.cpu().numpy().astype(np.float64), whole.cpu().numpy().astype(np.float64)
    assert np.all(b > 0)
    assert np.max(np.abs(a / b - 1.0)) <= 2.0 ** -23
    # a second pass on the same workspace, whose slots hold the first one's sums
    first = out.clone()
    gen.generate_batch(11, 2, B, bg, out, ws, status=status)
    torch.cuda.synchronize()
    assert torch.equal(first, out)


@pytest.mark.parametrize("name,over,chunks", [("paper_scale", dict(psd_length=16.0), 9), ("pr1_plain", {}, 1),
                                              ("pr1_plain", dict(psd_length=5.0), 40),
                                              ("paper_scale", dict(psd_length=8.0, precision=2), 21)])
def test_run_psd_whatever_the_workspace(name, over, chunks):
    """The run PSD with the workspace the query names and with the least that is accepted (fewer shares), against the
    mean of the chunks' PSDs in binary64 (each rounded to binary32: 2^-24 relative, as the result is)."""
    import ctypes

    import torch
    cfg = inputs.config(name, **over)
    gen = gwgen.Generator(cfg)
    z = gen.sizes
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 20, cfg["fs"], seed=4)).cuda()
    offs = torch.arange(chunks, device="cuda") * (z["K"] * z["L"] // 2)
    each = torch.empty((chunks, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    gen.welch_psd(bg, offs, each)
    want = each.double().mean(0).cpu().numpy()
    size = ctypes.c_int64()
    assert gwgen.lib().gw_run_psd_workspace_size(gen._h, chunks, ctypes.byref(size)) == 0
    least = -(-8 * chunks // 256) * 256 + -(-4 * chunks * z["D"] * z["Fw"] // 256) * 256
    for nbytes in (size.value, least):
        ws = torch.empty(nbytes // 8, dtype=torch.float64, device="cuda")
        psd = torch.zeros((z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
        assert gwgen.lib().gw_run_psd(gen._h, gwgen._ptr(bg), bg.shape[1], chunks, gwgen._ptr(psd), gwgen._ptr(ws), nbytes,
                                      gwgen._stream()) == 0
        torch.cuda.synchronize()
        # binary32 transforms pair other segments than the chunks do: 1e-6 covers their rounding
        assert np.max(np.abs(psd.cpu().numpy() / want - 1.0)) <= (1e-6 if cfg["precision"] == 1 else 2.0 ** -22)
    assert gwgen.lib().gw_run_psd(gen._h, gwgen._ptr(bg), bg.shape[1], chunks, gwgen._ptr(psd), gwgen._ptr(ws), least - 8,
                                  gwgen._stream()) == gwgen.GW_EINVAL
