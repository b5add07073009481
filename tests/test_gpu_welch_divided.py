"""Batches whose Welch stage does divide stretches (each case asserts it: its
workspace then holds the divided stretches' sums beside what a binary32 batch,
which never divides, needs): shares of more than one stretch and of more than
two, even and odd segment counts, both segment lengths, binary64, one
detector.  The sums are exact, so the PSDs equal those of the six-step call,
which divides nothing, bit for bit, and so does a call whose workspace has no
room for the sums."""

import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over,B", [
    ("pr1_plain", dict(psd_length=34.0), 800),                      # 1600 stretches of 17 pairs on 1536 places
    ("pr1_plain", dict(psd_length=33.0), 1550),                     # 3100 of 16: whole stretches inside a share
    ("pr1_short", dict(psd_length=34.0, det_ids=(1,)), 1600),       # one detector
    ("pr1_plain", dict(psd_length=34.0, precision=2), 530),
    ("paper_scale", dict(psd_length=33.0), 260),                    # 780 stretches of 16 pairs on 768 places
    ("paper_scale", dict(psd_length=34.0, t_window=2.0), 520),      # 1560 of 17: whole stretches inside a share
    ("paper_scale", dict(psd_length=33.0, precision=2, t_window=4.0), 175),
    ("sine_gaussian", dict(psd_length=24.0, det_ids=(2, 0)), 3)])   # pieces of one pair
def test_divided_stretches(name, over, B):
    import torch
    cfg = inputs.config(name, **over)
    gen = gwgen.Generator(cfg)
    least = gwgen.Generator(dict(cfg, precision=0)).workspace_size(B)
    assert gen.workspace_size(B) > least
    z = gen.sizes
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 20, cfg["fs"], seed=7)).cuda()
    whole = torch.empty((B, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    at = -(-96 * B // 256) * 256 + -(-8 * B // 256) * 256
    outs = []
    for nbytes in (gen.workspace_size(B), least):
        ws = torch.empty(nbytes // 8, dtype=torch.float64, device="cuda")
        out = torch.full((B, z["D"], z["N"]), float("nan"), dtype=torch.float32, device="cuda")
        gen.generate_batch(4, 3, B, bg, out, ws)
        _, offs = gen.workspace_views(ws, B)
        gen.welch_psd(bg, offs.clone(), whole)
        torch.cuda.synchronize()
        psd = ws.view(torch.uint8)[at:at + whole.numel() * 4].view(torch.float32).view(whole.shape)
        assert torch.equal(psd, whole)
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
