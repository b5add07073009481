"""Binary64 Welch sums do not depend on how a batch's stretches are divided
over the workgroups: the PSDs of a batch that divides them equal those of the
six-step call, which never does, bit for bit over 2.4e9 bins (plain binary64
sums in two groupings differ by about 1e-16, so that of as many bins a few
round to the other binary32 value), and a batch equals the union of its parts."""

import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


def test_psd_bits_of_cut_and_whole_stretches():
    import torch
    gen = gwgen.Generator(inputs.config("paper_scale", precision=2, t_window=2.0))
    z, B = gen.sizes, 100
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 22, gen.cfg["fs"], seed=3)).cuda()
    out = torch.empty((B, z["D"], z["N"]), dtype=torch.float32, device="cuda")
    ws = gen.alloc_workspace(B)
    _, offs = gen.workspace_views(ws, B)
    whole = torch.empty((B, z["D"], z["Fw"]), dtype=torch.float32, device="cuda")
    at = -(-96 * B // 256) * 256 + -(-8 * B // 256) * 256
    psd = ws.view(torch.uint8)[at:at + whole.numel() * 4].view(torch.float32).view(whole.shape)
    differ = torch.zeros((), dtype=torch.int64, device="cuda")
    for n in range(4000):
        gen.generate_batch(12, n, B, bg, out, ws)
        gen.welch_psd(bg, offs.clone(), whole)
        differ += (psd != whole).sum()
    assert int(differ) == 0


@pytest.mark.parametrize("name,B,parts", [("paper_scale", 96, (1, 2, 8)), ("pr1_plain", 520, (4, 65))])
def test_batch_equals_its_parts(name, B, parts):
    import torch
    gen = gwgen.Generator(inputs.config(name, precision=2))
    z = gen.sizes
    bg = torch.from_numpy(inputs.background(z["D"], 1 << 20, gen.cfg["fs"], seed=3)).cuda()
    want = torch.empty((B, z["D"], z["N"]), dtype=torch.float32, device="cuda")
    gen.generate_batch(5, 0, B, bg, want, gen.alloc_workspace(B))
    for n in parts:
        b = B // n
        got = torch.empty_like(want)
        ws = gen.alloc_workspace(b)
        for i in range(n):
            gen.generate_batch(5, i, b, bg, got[i * b:(i + 1) * b], ws)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
