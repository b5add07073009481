"""Range of the binary32 transforms: whitening and injection are linear, and a
power of two changes no rounding as long as nothing overflows, so windows of
samples of size 2^93 and 2^97 give the bits of ordinary ones, scaled."""

import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over", [("pr1_short", {}), ("pr1_plain", {}), ("paper_scale", dict(t_window=4.0)), ("paper_scale", {}),
                                       ("paper_scale", dict(t_window=16.0)), ("paper_scale", dict(precision=0)),
                                       ("bns_long", dict(t_window=32.0)), ("bns_long", dict(t_window=64.0))])
@pytest.mark.parametrize("order", (0, 1))
def test_large_samples(name, over, order):
    import torch
    gen = gwgen.Generator(inputs.config(name, **over))
    gen.set_tuning(gwgen.TUNE_ORD_WINDOW, order)
    z = gen.sizes
    g = torch.Generator(device="cuda").manual_seed(3)
    strain = torch.randn((1, z["D"], z["N"]), generator=g, device="cuda")
    psd = torch.rand((1, z["D"], z["Fw"]), generator=g, device="cuda") + 0.5
    hdet = torch.view_as_complex(torch.randn((1, z["D"], z["F"], 2), generator=g, device="cuda"))
    bg = torch.randn((z["D"], z["P"] + z["N"]), generator=g, device="cuda")
    offset = torch.zeros(1, dtype=torch.int64, device="cuda")
    want, injected = torch.empty_like(strain), torch.empty_like(strain)
    gen.whiten(strain, psd, want)
    gen.inject(bg, offset, hdet, injected)
    for power in (93, 97):
        scale = 2.0 ** power
        got = torch.empty_like(strain)
        gen.whiten(strain * scale, psd, got)
        assert torch.equal(got, want * scale)
        gen.inject(bg * scale, offset, hdet * scale, got)
        assert torch.equal(got, injected * scale)
