"""Waveforms of few samples, whose bins are shared by several workgroups,
against the same samples in a call with one workgroup a sample: the arithmetic
of a bin does not depend on the share, so the results are the same bits."""

import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over", [("paper_scale", {}), ("paper_scale", dict(precision=2)),
                                       ("pr1_short", {}), ("pr1_plain", dict(precision=0))])
def test_few_samples_equal_many(name, over):
    import torch
    cfg = inputs.config(name, **over)
    gen = gwgen.Generator(cfg)
    F, many = gen.sizes["F"], 1100
    params = torch.empty((gwgen.N_PARAMS, many), dtype=torch.float64, device="cuda")
    offset = torch.empty(many, dtype=torch.int64, device="cuda")
    gen.sample_params(5, 0, many, 1 << 20, params, offset)
    want = [torch.empty((many, F), dtype=torch.complex64, device="cuda") for _ in range(2)]
    gen.gen_fd_waveform(params, *want)
    for B in (1, 2, 63, 257, 700):
        got = [torch.full((B, F), complex(7.0, 7.0), dtype=torch.complex64, device="cuda") for _ in range(2)]
        gen.gen_fd_waveform(params[:, :B].contiguous(), *got)
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(torch.view_as_real(g), torch.view_as_real(w[:B]))
