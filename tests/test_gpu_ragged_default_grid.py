"""The default persistent Welch launch of uneven batches, three workgroups a
compute unit: the same bits as with one workgroup and as the launches per
segment length, for few signals and for more groups than places; and the
autotuner, which tries it, leaves a grid that gives these bits."""

import pytest

from paper_2407_19048_amd import gwgen, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", (5, 700))
def test_default_grid(B):
    import torch
    classes = inputs.ragged_classes()
    rg = gwgen.Ragged(classes, inputs.ragged_assignment(B))
    assert rg.get_tuning(gwgen.RTUNE_GRID_WELCH) == 3
    by_rate = {fs: torch.from_numpy(inputs.background(3, 1 << 20, fs, seed=2)).cuda() for fs in inputs.RAGGED_RATES}
    bgs = [by_rate[c["fs"]] for c in classes]
    out, ws = rg.alloc_out(), rg.alloc_workspace()

    def run():
        out.fill_(float("nan"))
        rg.generate(6, 1, bgs, out, ws)
        torch.cuda.synchronize()
        return out.clone(), rg.workspace_views(ws)[2].clone()

    got = []
    for mode, grid in ((0, 3), (0, 1), (1, 3)):
        rg.set_tuning(gwgen.RTUNE_WELCH_MODE, mode)
        rg.set_tuning(gwgen.RTUNE_GRID_WELCH, grid)
        rg.set_tuning(gwgen.RTUNE_ORD_WELCH, 0)
        got.append(run())
    for o, p in got[1:]:
        assert torch.equal(o, got[0][0]) and torch.equal(p, got[0][1])
    window = rg.get_tuning(gwgen.RTUNE_WINDOW_MODE), rg.get_tuning(gwgen.RTUNE_ORD_WINDOW)
    table = rg.autotune(bgs, out, ws, reps=2)
    assert set(table["welch"]) == {(o, g) for o in (0, 1) for g in (1, 2, 4)}
    assert rg.get_tuning(gwgen.RTUNE_GRID_WELCH) in (1, 2, 3, 4)
    print("tuned: mode %d, %d workgroups a compute unit" % (rg.get_tuning(gwgen.RTUNE_WELCH_MODE),
                                                            rg.get_tuning(gwgen.RTUNE_GRID_WELCH)), flush=True)
    # the radix orders round differently; mode and grid as tuned do not
    rg.set_tuning(gwgen.RTUNE_ORD_WELCH, 0)
    rg.set_tuning(gwgen.RTUNE_WINDOW_MODE, window[0])
    rg.set_tuning(gwgen.RTUNE_ORD_WINDOW, window[1])
    o, p = run()
    assert torch.equal(p, got[0][1]) and torch.equal(o, got[0][0])
