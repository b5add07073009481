"""The network's activation where its argument is infinite, very large or very
negative: the last hidden layer with such biases against silu in binary64,
rounded to bfloat16 (2^-9 relative, and one bfloat16 step more where binary32's
own rounding crosses a boundary: 2^-8; below 2e-36, the size of silu where
1 + exp(-z) nears the end of binary32's range, only the size counts), infinities
exactly; and gradients, which stay finite where every activation and
derivative is."""

import numpy as np
import pytest

from paper_2407_19048_amd import gwgen, inputs
from paper_2407_19048_amd import surrogate as GS

pytestmark = pytest.mark.gpu
BIAS2 = 16 * 256 + 256 + 2 * 256 * 256 + 256  # first bias of the last hidden layer in the flat layout
LARGE = (1e30, 1e36, 100.0, 88.0, 30.0, 1e-30)
SMALL = (-3e38, -1e36, -1e30, -1e4, -100.0, -88.6, -88.0, -87.5, -87.0, -80.0, -20.0, -1e-30)


def _made(values):
    import torch
    gen = gwgen.Generator(inputs.config("surrogate"))
    s = GS.Surrogate(gen, max_batch=64)
    w = np.zeros(s.n_weights, dtype=np.float32)  # the last hidden layer's arguments are its biases
    w[BIAS2:BIAS2 + len(values)] = values
    s.set_weights(w)
    return gen, s, torch.full((64, 4), 0.3, dtype=torch.float32, device="cuda")


def test_silu_of_extreme_arguments():
    import torch
    values = (np.inf,) + LARGE + SMALL
    gen, s, theta = _made(values)
    h = torch.full((64, 256), np.nan, dtype=torch.float32, device="cuda")
    s.hidden(theta, h)
    torch.cuda.synchronize()
    got = h.cpu().numpy()[:, :len(values)].astype(np.float64)
    z = np.asarray(values, dtype=np.float32).astype(np.float64)
    with np.errstate(over="ignore"):
        want = z / (1.0 + np.exp(-z))
    assert np.all(got[:, 0] == np.inf)
    for i in range(1, len(values)):
        assert np.all(np.abs(got[:, i] - want[i]) <= 2.0 ** -8 * abs(want[i]) + 2e-36), (values[i], got[0, i], want[i])


def test_gradients_of_extreme_arguments_are_finite():
    import torch
    gen, s, theta = _made((1e30, 100.0) + SMALL)
    grads = torch.full((s.n_weights,), np.nan, dtype=torch.float32, device="cuda")
    s.gradients(theta, torch.ones((64, 128), dtype=torch.float32, device="cuda"), grads)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(grads).all())
    # the output layer's weights are zero, so no gradient reaches the hidden layers
    assert not bool(grads[:BIAS2 + 256].any())
