"""GeLU and its derivative over every bf16 value from -13 to 13, against 64 bits: results are correctly rounded up to the
fp32 evaluation's own error, down to the far negative tail."""
import numpy as np
import pytest
import torch
from scipy.special import ndtr

from paper_2311_02382_amd import lss

pytestmark = pytest.mark.gpu


def _grid():
    u = torch.arange(-32768, 32768, dtype=torch.int32).to(torch.int16).view(torch.bfloat16)
    u = u[torch.isfinite(u) & (u.abs() <= 13)]
    return torch.nn.functional.pad(u, (0, -u.numel() % 128))


@pytest.mark.parametrize("slope", [False, True])
def test_every_bf16_value(slope):
    u = _grid()
    x = u.double().numpy()
    if slope:
        phi = np.exp(-0.5 * x * x) / np.sqrt(2 * np.pi)
        exact, terms = ndtr(x) + x * phi, ndtr(x) + np.abs(x) * phi         # the slope's two terms cancel near -0.75
        got = lss.lss_gelu_bwd(u.cuda(), torch.ones_like(u).cuda())
    else:
        exact = x * ndtr(x)
        terms = np.abs(exact)
        got = lss.lss_gelu_fwd(u.cuda())
    # half a unit of the last of 8 significant bits (2^-8 of the value at most), the polynomial and ten fp32 operations (2e-6 of the terms, of which the exponential's
    # argument of up to 122 is the most: 122 * 2^-24 * 0.7 = 5e-6), and bf16's smallest normal
    err = np.abs(got.double().cpu().numpy() - exact)
    assert (err <= 2.0 ** -8 * np.abs(exact) + 8e-6 * terms + 2.0 ** -126).all(), float((err / (terms + 1e-30)).max())


def test_infinities_and_nan_as_before():
    u = torch.zeros(128, dtype=torch.bfloat16)
    u[:3] = torch.tensor([float("inf"), float("-inf"), float("nan")])
    g = lss.lss_gelu_fwd(u.cuda()).float().cpu()
    assert g[0] == float("inf") and g[1].isnan() and g[2].isnan() and not g[3:].any()
    assert lss.lss_gelu_bwd(u.cuda(), torch.ones_like(u).cuda()).float().cpu()[:3].isnan().all()
