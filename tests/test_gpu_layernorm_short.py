"""LayerNorm's backward of short segments, one launch for dx, dgamma and dbeta: rows on either side of its 16 per row workgroup and 256 x 4 per
column thread, columns that do not fill a column workgroup, either side of the sizes at which it is taken, and gradients written over what is read."""
import pytest
import torch

from paper_2311_02382_amd import lss

pytestmark = pytest.mark.gpu


def _case(rows, E):
    gen = torch.Generator(device="cuda").manual_seed(rows * 7 + E)
    x, dy = ((torch.randn(rows, E, generator=gen, device="cuda") * 1.5 + 0.3).to(torch.bfloat16) for _ in range(2))
    gamma, beta = 1.0 + 0.2 * torch.randn(E, generator=gen, device="cuda"), torch.randn(E, generator=gen, device="cuda")
    _, mean, rstd = lss.lss_layernorm_fwd(x, gamma, beta)
    return x, dy, gamma, mean, rstd


@pytest.mark.parametrize("rows,E", [(1, 8), (15, 40), (17, 512), (255, 128), (256, 1032), (257, 2048), (511, 2048), (1023, 520), (1024, 1024),
                                    (1024, 8), (1025, 8), (513, 2048), (40, 2056)])
def test_gradients_against_64_bits(rows, E):
    x, dy, gamma, mean, rstd = _case(rows, E)
    dx, dg, db = lss.lss_layernorm_bwd(x, gamma, mean, rstd, dy)
    xh, d = (x.double() - mean.double()[:, None]) * rstd.double()[:, None], dy.double()
    g = d * gamma.double()
    want = rstd.double()[:, None] * (g - g.mean(1, keepdim=True) - xh * (g * xh).mean(1, keepdim=True))
    # sums of `rows` products in 32 bits: half a unit per addition, and those of at most 4 + 2 + 8 + 4 partial sums in a row behind them
    bound = (rows / 256 + 20) * 2.0 ** -23
    for got, terms in ((dg, d * xh), (db, d)):
        assert ((got.double() - terms.sum(0)).abs() <= bound * terms.abs().sum(0) + 1e-30).all()
    assert (dx.double() - want).norm() <= 2.0 ** -8 * want.norm() + 1e-30       # rounded to bf16 once
    again = lss.lss_layernorm_bwd(x, gamma, mean, rstd, dy)
    assert all(torch.equal(a, b) for a, b in zip((dx, dg, db), again))


@pytest.mark.parametrize("over", ["dx on x", "dx on dy", "dgamma on gamma", "dbeta on gamma"])
def test_gradients_written_over_inputs(over):
    x, dy, gamma, mean, rstd = _case(300, 512)
    want = lss.lss_layernorm_bwd(x.clone(), gamma.clone(), mean, rstd, dy.clone())
    to = {over.split()[0]: {"x": x, "dy": dy, "gamma": gamma}[over.split()[2]]}
    got = lss.lss_layernorm_bwd(x, gamma, mean, rstd, dy, **to)
    assert torch.equal(got[0], want[0])
    for a, b in zip(got[1:], want[1:]):
        assert (a - b).norm() <= 1e-5 * b.norm()
