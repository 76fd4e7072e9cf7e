"""LayerNorm's backward of short segments, one launch for dx, dgamma and dbeta: rows on either side of its 16 per row workgroup and 256 x 4 per
column thread, columns that do not fill a column workgroup, either side of the sizes at which it is taken, and gradients written over what is read.
Which kernels ran is read from the launch counters."""
import pytest
import torch

from paper_2311_02382_amd import lss, timing

pytestmark = pytest.mark.gpu


def _case(rows, E):
    gen = torch.Generator(device="cuda").manual_seed(rows * 7 + E)
    x, dy = ((torch.randn(rows, E, generator=gen, device="cuda") * 1.5 + 0.3).to(torch.bfloat16) for _ in range(2))
    gamma, beta = 1.0 + 0.2 * torch.randn(E, generator=gen, device="cuda"), torch.randn(E, generator=gen, device="cuda")
    _, mean, rstd = lss.lss_layernorm_fwd(x, gamma, beta)
    return x, dy, gamma, mean, rstd


def _launches(call):
    """What call() returns, and how often the kernel of one launch ran, and the first of two."""
    ids = {name: k for k, name in timing.kernel_names().items()}
    timing.reset()
    timing.enable(True)
    try:
        result = call()
        torch.cuda.synchronize()
    finally:
        timing.enable(False)
    return result, [timing.read(ids[name])[1] for name in ("layernorm_bwd_short_kernel", "layernorm_bwd_kernel")]


@pytest.mark.parametrize("rows,E,one", [(1, 8, True), (15, 40, True), (17, 512, True), (255, 128, True), (256, 1032, True), (257, 2048, True),
                                        (511, 2048, True), (719, 520, True), (720, 1024, True), (720, 8, True), (1008, 1040, True), (721, 8, False),
                                        (1023, 520, False), (1024, 1024, False), (1025, 8, False), (513, 2048, False), (40, 2056, False)])
def test_gradients_against_64_bits(rows, E, one):
    x, dy, gamma, mean, rstd = _case(rows, E)
    (dx, dg, db), launches = _launches(lambda: lss.lss_layernorm_bwd(x, gamma, mean, rstd, dy))
    assert launches == ([1, 0] if one else [0, 1])
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


@pytest.mark.parametrize("over,launch", [("dx on x", 0), ("dx on dy", 0), ("dgamma on gamma", 1), ("dbeta on gamma", 1)])
def test_gradients_written_over_inputs(over, launch):
    # (dx in an input's place: the one launch's two kinds of workgroup one after the other; a sum in the place of what is read: the two
    # launches, which add up in another order)
    x, dy, gamma, mean, rstd = _case(300, 512)
    want = lss.lss_layernorm_bwd(x.clone(), gamma.clone(), mean, rstd, dy.clone())
    to = {over.split()[0]: {"x": x, "dy": dy, "gamma": gamma}[over.split()[2]]}
    got, launches = _launches(lambda: lss.lss_layernorm_bwd(x, gamma, mean, rstd, dy, **to))
    assert launches[launch] == 1 and launches[1 - launch] == 0
    assert torch.equal(got[0], want[0])
    for a, b in zip(got[1:], want[1:]):
        if launch == 0:
            assert torch.equal(a, b)
        assert (a - b).norm() <= 1e-5 * b.norm()
