"""The decoder's input Rbar qbar against float64 products on the host, at sizes
around the edges of the fp64 product's tiles (128, 64 and 32 wide; which one
runs goes by the product's size), on every route to it: through L^-1 (2n > m),
by the triangular solve, and with the cross term projected (10n <= m)."""

import numpy as np
import pytest
import torch

import paper_2602_08376_amd as ok
from oracle import ojbkq as orc

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ok.library()


@pytest.mark.parametrize("m,n", [
    (1, 1), (5, 40), (32, 32), (33, 31), (64, 65), (100, 129), (257, 300), (130, 1030),   # L^-1
    (65, 20), (129, 33), (300, 100), (515, 200), (1100, 257), (2050, 600),                # solve
    (90, 9), (400, 33), (1300, 70),                                                       # projected
])
@pytest.mark.parametrize("mu", [1.0, 0.4])
def test_decoder_input(m, n, mu):
    T, group = 2 * m + 64, 48
    g = torch.Generator().manual_seed(m + n)
    W = torch.randn(n, m, generator=g) * 0.02
    X = torch.randn(m, T, generator=g)
    Xq = X + 0.05 * torch.randn(m, T, generator=g)
    s = ok.LayerSolver(m, n, 4, group, 0, 1)
    Wd = W.to(DEV)
    s.set_weights(Wd)
    s.accumulate(X.to(DEV), Xq.to(DEV))
    q = s.solve(Wd, mu)
    L = s.inspect("L").cpu().numpy()
    gq = s.inspect("gq").cpu().numpy()
    s.close()
    S = orc.expand_groups(q.scales.cpu().numpy(), m, group)
    Z = orc.expand_groups(q.zeros.cpu().numpy(), m, group)
    Wn = W.numpy().astype(np.float64)
    base = Wn + S * Z
    want = base @ L
    # m products summed in fp64 in two parts, each rounding below 2^-53 of them
    bound = 4 * (m + 4) * 2.0 ** -53 * (np.abs(base) + np.abs(S * Z)) @ np.abs(L)
    if mu != 1.0:
        Q = Xq.numpy().astype(np.float64)
        E = Q @ (X.numpy().astype(np.float64) - Q).T
        U = (1 - mu) * np.linalg.solve(L, E @ Wn.T).T
        want = want + U
        # the sums' own error (below 2^-30 of the row maxima's products a
        # token, of random sign) through a well-conditioned factor
        bound = bound + 1e-8 * np.abs(U).max()
    assert np.all(np.abs(gq - want) <= bound + 1e-300)


def test_products_in_place_give_the_same_every_time():
    # the triangular solve's leaves overwrite their own left operand: with
    # tiles narrower than a leaf, workgroups would read each other's results
    m, n = 6400, 128
    g = torch.Generator(device=DEV).manual_seed(9)
    X = torch.randn(m, 4096, generator=g, device=DEV)
    Xq = X + 0.05 * torch.randn(m, 4096, generator=g, device=DEV)
    W = torch.randn(n, m, generator=g, device=DEV) * 0.02
    s = ok.LayerSolver(m, n, 4, 64, 0, 1)
    s.accumulate(X, Xq)
    s.solve(W, 0.5)
    first = s.inspect("gq")
    for _ in range(40):
        s.solve(W, 0.5)
        assert torch.equal(s.inspect("gq"), first)
    s.close()
