"""The int8 token sums (Gram and cross term) against exact sums in float64, at
the edges of their tiles, steps and digits.

Every row is kept to 31 bits below 2^e with max|x| <= 2^e 127/128, so an
operand is off by at most 2^(e-32); the dropped digit products (a2 b4 and
a4 b2, those with p + q >= 7, and a3 b3 in the cross term) are at most
2^14 (2^-45 + 2^-46) + 2^14 (2 2^-54 + 2^-62) of 2^(e_i + e_j) each.  Together
less than 2^-29 of 2^(e_i + e_j) per token, whatever the signs."""

import pytest
import torch

import paper_2602_08376_amd as ok

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ok.library()


def sums(m, chunks):
    """G (lower triangle) and E as a staged context accumulates them: the two
    [m, m] float64 arrays behind the workspace's two leading scalars."""
    s = ok.LayerSolver(m, m, 4, 64, 0, 1)
    for X, Xq in chunks:
        s.accumulate(X, Xq)
    torch.cuda.synchronize()
    nb = 8 * m * m
    at = 512
    G = s.ws[at:at + nb].view(torch.float64).view(m, m).clone()
    at += (nb + 255) // 256 * 256
    E = s.ws[at:at + nb].view(torch.float64).view(m, m).clone()
    s.close()
    return G.tril(), E


def check(m, chunks):
    G, E = sums(m, chunks)
    refG = torch.zeros(m, m, dtype=torch.float64, device=DEV)
    refE = torch.zeros_like(refG)
    boundG = torch.zeros_like(refG)
    boundE = torch.zeros_like(refG)

    def top(A):   # 2^e of each row
        mx = A.abs().amax(1) * (128.0 / 127.0)
        return torch.where(mx > 0, torch.exp2(torch.ceil(torch.log2(mx))), torch.zeros_like(mx))

    for X, Xq in chunks:
        Q, D = Xq.double(), X.double() - Xq.double()
        refG += Q @ Q.T
        refE += Q @ D.T
        T = X.shape[1]
        boundG += T * 2.0 ** -29 * top(Q)[:, None] * top(Q)[None, :]
        boundE += T * 2.0 ** -29 * top(Q)[:, None] * top(D)[None, :]
    # fp64 rounding of the sums themselves, here and in the reference
    eps = 1e-13
    assert bool(((G - refG.tril()).abs() <= boundG + eps * boundG.amax() * 2 ** 29).all())
    assert bool(((E - refE).abs() <= boundE + eps * boundE.amax() * 2 ** 29).all())


@pytest.mark.parametrize("m", [1, 127, 129, 300])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 193, 1024, 1025, 3100])
def test_int8_sums_at_the_edges_of_steps_and_tiles(m, T):
    g = torch.Generator(device=DEV).manual_seed(100 * m + T)
    X = torch.randn(m, T, generator=g, device=DEV) * torch.exp(
        torch.randn(m, 1, generator=g, device=DEV))
    Xq = X + 0.02 * torch.randn(m, T, generator=g, device=DEV)
    check(m, [(X, Xq)])


@pytest.mark.parametrize("top", [1.0, 127.0 / 128.0, 127.5 / 128.0, 0.5, 1.0 - 2.0 ** -24])
def test_int8_sums_at_the_ends_of_the_top_digit(top):
    # row maxima at and around the largest value of an exponent, both signs,
    # and rows of zeros
    m, T = 130, 200
    g = torch.Generator(device=DEV).manual_seed(3)
    Xq = torch.rand(m, T, generator=g, device=DEV) * 2 * top - top
    Xq[:, 5], Xq[:, 77] = top, -top
    Xq[7] = 0.0
    X = Xq + torch.where(torch.rand(m, T, generator=g, device=DEV) < 0.5, top, -top)
    X[9] = Xq[9]
    check(m, [(X, Xq), (X[:, :70].contiguous(), Xq[:, :70].contiguous())])


def test_int8_sums_do_not_overflow():
    # digits -126, -128, -128, -128 of every value over the longest sub-chunk
    # (32704 tokens, from m = 4088 on): the largest int32 sum is 0.99 of 2^31
    m, T = 4096, 32704
    Xq = torch.full((m, T), -0x7E808080 / 2.0 ** 31, dtype=torch.float32, device=DEV)
    Xq[1::2] *= 0.5
    X = 2.0 * Xq
    G, E = sums(m, [(X, Xq)])
    x = Xq[:, 0].double()
    want = T * x[:, None] * x[None, :]
    assert bool(((G - want.tril()).abs() <= 2.0 ** -29 * T).all())
    assert bool(((E - want).abs() <= 2.0 ** -29 * T).all())
