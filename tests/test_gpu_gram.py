"""The int8 token sums (Gram and cross term) against exact sums in float64, at
the edges of their tiles, steps and digits.

Every row is kept to 31 bits below 2^e with max|x| <= 2^e 127/128, so an
operand is off by at most 2^(e-32), a product of two by 2^-31 (1 + 2^-33) of
2^(e_i + e_j); the dropped digit products (p + q >= 7) are at most
2^14 (2 2^-54 + 2^-62) < 2^-38.9 of it.  Together less than 2^-30.9 of
2^(e_i + e_j) per token, whatever the signs."""

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
    at = 2 * 256   # (each padded to 256 bytes; any other place fails the checks)
    G = s.ws[at:at + nb].view(torch.float64).view(m, m).clone()
    at += (nb + 255) // 256 * 256
    E = s.ws[at:at + nb].view(torch.float64).view(m, m).clone()
    s.close()
    return G.tril(), E


def top(A):
    """2^e of each row: the smallest power of two with max|x| <= 2^e 127/128."""
    mx = A.abs().amax(1)
    f = torch.frexp(mx).mantissa
    t = mx / f.clamp(min=0.5)   # (exact)
    return torch.where(f > 127.0 / 128.0, 2 * t, t)


def check(m, chunks):
    G, E = sums(m, chunks)
    refG = torch.zeros(m, m, dtype=torch.float64, device=DEV)
    refE = torch.zeros_like(refG)
    boundG = torch.zeros_like(refG)
    boundE = torch.zeros_like(refG)

    for X, Xq in chunks:
        Q, D = Xq.double(), X.double() - Xq.double()
        refG += Q @ Q.T
        refE += Q @ D.T
        T = X.shape[1]
        boundG += T * 2.0 ** -30.9 * top(Q)[:, None] * top(Q)[None, :]
        boundE += T * 2.0 ** -30.9 * top(Q)[:, None] * top(D)[None, :]
    # fp64 rounding of the sums themselves, here and in the reference
    eps = 1e-13
    assert bool(((G - refG.tril()).abs() <= boundG + eps * boundG.amax() * 2 ** 30.9).all())
    assert bool(((E - refE).abs() <= boundE + eps * boundE.amax() * 2 ** 30.9).all())


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
    # (32768 tokens, from m = 4096 on): the largest int32 sum is 0.99 of 2^31
    m, T = 4096, 32768
    Xq = torch.full((m, T), -0x7E808080 / 2.0 ** 31, dtype=torch.float32, device=DEV)
    Xq[1::2] *= 0.5
    X = 2.0 * Xq
    G, E = sums(m, [(X, Xq)])
    x = Xq[:, 0].double()
    want = T * x[:, None] * x[None, :]
    # (every value is held exactly: only the dropped products and fp64 rounding)
    assert bool(((G - want.tril()).abs() <= 2.0 ** -38.8 * T).all())
    assert bool(((E - want).abs() <= 2.0 ** -38.8 * T).all())


def _rows(kind, m, T, g):
    """(X, X~) whose rows and differences are whole multiples of 2^(e-31)."""
    def rand(*size):   # 16-bit fractions in [1/2, 0.99]
        return 0.5 + torch.randint(0, 32112, size, generator=g, device=DEV).float() / 65536

    def fine(*size):   # all 24 bits, in [1/2, 0.99]
        return 0.5 + torch.randint(0, 8220000, size, generator=g, device=DEV).float() / 2.0 ** 24

    sign = torch.randint(0, 2, (m, T), generator=g, device=DEV).float() * 2 - 1
    if kind == "constant":
        Xq = fine(m, 1).expand(m, T).contiguous()
        return Xq * 0.5, Xq
    if kind == "equal":         # every row the same, and twice or half of it
        r = sign[:1] * fine(1, T)
        return -r * (1 << torch.arange(m, device=DEV)[:, None] % 3).float(), \
            r.expand(m, T).contiguous()
    if kind == "proportional":  # D = X~ / 2
        Xq = sign * rand(m, T)
        return 1.5 * Xq, Xq
    if kind == "mean":          # a large mean, a small spread
        Xq = 0.75 + (rand(m, T) - 0.75) / 512
        return Xq + (rand(m, T) - 0.75) / 512, Xq
    if kind == "half":          # a model run in fp16
        Xq = torch.randn(m, T, generator=g, device=DEV).clamp(-4, 4).half()
        X = (Xq.float() + 0.02 * torch.randn(m, T, generator=g, device=DEV)).half()
        return X.float(), Xq.float()
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["constant", "equal", "proportional", "mean", "half"])
def test_int8_sums_of_operands_held_exactly(kind):
    # Nothing is lost in the split, so only the dropped products, p + q >= 7,
    # are missing: 2^14 (2 2^-54 + 2^-62) of 2^(e_i + e_j) per token, the same
    # sign at every token or not.  Leaving out any product with p + q <= 6
    # (2^-32, most of it at every token of these rows) shows.
    m, T = 130, 2000
    g = torch.Generator(device=DEV).manual_seed(17)
    X, Xq = _rows(kind, m, T, g)
    Q, D = Xq.double(), X.double() - Xq.double()
    for A in (Q, D):
        v = A / top(A).clamp(min=2.0 ** -100)[:, None] * 2.0 ** 31
        assert bool((v == v.round()).all())
    G, E = sums(m, [(X, Xq)])
    for got, B, low in ((G, Q, True), (E, D, False)):
        want = Q @ B.T
        # (fp64 sums of T exact products: here and, in fewer parts, there)
        bound = (T * 2.0 ** -38.9 * top(Q)[:, None] * top(B)[None, :]
                 + T * 2.0 ** -52 * (Q.abs() @ B.abs().T))
        off = (got - want).abs()
        if low:
            off = off.tril()
        assert bool((off <= bound).all()), float((off / bound).max())
