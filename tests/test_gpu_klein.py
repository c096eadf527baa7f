"""The Klein draws alone, decision by decision against the oracle.

R is diagonal, so no draw depends on another: every code must equal the
oracle's inverse-CDF draw from float64 weights.  The float32 weights decide a
draw only where the uniform is further from every running sum than their error
bound, so none may differ; the boxes from one bit (two points) to eight, the
temperatures from a few units (several likely points) to ones where the
nearest point is certain, and centres inside, at the edge of and far outside
the box."""

import numpy as np
import pytest
import torch

import paper_2602_08376_amd as ok
from oracle import ojbkq as orc
from parity import np64

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ok.library()


@pytest.mark.parametrize("decode", ["int8", "fp64"])
@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("m,K,steep", [(70, 24, 1.05), (70, 24, 1.7), (33, 400, 1.05), (5, 3, 1.2)])
def test_draws_equal_the_oracle(bits, m, K, steep, decode):
    n, qmax = 12, (1 << bits) - 1
    g = torch.Generator().manual_seed(1000 * bits + m + K)
    # R_ii from 1 up: kappa_i = ln(rho) R_ii^2
    d = steep ** (8.0 * torch.rand(m, generator=g, dtype=torch.float64))
    R = torch.diag(d)
    qbar = -2.5 + (qmax + 5.0) * torch.rand(n, m, generator=g, dtype=torch.float64)
    near = torch.rand(n, m, generator=g) < 0.3    # centres next to a rounding boundary
    qbar[near] = torch.floor(qbar[near]) + 0.5 + 1e-3 * torch.randn(int(near.sum()), generator=g,
                                                                    dtype=torch.float64)
    S = torch.ones(n, 1, dtype=torch.float32)
    codes, res, win, pc, pr = ok.decode_stage(R.to(DEV), qbar.to(DEV), S.to(DEV), bits, 0, K, 77,
                                              want_paths=True, decode=decode)
    dec = orc.decode(R.numpy(), qbar.numpy(), S.numpy(), bits, 0, K, 77)
    assert np.array_equal(np64(pc), dec.path_codes)
    # some draw is not the nearest point, or the case shows nothing
    if steep < 1.1 and m > 5:
        assert (dec.path_codes[:, 1:] != dec.path_codes[:, :1]).any()
