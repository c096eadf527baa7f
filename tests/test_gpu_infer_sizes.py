"""Packing and the dequantize-and-multiply product where their kernels change:
few tokens (feature chunks of 128 dealt to eight waves), the two tile sizes,
rows of X at any alignment, and rows read up to the last element of X."""

import numpy as np
import pytest
import torch

import paper_2602_08376_amd as ok
from oracle import infer as oi
from oracle import ojbkq as orc

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ok.library()


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("n,m", [(5, 31), (3, 32), (7, 33), (2, 4096), (1100, 257), (1, 65536),
                                 (2, 65537)])
@pytest.mark.parametrize("permuted", [False, True])
def test_pack_codes(bits, n, m, permuted):
    rng = np.random.default_rng(bits + m)
    codes = rng.integers(0, 256, size=(n, m), dtype=np.uint8)   # only the low bits count
    perm = rng.permutation(m).astype(np.int32)
    t = torch.from_numpy(np.concatenate([np.zeros(1, np.uint8), codes.ravel()])).to(DEV)
    t = t[1:].view(n, m)                                        # rows at odd addresses
    got = ok.pack_codes(t, bits, perm=torch.from_numpy(perm).to(DEV) if permuted else None)
    low = codes & ((1 << bits) - 1)
    assert np.array_equal(got.cpu().numpy().view(np.uint32),
                          oi.pack_codes(low[:, perm] if permuted else low, bits))


@pytest.mark.parametrize("n,m,T,bits,group,ld,permuted", [
    (16, 128, 1, 4, 128, 0, False),      # one chunk, seven idle waves
    (33, 1025, 1, 4, 128, 3, True),      # one token of a wider X, a chunk of one feature
    (40, 300, 7, 3, 16, 0, False),       # scale groups of 16: two in a lane's run
    (40, 300, 8, 3, 48, 1, True),        # from eight tokens on: 16-byte loads
    (17, 1152, 16, 8, 64, 0, False),     # nine chunks: the first wave has two
    (65, 260, 17, 2, 0, 5, False),
    (100, 2000, 33, 5, 32, 0, True),
    (8192, 256, 20, 4, 128, 0, False),   # 32 channels per workgroup
    (16384, 160, 9, 6, 32, 0, False),    # 64
    (2100, 130, 1000, 4, 64, 0, False),  # 512 workgroups and a few: the small tiles
    (2100, 130, 1003, 7, 64, 0, True),   # rows of odd length, the last one cut
    (2100, 192, 1000, 1, 64, 8, False),
    (4300, 200, 4100, 4, 64, 0, False),  # the large tiles, ragged in every direction
    (4300, 200, 4101, 3, 64, 2, True),
    (32769, 72, 1, 4, 0, 0, False),      # an output head: the last rows of X hold fewer than
    (32769, 130, 2, 3, 64, 0, True),     # eight elements from their first on
    (33000, 65, 3, 4, 16, 0, False),
    (32769, 72, 7, 5, 0, 1, False),
    (32769, 72, 9, 2, 0, 0, False),
    (32769, 130, 65, 4, 64, 0, True),
    (32769, 511, 32, 4, 0, 0, False),    # either side of the few-token product's limits
    (32769, 512, 32, 3, 64, 0, True),
    (32769, 512, 33, 4, 64, 0, False),
    (33000, 520, 1, 8, 16, 0, False),
])
def test_product_at_the_edges_of_its_kernels(n, m, T, bits, group, ld, permuted):
    rng = np.random.default_rng(n + m + T)
    W = (rng.standard_normal((n, m)) * 0.02).astype(np.float32)
    S, Z = orc.scales_zeros(W[:64], bits, group)
    S, Z = (np.tile(A, (n // 64 + 1, 1))[:n].copy() for A in (S, Z))
    codes = rng.integers(0, 1 << bits, size=(n, m), dtype=np.uint8)
    perm = rng.permutation(m).astype(np.int32) if permuted else None
    # X ends exactly at its last element; the row padding is NaN and stays out
    buf = torch.full(((m - 1) * (T + ld) + T,), float("nan"), dtype=torch.float16, device=DEV)
    X = torch.as_strided(buf, (m, T), (T + ld, 1))
    x16 = rng.standard_normal((m, T)).astype(np.float16)
    X.copy_(torch.from_numpy(x16).to(DEV))
    dperm = None if perm is None else torch.from_numpy(perm).to(DEV)
    P = ok.pack_codes(torch.from_numpy(codes).to(DEV), bits, perm=dperm)
    # with a permutation the scales are those of the permuted groups
    args = (P, torch.from_numpy(S).to(DEV), torch.from_numpy(Z).to(DEV), m, bits, group, X)
    Y = ok.dequant_matmul(*args, perm=dperm, workspace=True)
    # (where both make one pass over the codes, the same kernel twice)
    assert torch.equal(Y, ok.dequant_matmul(*args, perm=dperm, workspace=False))
    W16 = oi.dequantize_fp16(codes if perm is None else codes[:, perm], S, Z, group)
    xp = x16 if perm is None else x16[perm]
    rows = np.unique(np.concatenate([np.arange(min(n, 40)), np.arange(max(0, n - 40), n)]))
    cols = np.unique(np.concatenate([np.arange(min(T, 40)), np.arange(max(0, T - 40), T)]))
    ref = oi.dequant_matmul(W16[rows], xp[:, cols])
    bound = oi.summation_bound(W16[rows], xp[:, cols])
    got = Y.cpu().numpy().astype(np.float64)[np.ix_(rows, cols)]
    assert np.all(np.abs(got - ref) <= bound + 1e-30)
    # every other element against float64 on the GPU
    full = torch.from_numpy(W16).to(DEV).double() @ torch.from_numpy(xp).to(DEV).double()
    assert float((Y.double() - full).norm() / full.norm()) < 1e-6


@pytest.mark.parametrize("n,m,T,one_pass", [(32769, 512, 1, True), (32769, 512, 32, True),
                                            (32769, 512, 33, False), (32769, 504, 32, False),
                                            (4096, 512, 100, True), (256, 512, 4096, True),
                                            (256, 512, 4097, False), (600, 512, 2047, True),
                                            (600, 512, 2048, False)])
def test_few_tokens_leave_the_workspace(n, m, T, one_pass):
    g = torch.Generator(device=DEV).manual_seed(n + T)
    P = torch.randint(0, 2 ** 31 - 1, (n, ok.packed_words(m, 4)), generator=g, device=DEV,
                      dtype=torch.int32)
    S = torch.rand(n, 1, generator=g, device=DEV) + 0.5
    Z = torch.full((n, 1), 8.0, device=DEV)
    X = torch.randn(m, T, generator=g, device=DEV).half()
    ws = torch.full((int(ok.library().ojbkq_dequant_matmul_workspace_bytes(n, m)),), 0xAB,
                    dtype=torch.uint8, device=DEV)
    Y = ok.dequant_matmul(P, S, Z, m, 4, 0, X, workspace=ws)
    assert bool((ws == 0xAB).all()) == one_pass
    assert torch.equal(Y, ok.dequant_matmul(P, S, Z, m, 4, 0, X))
    # the other form: the same sums, in another order where only this one
    # forms W_hat (m fp16 products in float32 each)
    other = ok.dequant_matmul(P, S, Z, m, 4, 0, X, workspace=False)
    codes = (P.view(n, -1, 1) >> torch.arange(0, 32, 4, device=DEV)).bitwise_and(15).view(n, m)
    W = (S * (codes - Z)).half().abs().double()
    bound = 2 * m * 2.0 ** -24 * (W @ X.abs().double())
    assert bool(((Y - other).abs() <= bound).all())


def test_few_tokens_allocate_no_workspace():
    # by default the binding allocates the workspace, but not for a product
    # that always leaves it alone
    n, m = 32769, 512
    P = torch.zeros(n, ok.packed_words(m, 4), device=DEV, dtype=torch.int32)
    S, Z = torch.ones(n, 1, device=DEV), torch.zeros(n, 1, device=DEV)
    size = int(ok.library().ojbkq_dequant_matmul_workspace_bytes(n, m))
    for T, allocates in ((1, False), (32, False), (33, True)):
        X = torch.ones(m, T, device=DEV).half()
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        ok.dequant_matmul(P, S, Z, m, 4, 0, X)
        grown = torch.cuda.max_memory_allocated() - before
        assert (grown >= size) == allocates, (T, grown, size)
