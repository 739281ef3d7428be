"""The choice of int8 tiles for a product whose caller did not ask for them.

Every m X2 of both operands has to fit int8: 2q m_k <= 127, or 128 with the full decoder,
whose tie rules decode the one code word of the points +-2q e_i to -2q e_0.  The cases sit on
both sides of that line, with codes drawn over all words so that the extreme one occurs (it is
planted as well), on the paths of M <= 2, M <= 64 and above.

Bar: integer sums below 2^24 are exact in every element type, and the rounding of the sum, of
r_A (r_W s) and of their product leaves each output within 4e-7 of the oracle's value.
"""

import numpy as np
import pytest

from nq_gpu import upload_coded
from oracle import layout, nestquant


def extreme_word(q):
    """The codes of 2q e_0 (G^-1 P mod q; even q only)."""
    return np.array([2 * q, 10 * q // 4] + [-q] * 6) % q


@pytest.mark.parametrize("q", [2, 4, 6, 8, 10, 12, 14, 16])
def test_extreme_word_decodes_to_minus_2q(q):
    c = np.tile(extreme_word(q), (1, 1, 1)).astype(np.int64)
    T = nestquant.integer_tiles(c, np.ones((1, 1), np.int64), q).reshape(-1)
    assert T.tolist() == [-2 * q] + [0] * 7


CASES = [
    # (M, N, K, q, k, mult, decoder)
    (65, 70, 264, 16, 4, None, "full"),            # 128: int8, full decoder
    (300, 257, 1000, 16, 4, None, "full"),
    (40, 33, 264, 16, 4, None, "full"),
    (2, 33, 264, 16, 4, None, "full"),
    (65, 70, 264, 16, 4, None, "m"),               # 128 with NestQuantM: 16-bit tiles
    (65, 70, 264, 8, 2, (3, 8), "full"),           # 128 through the multiples
    (65, 70, 264, 8, 2, (3, 9), "full"),           # 144: 16-bit tiles
    (65, 70, 136, 15, 4, None, "m"),               # 120
    (17, 70, 136, 14, 4, None, "m"),               # 112
    (130, 129, 72, 14, 4, None, "full"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_product_on_both_sides_of_the_int8_bound(case):
    import torch
    import paper_2502_09720_amd as nq
    M, N, K, q, k, mult, decoder = case
    rng = np.random.default_rng(M * N + K + q)
    base = nestquant.default_base(q, k) if mult is None else 0.5 / q
    ops, dev = [], []
    for rows in (M, N):
        c = rng.integers(0, q, (rows, K // 8, 8))
        t = rng.integers(1, k + 1, (rows, K // 8))
        if q % 2 == 0:
            c[:, 0], t[:, 0] = extreme_word(q), k
        r = rng.uniform(0.5, 2.0, rows).astype(np.float32)
        ops.append((nestquant.integer_tiles(c, t, q, decoder, mult), r))
        dev.append(upload_coded(layout.pack_codes(c), layout.pack_beta(t), r, rows, K, q, k,
                                base, 1 if decoder == "m" else 0, mult=mult))
    (TA, ra), (TW, rw) = ops
    C = nestquant.product_from_tiles(TA, ra, base, TW, rw, base)
    assert K * np.abs(TA).max() * np.abs(TW).max() < 2 ** 24
    for got in (nq.matmul(*dev), nq.matmul_direct(*dev)):
        g = got.double().cpu().numpy()
        assert np.all(np.abs(g - C) <= 4e-7 * np.abs(C))


@pytest.mark.gpu
def test_both_products_take_the_same_tiles():
    """q = 16 with NestQuantM and three betas: every m X2 in use fits int8 (a fourth beta's
    would not), with a workspace and without one.  Both then agree bit for bit and with the
    oracle on sums that fp32 does not hold: rows of long points against near copies of
    themselves, beyond 2^26 (inner products of 2E8 are multiples of 4)."""
    import torch
    import paper_2502_09720_amd as nq
    M, N, K, q, k = 65, 70, 65536, 16, 3
    rng = np.random.default_rng(k)
    base = nestquant.default_base(q, k)
    words = rng.integers(0, q, (1, 100000, 8))
    X = nestquant.integer_tiles(words, np.ones((1, 100000), np.int64), q, "m").reshape(-1, 8)
    longest = words[0][np.argsort(-(X.astype(np.int64) ** 2).sum(1))[:500]]
    ca = longest[rng.integers(0, 500, (M, K // 8))]
    cw = longest[rng.integers(0, 500, (N, K // 8))]
    cw[:M] = np.where(rng.random((M, K // 8, 1)) < 0.02, cw[:M], ca)
    ops, dev = [], []
    for c in (ca, cw):
        t = np.full(c.shape[:2], k)
        r = rng.uniform(0.5, 2.0, len(c)).astype(np.float32)
        ops.append((nestquant.integer_tiles(c, t, q, "m"), r))
        dev.append(upload_coded(layout.pack_codes(c), layout.pack_beta(t), r, len(c), K, q, k,
                                base, 1))
    (TA, ra), (TW, rw) = ops
    S = (TA.astype(np.int64) * TW[:M]).sum(1)
    assert S.min() > 2 ** 26 and np.any(S % 8 != 0)
    C = nestquant.product_from_tiles(TA, ra, base, TW, rw, base)
    ex, direct = nq.matmul(*dev), nq.matmul_direct(*dev)
    assert torch.equal(ex, direct)
    assert np.all(np.abs(ex.double().cpu().numpy() - C) <= 4e-7 * np.abs(C))


@pytest.mark.gpu
@pytest.mark.parametrize("decoder", ["full", "m"])
@pytest.mark.parametrize("M,K", [
    (1, 43680), (2, 21840),       # the last rows whose points the integer-dot kernel holds
    (1, 43696), (2, 21848),       # past them: int8 tiles decoded inside the product kernel
    (1, 49152), (2, 24576),       # the last that fit there
    (1, 49160), (2, 24584),       # past them: A's tile in the workspace
])
def test_long_rows_of_one_and_two(M, K, decoder):
    """One and two activation rows on both sides of the limits of what a workgroup holds of
    them.  Every sum is an exact int32 on each path."""
    import paper_2502_09720_amd as nq
    N, q, k = 33, 14, 4
    rng = np.random.default_rng(M + K)
    base = nestquant.default_base(q, k)
    ops, dev = [], []
    for rows in (M, N):
        c = rng.integers(0, q, (rows, K // 8, 8))
        t = rng.integers(1, k + 1, (rows, K // 8))
        r = rng.uniform(0.5, 2.0, rows).astype(np.float32)
        ops.append((nestquant.integer_tiles(c, t, q, decoder), r))
        dev.append(upload_coded(layout.pack_codes(c), layout.pack_beta(t), r, rows, K, q, k,
                                base, 1 if decoder == "m" else 0))
    (TA, ra), (TW, rw) = ops
    C = nestquant.product_from_tiles(TA, ra, base, TW, rw, base)
    g = nq.matmul(*dev).double().cpu().numpy()
    assert np.all(np.abs(g - C) <= 4e-7 * np.abs(C))
