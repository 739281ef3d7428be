"""The tile sizes of the workspace product (M > 64: 256x256, 256x128, 128x128, 128x64 and 64x64)
and of the product without a workspace (256x128, 128x128, 64x128 and 64x64), picked by how many
fill the CUs, each with whole and ragged edges, in every element type.

Bar: the codes are drawn over all words and every sum stays below 2^24 (checked), so it is
exact in each type; the rounding of the scales leaves an output within 4e-7 of the oracle's.
"""

import numpy as np
import pytest

from nq_gpu import upload_coded
from oracle import layout, nestquant

pytestmark = pytest.mark.gpu

SHAPES = [
    # (M, N, K): the tile that the rule takes
    (65, 64, 72), (128, 130, 136), (777, 1024, 64),           # 64x64
    (300, 4096, 72), (384, 4000, 136),                        # 128x64
    (1000, 4096, 72), (1024, 4090, 64),                       # 128x128
    (2048, 4096, 72), (1900, 4010, 136),                      # 256x128
    (4096, 4096, 72), (4000, 4090, 64),                       # 256x256
]
# The same tiles with their ring of LDS buffers (two to four stages of 128 int8 or 64 or 32
# 16-bit values a row) used again: 9 to 11 stages in int8, 18 and more in the 16-bit types.
LONG = [
    (65, 64, 1160), (777, 1024, 1408),                        # 64x64
    (300, 4096, 1160), (384, 4000, 1280),                     # 128x64
    (1000, 4096, 1160), (1024, 4090, 1280),                   # 128x128
    (2048, 4096, 1160), (1900, 4010, 1280),                   # 256x128
    (4000, 4090, 1160),                                       # 256x256
]
TYPES = {   # q, k, mult, decoder
    "i8": (14, 4, None, "full"),
    "bf16": (16, 4, None, "m"),
    "f16": (14, 4, (6, 8, 10, 16), "full"),
}


DIRECT = [
    (16, 1000, 264), (33, 1024, 136),                         # 64x64
    (1, 64, 136), (100, 1000, 264),                           # 64x128 (100 rows in f16: 64x64)
    (300, 4096, 136), (500, 4090, 72),                        # 64x128
    (600, 4096, 136), (640, 4090, 72),                        # 128x128
    (1500, 4096, 136), (1536, 4090, 72),                      # 256x128
]
DIRECT_LONG = [(16, 1000, 1160), (300, 4096, 1160), (600, 4096, 1160), (1500, 4096, 1160)]


@pytest.mark.parametrize("et", list(TYPES))
@pytest.mark.parametrize("shape", SHAPES + LONG, ids=lambda s: "x".join(map(str, s)))
def test_tile_sizes(shape, et):
    import paper_2502_09720_amd as nq
    _check(nq.matmul, shape, et)


@pytest.mark.parametrize("et", list(TYPES))
@pytest.mark.parametrize("shape", DIRECT + DIRECT_LONG, ids=lambda s: "x".join(map(str, s)))
def test_direct_tile_sizes(shape, et):
    import paper_2502_09720_amd as nq
    _check(nq.matmul_direct, shape, et)


def _check(product, shape, et):
    import torch
    (M, N, K), (q, k, mult, decoder) = shape, TYPES[et]
    rng = np.random.default_rng(M + 7 * N + K)
    base = nestquant.default_base(q, k) if mult is None else 0.5 / q
    ops, dev = [], []
    for rows in (M, N):
        c = rng.integers(0, q, (rows, K // 8, 8))
        t = rng.integers(1, k + 1, (rows, K // 8))
        r = rng.uniform(0.5, 2.0, rows).astype(np.float32)
        ops.append((nestquant.integer_tiles(c, t, q, decoder, mult), r))
        dev.append(upload_coded(layout.pack_codes(c), layout.pack_beta(t), r, rows, K, q, k,
                                base, 1 if decoder == "m" else 0, mult=mult))
    (TA, ra), (TW, rw) = ops
    C = nestquant.product_from_tiles(TA, ra, base, TW, rw, base)
    peak = (np.abs(TA).astype(np.float64) @ np.abs(TW).T.astype(np.float64)).max()
    assert peak < 2 ** 24
    out = torch.full((M, N + 8), 7.0, device="cuda")
    got = product(*dev, out=out[:, :N])
    g = got.double().cpu().numpy()
    assert np.all(np.abs(g - C) <= 4e-7 * np.abs(C))
    assert bool((out[:, N:] == 7.0).all())
