"""Rows of up to 32 blocks coded by one-wave workgroups of 4 and of 12 passes, which the encoder
takes from 32768 / 16384 / 8192 and from 1572864 / 786432 / 393216 rows on (8, 16 and 32 lanes a
row); fewer rows take workgroups of one pass.

Bar: codes, beta words and scales bit for bit the oracle's on a sample of the rows (the first
and last workgroups, the last one part full, and rows drawn from all of them), and bit for bit
those that the one-pass form gives on slices of the rows.
"""

import numpy as np
import pytest

import workloads
from nq_gpu import first_mismatch, oracle_encode, to_device, u32

pytestmark = pytest.mark.gpu

CASES = [
    # (rows, cols, dtype, dist, q, k, mult, decoder, entries between the rows)
    # 4 passes: 8, 16 and 32 lanes, whole and part rows
    (32773, 64, "bf16", "t4", 14, 4, None, "full", 0),
    (33000, 40, "f32", "normal", 16, 4, None, "m", 0),
    (16387, 128, "f16", "normal", 14, 4, None, "m", 0),
    (16400, 72, "bf16", "t4", 14, 4, (6, 8, 10, 16), "full", 8),
    (8193, 256, "f32", "t4", 7, 4, None, "full", 0),
    (8300, 200, "bf16", "normal", 16, 3, None, "m", 16),
    # 12 passes
    (1572869, 64, "f16", "t4", 14, 4, None, "full", 0),
    (1572900, 40, "bf16", "t4", 16, 4, None, "m", 0),
    (786439, 128, "bf16", "t4", 16, 4, None, "m", 0),
    (786500, 104, "f32", "t4", 14, 2, (3, 9), "full", 0),
    (393217, 256, "f32", "t4", 14, 4, None, "full", 0),
    (393300, 200, "f16", "normal", 7, 4, None, "m", 8),
]


@pytest.fixture(scope="module")
def nq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_09720_amd as nq
    nq.library()
    return nq


def _rows(rows, cols, dtype, dist, gap=0):
    """(device matrix, host values of a row): a block of 4096 rows drawn on the host, repeated
    with a factor of its own for each repetition, so that any row is known on the host."""
    import torch
    store, x32 = workloads.random_rows(rows + cols, 4096, cols, dtype=dtype, dist=dist)
    x32[7] = 0.0
    _, block = workloads.round_to(x32.astype(np.float64), dtype)
    factor = 2.0 ** (np.arange(-(-rows // 4096)) % 3)              # exact in every type
    big = torch.zeros(rows, cols + gap, dtype={"f32": torch.float32, "f16": torch.float16,
                                               "bf16": torch.bfloat16}[dtype], device="cuda")
    x = big[:, :cols]
    dev = torch.from_numpy(block).cuda()
    for i, f in enumerate(factor):
        part = x[4096 * i:4096 * (i + 1)]
        part.copy_(dev[:len(part)] * float(f))
    host = x[torch.from_numpy(np.arange(0, rows, max(1, rows // 500))).cuda()].float().cpu()
    idx = np.arange(0, rows, max(1, rows // 500))
    want = block[idx % 4096] * factor[idx // 4096].astype(np.float32)[:, None]
    assert np.array_equal(host.numpy(), want)
    return x, lambda i: block[i % 4096] * factor[i // 4096].astype(np.float32)[:, None]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v).replace(" ", "") for v in c))
def test_multi_pass_workgroups(nq, case):
    import torch
    rows, cols, dtype, dist, q, k, mult, decoder, gap = case
    x, host = _rows(rows, cols, dtype, dist, gap)
    opts = dict(q=q, k=k, base=None if mult is None else 0.5 / q, mult=mult,
                decoder=1 if decoder == "m" else 0)
    got = nq.encode(x, **opts)
    nb = cols // 8
    codes, beta = got.codes.view(rows, nb), got.beta.view(rows, -1)
    rng = np.random.default_rng(rows)
    idx = np.unique(np.concatenate([np.arange(200), np.arange(rows - 200, rows),
                                    rng.integers(0, rows, 1500)]))
    at = torch.from_numpy(idx).cuda()
    oc, ob, os_ = oracle_encode(host(idx), q, k, opts["base"], decoder, "first", mult)
    assert first_mismatch(u32(got.scales[at]), os_.view(np.uint32)) is None
    m = first_mismatch(u32(codes[at]), oc)
    assert m is None, m
    m = first_mismatch(u32(beta[at]), ob)
    assert m is None, m
    for i in (0, rows // 2, rows - 4000):                 # the one-pass form
        one = nq.encode(x[i:i + 4000], **opts)
        assert torch.equal(one.codes.view(4000, nb), codes[i:i + 4000])
        assert torch.equal(one.beta.view(4000, -1), beta[i:i + 4000])
        assert torch.equal(one.scales, got.scales[i:i + 4000])


@pytest.mark.parametrize("rows,cols,dtype,q,decoder", [
    (32773, 64, "f16", 14, 0), (16387, 120, "bf16", 16, 1), (8197, 256, "f32", 16, 0),
    (393223, 256, "bf16", 14, 0), (786437, 96, "f16", 16, 1),
])
def test_multi_pass_workgroups_write_tiles(nq, rows, cols, dtype, q, decoder):
    """The same forms inside encode_matmul: the codes, and the product of the tiles that the
    encoder writes beside them, are those of encode and matmul."""
    import torch
    x, _ = _rows(rows, cols, dtype, "t4")
    wstore, _ = workloads.random_rows(5, 40, cols, dtype="bf16", scale=0.02)
    w = nq.encode(to_device(wstore, "bf16"), q=q, k=4, decoder=decoder)
    a1 = nq.encode(x, q=q, k=4, decoder=decoder)
    a2, c2 = nq.encode_matmul(x, w, q=q, k=4, decoder=decoder)
    assert torch.equal(a1.codes, a2.codes) and torch.equal(a1.beta, a2.beta)
    assert torch.equal(a1.scales, a2.scales)
    assert torch.equal(nq.matmul(a1, w), c2)
