"""The encoder's byte form of the nearest point, the root bound and the code (nq_e8b.hpp),
built for the host with its AMDGCN instructions written out in C++
(tests/host/nq_e8b_host.cpp), against the oracle.  CPU only.

nearest_e8_bytes may decline a vector (its two candidates too close for fp32, an exact half);
whatever it does return has to be Alg. 5's point, ties included.
"""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from conftest import ROOT
from oracle import lattice, voronoi

CSRC = os.path.join(ROOT, "paper_2502_09720_amd", "csrc")
MAX = 29.0      # kE8BytesMax


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    clang = "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        clang = shutil.which("clang++")
    if clang is None:
        pytest.skip("needs clang++ (ext_vector_type and __builtin_elementwise_max)")
    so = str(tmp_path_factory.mktemp("e8b") / "nq_e8b_host.so")
    cmd = [clang, "-std=c++17", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-Wall", "-I",
           CSRC, os.path.join(ROOT, "tests", "host", "nq_e8b_host.cpp"), "-o", so]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    so = ctypes.CDLL(so)
    so.nq_e8b_nearest.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_float,
                                  ctypes.c_void_p, ctypes.c_void_p]
    so.nq_e8b_code.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                               ctypes.c_void_p, ctypes.c_void_p]
    so.nq_e8b_first.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64,
                                ctypes.c_float, ctypes.c_void_p, ctypes.c_int, ctypes.c_int,
                                ctypes.c_int] + [ctypes.c_void_p] * 3
    return so


def _vectors(kind, n=60000):
    rng = np.random.default_rng(sum(map(ord, kind)))
    if kind == "normal":
        x = rng.standard_normal((n, 8)) * rng.choice([0.1, 1.0, 5.0], (n, 1))
    elif kind == "uniform":
        x = rng.uniform(-MAX, MAX, (n, 8))
    elif kind == "quarters":                 # exact halves, repeated distances, zeros of both signs
        x = rng.integers(-16, 17, (n, 8)) / 4.0
        x = np.where(rng.random((n, 8)) < 0.1, -0.0, x)
    elif kind == "sixteenths":
        x = rng.integers(-200, 201, (n, 8)) / 16.0
    elif kind == "tiny":                     # tiny entries of both signs beside lattice points
        x = rng.integers(-3, 4, (n, 8)) + rng.choice([0.0, 1e-30, -1e-30, 1e-9, -1e-9], (n, 8))
        x = np.where(rng.random((n, 8)) < 0.3, rng.choice([1e-40, -1e-40, -0.0], (n, 8)), x)
    else:                                    # around lattice points and their midpoints
        x = rng.integers(-8, 9, (n, 8)) / 2.0 + rng.standard_normal((n, 8)) * 1e-6
    return np.clip(x, -MAX, MAX).astype(np.float32)


@pytest.mark.parametrize("c", [1.0, 0.7432158])
@pytest.mark.parametrize("kind", ["normal", "uniform", "quarters", "sixteenths", "tiny", "near"])
def test_nearest_point(lib, kind, c):
    x = _vectors(kind)
    p = np.empty(x.shape, np.int32)
    ok = np.empty(len(x), np.uint8)
    lib.nq_e8b_nearest(x.ctypes.data, len(x), c, p.ctypes.data, ok.ctypes.data)
    y = x * np.float32(c)
    ok = ok.astype(bool)
    want = lattice.nearest_e8(y[ok].astype(np.float64))
    bad = np.nonzero(np.any(p[ok] != want, axis=1))[0]
    assert bad.size == 0, (y[ok][bad[:2]].tolist(), p[ok][bad[:2]], want[bad[:2]])
    if kind in ("normal", "uniform"):
        assert ok.mean() > 0.999             # it declines next to nothing on ordinary input


def _points(q, wide, n=40000):
    """Points of 2E8: nearest points of vectors over the whole cell of q 2E8 and its rim."""
    rng = np.random.default_rng(q + 100 * wide)
    x = rng.standard_normal((n, 8))
    x *= rng.uniform(0, 1.3 * q, (n, 1)) / np.linalg.norm(x, axis=1, keepdims=True)
    grid = rng.integers(-q, q + 1, (n, 8)).astype(np.float64)
    one = np.zeros((16, 8))
    one[np.arange(16), np.arange(16) // 2] = np.where(np.arange(16) % 2, q, -q)
    return np.unique(lattice.nearest_e8(np.concatenate([x, grid / 2, one])), axis=0)


ROOTS = None


def _root_bound(P):
    global ROOTS
    if ROOTS is None:
        g = np.indices((3,) * 8).reshape(8, -1).T - 1
        ints = g[(g ** 2).sum(1) == 2]
        s = np.indices((2,) * 8).reshape(8, -1).T * 2 - 1
        ROOTS = np.concatenate([2 * ints, s[(s < 0).sum(1) % 2 == 0]])      # twice the roots
    return np.concatenate([(P[i:i + 4096] @ ROOTS.T).max(1) for i in range(0, len(P), 4096)]) // 2


def _root_bound_real(x):
    """max over the roots of <x, root> (the bound of the point's integers, of reals)."""
    _root_bound(np.zeros((1, 8), np.int64))
    return (x.astype(np.float64) @ ROOTS.T.astype(np.float64)).max(1) / 2


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("q", list(range(2, 17)))
def test_root_bound_and_code(lib, q, wide):
    P = np.ascontiguousarray(_points(q, wide), np.int32)
    P = P[np.abs(P).max(1) <= 60]
    bound, words = np.empty(len(P), np.int32), np.empty(len(P), np.uint32)
    lib.nq_e8b_code(P.ctypes.data, len(P), q, wide, bound.ctypes.data, words.ctypes.data)
    M = _root_bound(P)
    assert np.array_equal(bound, M)
    take = M < 2 * q
    if wide:                                 # NestQuantM's box
        take = (np.abs(P[:, 0]) <= 2 * q) & (np.abs(P[:, 1:]).max(1) <= q)
    assert take.any()
    want = voronoi.encode_point(P[take], q)
    got = (words[take][:, None] >> (4 * np.arange(8, dtype=np.uint32))) & 15
    bad = np.nonzero(np.any(got != want, axis=1))[0]
    assert bad.size == 0, (q, P[take][bad[:2]], got[bad[:2]], want[bad[:2]])


# The row's limits: which beta a block starts at and whether the byte form may take it there.
# Scales at which r beta_1 and r beta_k lie on the two sides of 1e-30, where the thresholds
# change their arithmetic, or near fp32's underflow, among ordinary ones.
SCALES = [1.0, 1e30, 2e37, 5.6e-30, 5e-30, 3e-30, 1e-29, 2e-32, 1e-37, 2e-38]
SETS = [   # q, k, multiples of 0.5 / q (None: the uniform grid)
    (14, 4, None), (16, 4, None), (7, 2, None), (14, 1, None), (2, 4, None),
    (14, 4, (4, 8, 16, 40)), (14, 4, (1, 4, 16, 64)), (16, 4, (1, 2, 3, 64)), (5, 2, (1, 64)),
]


@pytest.mark.parametrize("decoder", [0, 1])
@pytest.mark.parametrize("q,k,mult", SETS, ids=lambda v: str(v).replace(" ", ""))
def test_first_beta_of_any_scale(lib, q, k, mult, decoder):
    """Blocks of up to 100 times the row scale: the beta that a block starts at is one that no
    smaller beta's point would have been kept for, and a point the byte form settles is Alg. 5's."""
    rng = np.random.default_rng(1000 * q + k)
    n = 4000
    z = rng.standard_normal((n, 8)) * rng.choice([0.05, 1.0], (n, 1))
    z[np.arange(n), rng.integers(0, 8, n)] = np.where(
        rng.random(n) < 0.5, -1, 1) * 10.0 ** rng.uniform(-1, 2, n)
    beta = np.array([m * 0.5 / q for m in mult] if mult else
                    [t * 10.0 / (k * q) for t in range(1, k + 1)])
    for scale in SCALES:
        r = np.float32(scale)
        if 1.0 / (float(r) * beta[0]) > 3e38:
            continue                         # no finite multiplier at the smallest beta
        x = np.clip(z * float(r), -3e38, 3e38).astype(np.float32)
        a = np.abs(x.astype(np.float64))
        mx = _root_bound_real(x) if decoder == 0 else \
            np.maximum(2 * a[:, 1:].max(1), a[:, 0])
        mx = np.minimum(mx, 3.4e38).astype(np.float32)
        t0, ok = np.empty(n, np.int32), np.empty(n, np.uint8)
        p = np.empty((n, 8), np.int32)
        lib.nq_e8b_first(x.ctypes.data, mx.ctypes.data, n, r, beta.ctypes.data, k, q, decoder,
                         t0.ctypes.data, p.ctypes.data, ok.ctypes.data)
        ok = ok.astype(bool)
        assert t0.max() < k
        kept = []
        for b in beta:
            y = (x * np.float32(1.0 / (float(r) * b))).astype(np.float64)
            P = lattice.nearest_e8(y)
            kept.append((P, ~voronoi.overloaded(P, q, "m" if decoder else "full")))
        for t in range(k):
            take = ok & (t0 == t)
            bad = np.nonzero(np.any(p[take] != kept[t][0][take], axis=1))[0]
            assert bad.size == 0, (scale, t, x[take][bad[:2]] / r, p[take][bad[:2]])
            assert not np.any(kept[t][1] & (t0 > t)), (scale, t)
        if scale == 1.0:
            assert ok.mean() > 0.5
