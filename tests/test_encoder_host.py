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
