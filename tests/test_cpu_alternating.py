"""The alternating quantizer's kernels, run on the CPU from their source (tests/hip_on_cpu) with the waves of a workgroup in ascending and in
descending order between barriers: what one wave reads of another may not depend on which of them is ahead.  Same bar as on the GPU: bit
for bit as the oracle on every vector whose decisions it reports as robust."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def degenerate_rows(K):
    """All planes after the first, or after the second, have a zero residual, so that the first Gram matrix is singular and the scales of the
    greedy start are the result; the values are such that every sum is exact."""
    k = np.arange(K)
    return np.stack([np.zeros(K), np.full(K, 0.25), np.where(k % 3 == 0, -0.5, 0.5), np.where(k % 2 == 0, 0.5, -0.25),
                     np.where(k % 4 == 0, 1.5, 0.5) * np.where(k % 8 < 4, 1, -1)]).astype(np.float32)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("alternating") / "alternating.so")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-fPIC", "-shared", "-w", "-I", os.path.join(HERE, "hip_on_cpu"),
                        os.path.join(HERE, "hip_on_cpu", "alternating.cpp"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lib = ctypes.CDLL(out)
    lib.quantize_alternating.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int] + [ctypes.c_void_p] * 3 + [ctypes.c_int]
    return lib


def _run(lib, W, q, iters, backwards):
    V, n = W.shape
    alpha, packed, status = np.empty((q, V), np.float32), np.empty((q, V, n // 32), np.uint32), np.empty(1, np.int32)
    assert lib.quantize_alternating(W.ctypes.data, V, n, q, iters, alpha.ctypes.data, packed.ctypes.data, status.ctypes.data, backwards) == 0
    return alpha, packed, int(status[0])


@pytest.mark.parametrize("backwards", [0, 1])
@pytest.mark.parametrize("iters", [2, 13])
@pytest.mark.parametrize("n", [96, 1056, 2560, 4128])
@pytest.mark.parametrize("q", [2, 3, 4])
def test_no_wave_depends_on_the_others_pace(kernels, oracle, q, n, iters, backwards):
    rng = np.random.default_rng(n + q)
    W = np.concatenate([degenerate_rows(n), rng.standard_normal((2, n)).astype(np.float32)])
    alpha, packed, status = _run(kernels, W, q, iters, backwards)
    a_ref, b_ref, margin, _ = oracle.quantize_alternating(W, q, iters=iters, with_margin=True)
    robust = (margin[:, 0] >= 1e-9) & (margin[:, 1] >= 2.0 ** -40)
    assert status == 0 and robust.sum() >= 6
    assert np.array_equal(alpha[:, robust], a_ref[:, robust])
    assert np.array_equal(packed[:, robust], oracle.pack(b_ref)[:, robust])


@pytest.mark.parametrize("n", [1056, 4128])
def test_non_finite_vectors_in_either_order(kernels, n):
    W = np.random.default_rng(n).standard_normal((3, n)).astype(np.float32)
    clean = [_run(kernels, W, 3, 13, b) for b in (0, 1)]
    assert all(np.array_equal(a, b) for a, b in zip(*clean))
    W[0, 3], W[2, n - 1] = np.inf, np.nan
    for backwards in (0, 1):
        alpha, packed, status = _run(kernels, W, 3, 13, backwards)
        assert status == 2 and np.array_equal(alpha[:, 1], clean[0][0][:, 1]) and np.array_equal(packed[:, 1], clean[0][1][:, 1])
