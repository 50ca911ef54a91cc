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
    lib.quantize_alternating.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int] + [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_void_p]
    lib.last_kernel.restype = ctypes.c_char_p
    return lib


def _run(lib, W, q, iters, backwards=0):
    """(scales, words, non-finite vectors, operations over lanes)"""
    V, n = W.shape
    alpha, packed, status, operations = np.empty((q, V), np.float32), np.empty((q, V, n // 32), np.uint32), np.empty(1, np.int32), np.empty(1, np.int64)
    assert lib.quantize_alternating(W.ctypes.data, V, n, q, iters, alpha.ctypes.data, packed.ctypes.data, status.ctypes.data, backwards,
                                    operations.ctypes.data) == 0
    return alpha, packed, int(status[0]), int(operations[0])


@pytest.mark.parametrize("backwards", [0, 1])
@pytest.mark.parametrize("iters", [2, 13])
@pytest.mark.parametrize("n", [96, 1056, 2560, 4128])
@pytest.mark.parametrize("q", [2, 3, 4])
def test_no_wave_depends_on_the_others_pace(kernels, oracle, q, n, iters, backwards):
    rng = np.random.default_rng(n + q)
    W = np.concatenate([degenerate_rows(n), rng.standard_normal((2, n)).astype(np.float32)])
    alpha, packed, status, _ = _run(kernels, W, q, iters, backwards)
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
        alpha, packed, status, _ = _run(kernels, W, 3, 13, backwards)
        assert status == 2 and np.array_equal(alpha[:, 1], clean[0][0][:, 1]) and np.array_equal(packed[:, 1], clean[0][1][:, 1])


@pytest.mark.parametrize("q,n,line", [(2, 96, 8), (3, 256, 8), (4, 1024, 8), (3, 1056, 12)])
def test_no_sorting_for_an_element_far_below_the_levels(kernels, q, n, line):
    """With such an element every round takes the fp64 distances.  The vector reaches its fixed point in two rounds, so that it costs one round
    below and at the line of the sorted form the same but for the question itself; without the element the sorting shows."""
    rng = np.random.default_rng(n)
    levels = np.array([sum((1 if c >> i & 1 else -1) * 2.0 ** -i for i in range(q)) for c in range(2 ** q)])
    W = (levels[rng.integers(0, 2 ** q, (1, n))] + 0.01 * rng.standard_normal((1, n))).astype(np.float32)
    sorting = _run(kernels, W, q, line)[3] - _run(kernels, W, q, line - 1)[3]
    assert sorting > 40
    W[0, n // 2] = 1e-12
    below, at = _run(kernels, W, q, line - 1), _run(kernels, W, q, line)
    assert np.array_equal(below[0], at[0]) and np.array_equal(below[1], at[1])
    assert abs(at[3] - below[3]) <= 8 * (1 if n <= 1024 else 2)


@pytest.mark.parametrize("q,n,rounds", [(2, 32, None), (2, 64, 8), (2, 1024, 8), (2, 1056, None), (3, 32, 8), (3, 1024, 8), (3, 1056, 12), (3, 3072, 12),
                                        (3, 3104, 15), (3, 4096, 15), (3, 4128, None), (4, 32, None), (4, 64, 12), (4, 256, 12), (4, 288, 8),
                                        (4, 1024, 8), (4, 1056, None)])
def test_short_vectors_are_sorted_only_where_they_repay_it(kernels, q, n, rounds):
    """The number of rounds from which the form with sorted elements is launched; None: not even for 1000."""
    W = np.tile(np.float32([0.5, -0.25, 0.25, -0.5]), n // 4)[None]
    for iters, sorts in ((1000, rounds is not None), (rounds, True), (rounds and rounds - 1, False)):
        if iters is not None:
            _run(kernels, W, q, iters)
            name = kernels.last_kernel().decode()
            assert "alternating_reg_kernelILi%dE" % q in name and ("ELb1E" in name) == sorts, (iters, name)
