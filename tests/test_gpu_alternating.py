"""Parity of bcq_quantize_alternating (Appendix C, Eq. ap4) with the CPU oracle, through the C ABI.

Sign planes, packed words and the fp32 scales are compared bit for bit on every vector whose decisions the oracle
reports as robust: the gap between the best and the second-best level of every element in every round is at least
1e-9 of sum_i |alpha_i| (the two sides add the same fp64 numbers in different orders, which moves alpha by about
1e-16), and no returned alpha sits within 2^-40 of an fp32 rounding boundary.  Fragile vectors must be rare."""
import numpy as np
import pytest

from _util import packed_to_host, to_dev
from test_cpu_alternating import degenerate_rows
from paper_2210_03858_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bcq():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2210_03858_amd as p
    p.load()
    return p


def _check(bcq, oracle, W, q, iters=15, g=None):
    import torch
    N, K = W.shape
    gg = K if g is None else g
    V = N * (K // gg)
    a_ref, b_ref, margin, done = oracle.quantize_alternating(W, q, iters=iters, g=g, with_margin=True)
    ws = torch.full((4,), 77, dtype=torch.int32, device="cuda")
    alpha, packed, planes = bcq.bcq_quantize_alternating(to_dev(W), q, iters=iters, g=g, want_planes=True, workspace=ws)
    torch.cuda.synchronize()
    assert int(ws[0].item()) == 0
    packed = packed_to_host(packed)
    planes_gpu = oracle.unpack(packed, K)
    assert np.array_equal(planes.cpu().numpy(), planes_gpu)
    alpha_v = alpha.cpu().numpy().reshape(q, V)
    a_ref = a_ref.reshape(q, V)
    pv, bv = planes_gpu.reshape(q, V, gg), b_ref.reshape(q, V, gg)
    robust = (margin[:, 0] >= 1e-9) & (margin[:, 1] >= 2.0 ** -40)
    assert (~robust).sum() <= max(1, V // 1000), (~robust).sum()
    assert np.array_equal(alpha_v[:, robust].view(np.uint32), a_ref[:, robust].view(np.uint32))
    assert np.array_equal(pv[:, robust], bv[:, robust])
    # fragile vectors: still a valid quantization whose error is as good as the oracle's, up to the flipped decision
    for v in np.nonzero(~robust)[0]:
        w = W.reshape(V, gg)[v].astype(np.float64)
        e_gpu = ((w - (alpha_v[:, v].astype(np.float64)[:, None] * pv[:, v]).sum(axis=0)) ** 2).sum()
        e_ref = ((w - (a_ref[:, v].astype(np.float64)[:, None] * bv[:, v]).sum(axis=0)) ** 2).sum()
        assert e_gpu <= e_ref * 1.05 + 1e-30
    return done


@pytest.mark.parametrize("q,N,K,g", [(1, 16, 128, None), (2, 40, 256, None), (3, 64, 1024, None), (4, 32, 1280, None),
                                     (3, 24, 1024, 256), (4, 10, 4096, None), (2, 6, 16384, None), (5, 8, 160, None),
                                     (8, 4, 256, 64), (3, 50, 96, 32)])
def test_alternating_bit_exact(bcq, oracle, q, N, K, g):
    W = synth.weights(1, "out", N, K, extra=7 * K + q)
    done = _check(bcq, oracle, W, q, g=g)
    if q > 1:
        assert done.max() > 1   # the refinement really runs


def test_alternating_zero_iterations_and_few(bcq, oracle):
    W = synth.weights(1, "out", 48, 512)
    _check(bcq, oracle, W, 3, iters=0)
    _check(bcq, oracle, W, 3, iters=1)
    _check(bcq, oracle, W, 3, iters=4)


def test_alternating_degenerate_rows_and_outliers(bcq, oracle):
    W = synth.weights(4, "qkv", 256, 512, outliers=True)
    W[5] = 0.0
    W[6, ::2] = 0.0
    W[7, :3] = [-0.0, 0.0, 1.0]
    W[8] = 0.25          # constant vector: every plane after the first has a zero residual
    W[9, :] = np.where(np.arange(512) % 2 == 0, 0.5, -0.25)
    _check(bcq, oracle, W, 3)


def test_alternating_reports_nonfinite_vectors(bcq):
    import torch
    W = synth.weights(1, "out", 64, 256)
    W[3, 7] = np.inf
    W[40, 0] = np.nan
    ws = torch.zeros((4,), dtype=torch.int32, device="cuda")
    bcq.bcq_quantize_alternating(to_dev(W), 2, workspace=ws)
    torch.cuda.synchronize()
    assert int(ws[0].item()) == 2


def test_alternating_gpt2_medium_layer(bcq, oracle):
    """One full (h, h) layer of the GPT-2-medium block, q = 3, 15 rounds."""
    W = synth.weights(2, "out", 1024, 1024)
    _check(bcq, oracle, W, 3)


@pytest.mark.parametrize("q,N,K,g", [(3, 9, 288, None), (2, 7, 512, None), (6, 5, 544, None), (7, 4, 1056, None),
                                     (1, 3, 32, None), (4, 3, 2080, None), (3, 2, 8192, 256)])
def test_alternating_wave_counts_and_plane_counts(bcq, oracle, q, N, K, g):
    """One, two and four waves per vector with partly idle waves, every specialisation by q, same bar as above."""
    _check(bcq, oracle, synth.weights(1, "out", N, K, extra=11 * K + q), q, g=g)


@pytest.mark.parametrize("q,N,K,g", [(5, 6, 256, 32), (6, 4, 768, None), (7, 3, 512, 256), (8, 5, 1056, None)])
def test_alternating_bisection(bcq, oracle, q, N, K, g):
    """Five planes and more find the nearest level by bisection: same bar, with a zero and a constant row."""
    W = synth.weights(1, "out", N, K, extra=q)
    W[0], W[1] = 0.0, 0.25
    _check(bcq, oracle, W, q, g=g)


@pytest.mark.parametrize("kind", ["normal", "small", "large"])
@pytest.mark.parametrize("N,K", [(40, 32), (12, 256), (12, 288), (8, 512), (8, 544), (6, 1024), (6, 1056), (3, 4096), (2, 4128), (2, 14336), (1, 16384)])
def test_registers_and_thresholds(bcq, oracle, N, K, kind):
    """One to eight waves with 4 to 32 elements per lane, at and behind each limit.  Scaling by a power of two changes no
    decision; above 1e30 every round compares distances (all levels) instead of thresholds.  (Elements far above or below
    the levels get there too, but are no input for this check: from 2^-30 of sum |alpha| down, an element's two nearest
    levels +l and -l differ in distance by less than the 1e-9 of it that make a vector robust.)"""
    for q in (1, 2, 3, 4):
        W = synth.weights(1, "out", N, K, extra=11 * K + q)
        W *= np.float32({"normal": 1.0, "small": 2.0 ** -60, "large": 2.0 ** 106}[kind])
        _check(bcq, oracle, W, q, iters=6)


@pytest.mark.parametrize("K", [64, 256, 1024, 4096, 16384])
def test_ties_at_floats(bcq, oracle, K):
    """Levels at the odd multiples of 1 / 64 up to 2^q - 1 of them, elements on every level and one step below it, which is
    the middle of two levels, on both sides of zero: the greedy start already ends there, the refit returns the same
    scales exactly (powers of four for K: the oracle's solve takes its square root), and every tie has to go to the larger
    level for the planes to stay as they are."""
    rng = np.random.default_rng(K)
    for q in (1, 2, 3, 4):
        levels = np.arange(-(2 ** q - 1), 2 ** q, 2)
        vector = np.tile(np.concatenate((levels, levels - 1)), K // (2 * 2 ** q))
        W = np.stack([rng.permutation(vector) for _ in range(6)]).astype(np.float32) / 64.0
        alpha, packed, _ = bcq.bcq_quantize_alternating(to_dev(W), q, iters=15)
        want = np.array([2.0 ** (q - 1 - i) / 64.0 for i in range(q)], dtype=np.float32)
        assert np.array_equal(alpha.cpu().numpy().reshape(q, 6), np.repeat(want[:, None], 6, axis=1))
        planes = oracle.unpack(packed_to_host(packed), K).reshape(q, 6, K)
        assert np.array_equal((planes * want[:, None, None]).sum(axis=0), (W * 64.0 + (W * 64.0 % 2 == 0)) / 64.0)
        a_ref, b_ref = oracle.quantize_alternating(W, q, iters=15)[:2]
        assert np.array_equal(planes, b_ref.reshape(q, 6, K)) and np.array_equal(alpha.cpu().numpy().reshape(q, 6), a_ref.reshape(q, 6))


@pytest.mark.parametrize("K", [64, 1024, 2048, 6144])
@pytest.mark.parametrize("factor", [2.0 ** -60, 2.0 ** 22])
def test_elements_far_from_the_levels(bcq, oracle, K, factor):
    """One element of every vector far below or above the levels takes the rounds to the fp64 distances.  Its own decision may hang
    on the last bit of a scale, the vector's error may not: 1e-6 of it is far above what one such element can change."""
    for q in (2, 3, 4):
        W = synth.weights(1, "out", 6, K, extra=K + q)
        W[:, K - 5] = np.where(W[:, K - 5] == 0, 0.01, W[:, K - 5]) * np.float32(factor)
        alpha, packed, _ = bcq.bcq_quantize_alternating(to_dev(W), q, iters=15)
        a = alpha.cpu().numpy().reshape(q, 6, 1).astype(np.float64)
        b = oracle.unpack(packed_to_host(packed), K).reshape(q, 6, K)
        a_ref, b_ref = oracle.quantize_alternating(W, q, iters=15)[:2]
        w64 = W.astype(np.float64)
        e_gpu = ((w64 - (a * b).sum(0)) ** 2).sum(1)
        e_ref = ((w64 - (a_ref.reshape(q, 6, 1).astype(np.float64) * b_ref.reshape(q, 6, K)).sum(0)) ** 2).sum(1)
        assert (e_gpu <= (1.0 + 1e-6) * e_ref).all() and (e_ref <= (1.0 + 1e-6) * e_gpu).all(), (e_gpu / e_ref)


@pytest.mark.parametrize("K", [1056, 4096, 16384])
def test_nonfinite_vectors_of_several_waves(bcq, oracle, K):
    """An infinity in the first wave's elements and a NaN in the last one's: both counted, the other vectors as ever."""
    import torch
    for q in (1, 3, 4):
        W = synth.weights(1, "out", 5, K, extra=q)
        clean = W.copy()
        W[1, 3], W[3, K - 1] = np.inf, np.nan
        ws = torch.zeros((4,), dtype=torch.int32, device="cuda")
        alpha, packed, _ = bcq.bcq_quantize_alternating(to_dev(W), q, workspace=ws)
        assert int(ws[0].item()) == 2
        alpha_c, packed_c, _ = bcq.bcq_quantize_alternating(to_dev(clean), q)
        keep = [0, 2, 4]
        assert torch.equal(alpha.reshape(q, 5)[:, keep], alpha_c.reshape(q, 5)[:, keep])
        assert torch.equal(packed.reshape(q, 5, -1)[:, keep], packed_c.reshape(q, 5, -1)[:, keep])


@pytest.mark.parametrize("kind", ["normal", "heavy", "grid", "two"])
@pytest.mark.parametrize("N,K", [(9, 32), (9, 96), (6, 256), (6, 288), (5, 480), (5, 544), (5, 992), (5, 1024), (4, 1056), (4, 2560),
                                 (3, 4096)])
def test_rounds_from_the_sorted_elements(bcq, oracle, N, K, kind):
    """One to four waves, with idle lanes and none, one round below and at the lines from which their elements are sorted: normal
    and heavy-tailed weights (levels that change their order, counts that stay), weights on a coarse grid (ties with the greedy levels
    and equal elements on both sides of a threshold) and two magnitudes (the later planes have next to nothing left).  Same bar."""
    rng = np.random.default_rng(K + N)
    for q in (2, 3, 4):
        W = rng.standard_normal((N, K)).astype(np.float32)
        if kind == "heavy":
            W = np.sign(W) * (np.abs(W) ** 3 + 0.01)  # (elements next to zero are as near to +l as to -l: no robust vectors)
        if kind == "grid":
            W = np.round(W * 8 + 0.25) / 8 + np.float32(1e-3) * rng.standard_normal((N, 1)).astype(np.float32)
        if kind == "two":
            W = np.where(np.abs(W) > 0.6, 0.7, 0.3) * np.sign(W) + np.float32(1e-6) * W
        for iters in (7, 8, 15) if K <= 1024 else (11, 12, 15):
            _check(bcq, oracle, W.astype(np.float32), q, iters=iters)


@pytest.mark.parametrize("K", [1056, 2560, 4096, 4128])
def test_singular_first_round_of_several_waves(bcq, oracle, K):
    """Zero, constant and two-magnitude vectors return the scales of the greedy start: refused by the start from the sorted elements, and in
    the forms that do not sort."""
    for q in (2, 3, 4):
        W = np.concatenate([degenerate_rows(K), synth.weights(1, "out", 3, K, extra=K + q)])
        for iters in (0, 1, 11, 12, 15):
            _check(bcq, oracle, W, q, iters=iters)
