"""Backward products whose rows of dy are not 16-byte aligned, large enough for the padded bf16 matrix-core forms.

The input gradient multiplies with 24-bit weights (three bf16 terms), so its error is one rounding to bf16, 2^-8 of the
value, and an fp32 accumulation (5 % allowed on top); the scale gradient is an fp32 sum of exact products."""
import numpy as np
import pytest

from _util import TOL_F32, make_case, nmax_err, packed_to_dev, to_dev, to_host

pytestmark = pytest.mark.gpu


def _ws(bcq, op, T, N, K, g, q, small):
    import torch
    n = 16 if small else bcq.workspace_bytes_grouped(op, T, N, K, g, q, 1)
    return torch.empty((max(n, 16),), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("T,N,K,g,q,q_train", [(333, 1500, 1056, 1056, 3, 3), (800, 1001, 512, 32, 4, 1),
                                               (6000, 7, 10240, 10240, 2, 2), (97, 4097, 1024, 512, 2, 1),
                                               (31, 4404, 2976, 2976, 1, 1)])
@pytest.mark.parametrize("small", [False, True])
def test_unaligned_backward(oracle, T, N, K, g, q, q_train, small):
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, dy = make_case(1, "out", T, N, K, q, "bf16", oracle, extra=T + N, g=g)
    d_packed, d_alpha, d_dy = packed_to_dev(packed), to_dev(alpha.reshape(q, N, K // g)), to_dev(dy, "bf16")
    a_or = alpha.reshape(q, N) if g == K else alpha
    dx = bcq.bcq_linear_bwd_input_grouped(d_packed, d_alpha, d_dy, g, workspace=_ws(bcq, 2, T, N, K, g, q, small))
    assert nmax_err(to_host(dx), oracle.bwd_input(a_or, planes, dy)) <= 1.05 * 2.0 ** -8
    da = bcq.bcq_linear_bwd_alpha_grouped(d_packed, to_dev(x, "bf16"), d_dy, g, q_train=q_train,
                                          workspace=_ws(bcq, 3, T, N, K, g, q, small))
    ref = oracle.bwd_alpha(planes, x, dy, q_train=q_train, grad_scale=1.0, g=g)
    assert nmax_err(to_host(da).reshape(ref.shape), ref) <= TOL_F32


def test_unaligned_input_gradient_keeps_infinities_and_nan(oracle):
    import torch
    import paper_2210_03858_amd as bcq
    T, N, K, q = 260, 1500, 1056, 2
    _, alpha, planes, packed, _, dy = make_case(1, "out", T, N, K, q, "bf16", oracle)
    dy[3, 70], dy[9, 5], dy[20, 1499] = np.inf, np.nan, -np.inf
    alpha = alpha.reshape(q, N, 1)
    args = packed_to_dev(packed), to_dev(alpha), to_dev(dy, "bf16"), K
    ref = bcq.bcq_linear_bwd_input_grouped(*args).float()  # without a workspace: one fp64 sum
    got = bcq.bcq_linear_bwd_input_grouped(*args, workspace=_ws(bcq, 2, T, N, K, K, q, False)).float()
    for t in (3, 9, 20):
        finite = ref[t].isfinite()
        assert torch.equal(finite, got[t].isfinite()) and torch.equal(ref[t].isnan(), got[t].isnan())
        assert torch.equal(ref[t][~finite & ~ref[t].isnan()], got[t][~finite & ~ref[t].isnan()])


@pytest.mark.parametrize("scale", [3.4e38, -3.3961776e38, 1e-37])
def test_unaligned_input_gradient_at_the_ends_of_the_weights_range(oracle, scale):
    """Weights beyond bf16's largest value, and ones whose lower terms are subnormal bf16 values (and may be flushed, which
    leaves 16 significant bits): one rounding of the result, as for all others."""
    import paper_2210_03858_amd as bcq
    T, N, K = 260, 1500, 1056
    _, alpha, _, packed, _, dy = make_case(1, "out", T, N, K, 1, "bf16", oracle)
    alpha, dy = alpha.reshape(1, N, 1).copy(), dy.copy()
    alpha[0, 7], dy[:, 7], dy[5] = scale, 0.0, 0.0
    dy[5, 7] = 2.0 ** -20 if abs(scale) > 1.0 else 2.0 ** 20
    args = packed_to_dev(packed), to_dev(alpha), to_dev(dy, "bf16"), K
    ref = bcq.bcq_linear_bwd_input_grouped(*args).double()  # without a workspace: one fp64 sum
    got = bcq.bcq_linear_bwd_input_grouped(*args, workspace=_ws(bcq, 2, T, N, K, K, 1, False)).double()
    assert ref.isfinite().all() and got.isfinite().all()
    assert ((got - ref).abs().amax(1) <= 1.05 * 2.0 ** -7 * ref.abs().amax(1)).all()  # each rounds once


@pytest.mark.parametrize("T,N,K,g", [(6000, 50257, 64, 64), (5400, 50257, 64, 32), ((1 << 20) + 100, 7, 32, 32)])
def test_scale_gradient_in_pieces(T, N, K, g):
    """More tokens than one padded copy of dy holds (512 MiB, 2^20 tokens): partial sums of two pieces."""
    import torch
    import paper_2210_03858_amd as bcq
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    packed = torch.randint(-2 ** 31, 2 ** 31, (2, N, K // 32), dtype=torch.int32, device="cuda", generator=gen)
    x = torch.randn((T, K), device="cuda", generator=gen).bfloat16()
    dy = torch.empty((T, N), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    ref = bcq.bcq_linear_bwd_alpha_grouped(packed, x, dy, g)  # without a workspace: one fp64 sum
    got = bcq.bcq_linear_bwd_alpha_grouped(packed, x, dy, g, workspace=_ws(bcq, 3, T, N, K, g, 2, False))
    assert nmax_err(to_host(got), to_host(ref)) <= TOL_F32
