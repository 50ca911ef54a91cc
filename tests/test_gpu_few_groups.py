"""The forward of at most 32 tokens with group-wise scales in one kernel at the edges of its plan: one, two and four words to a
lane, both token tiles, ragged rows and columns, one and several turns of the waves, and the contraction in parts.

The kernel multiplies bf16 weights (the scales' fp32 sums rounded once) with the activations as they are, so against fp64 products
of those weights only its fp32 sums and the one rounding of the result differ: 2^-8 of every value and, for at most 2^14 terms added
in some order, 1e-5 of the largest.  The profiler names the kernel that ran.
"""
import pytest
import torch

import paper_2210_03858_amd as bcq
from test_gpu_few import _layer, _run

pytestmark = pytest.mark.gpu


def _rounded(packed, alpha, g):
    """sum_i alpha_i B_i in fp32, plane by plane, rounded once to bf16."""
    q, N, words = packed.shape
    bits = torch.arange(32, dtype=torch.int32, device="cuda")
    w = torch.zeros((N, words * 32), device="cuda")
    for i in range(q):
        w = w + alpha[i].repeat_interleave(g, dim=1) * (2 * ((packed[i].unsqueeze(-1) >> bits) & 1) - 1).reshape(N, -1)
    return w.bfloat16().double()


@pytest.mark.parametrize("T,N,K,g,q", [
    (1, 1, 64, 32, 1), (4, 6144, 2048, 128, 3), (3, 33, 384, 128, 4), (16, 4100, 1152, 384, 2),         # four words
    (16, 20, 256, 128, 3), (17, 2050, 640, 128, 2), (32, 4097, 2560, 64, 4), (5, 300, 192, 64, 3),      # two, and down for few waves
    (31, 70, 288, 96, 1), (16, 515, 1056, 96, 3), (8, 40, 160, 32, 4),  # one
    (32, 1280, 5120, 32, 4), (13, 303, 10624, 128, 3), (32, 16, 16384, 64, 2), (2, 2048, 8192, 128, 3), (15, 100, 4128, 32, 2)])  # turns, parts
def test_few_tokens_with_groups(T, N, K, g, q):
    packed, alpha, x, _ = _layer(q, N, K, g, T, T + N + K)
    y = _run("canonical", packed, alpha, x, g, kernel="group_fwd_kernel").double()
    ref = x.double() @ _rounded(packed, alpha, g).t()
    assert ((y - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max()).all()


@pytest.mark.parametrize("T,N,K,g,q", [(4, 40, 288, 96, 2), (20, 300, 1088, 64, 3), (8, 100, 640, 128, 4)])
def test_non_finite_token_keeps_to_itself(T, N, K, g, q):
    """An infinity in the last columns gives its token infinities of the weights' signs, a NaN gives NaN, no other token changes."""
    packed, alpha, x, _ = _layer(q, N, K, g, T, N)
    clean = _run("canonical", packed, alpha, x, g, kernel="group_fwd_kernel")
    x[1, K - 1], x[3, 0] = float("inf"), float("nan")
    y = _run("canonical", packed, alpha, x, g, kernel="group_fwd_kernel")
    sign = _rounded(packed, alpha, g)[:, K - 1].sign()
    assert (y[1].double() == float("inf") * sign)[sign != 0].all() and y[3].isnan().all()
    keep = (torch.arange(T, device="cuda") != 1) & (torch.arange(T, device="cuda") != 3)
    assert torch.equal(y[keep], clean[keep])
