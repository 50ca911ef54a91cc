"""The one-kernel forward (32 .. 512 tokens of bf16, or group-wise scales; q <= 4) at the edges of its tiles.

With one-hot tokens a result is one weight, so the whole expanded matrix is compared bit for bit with the fp32 sums of
the scales (same order) rounded once to bf16.  With random tokens the error is that of rounding every weight and the
result to bf16: 2^-8 of the value each at most, and the weights' errors average over the contraction, so the
normalised error stays below 2^-8 (result) + 4 * 2^-8 / sqrt(3) / sqrt(K) * |y|_max-scale, under 1e-2 from 32 columns on."""
import numpy as np
import pytest

from _util import make_case, nmax_err, packed_to_dev, to_dev, to_host

pytestmark = pytest.mark.gpu


def _workspace(bcq, T, N, K, g, q):
    import torch
    return torch.empty((max(bcq.workspace_bytes_grouped(1, T, N, K, g, q, 1), 16),), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("N,K,g,q", [(33, 32, 32, 1), (40, 288, 96, 2), (64, 288, 32, 3), (31, 416, 32, 4),
                                     (100, 160, 160, 4), (65, 480, 160, 3), (32, 512, 128, 2), (1, 256, 64, 4)])
def test_expanded_weights_bit_exact(oracle, N, K, g, q):
    import torch
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, _, _ = make_case(1, "out", 1, N, K, q, "bf16", oracle, extra=N + K, g=g)
    alpha = alpha.reshape(q, N, K // g)
    what = np.zeros((N, K), dtype=np.float32)
    for i in range(q):
        what = what + np.repeat(alpha[i], g, axis=1) * planes[i].astype(np.float32)
    ref = torch.from_numpy(what).to(torch.bfloat16).t().contiguous()  # y[t = k][n]
    T = max(K, 81)  # more tokens than the streaming kernels take; the rest are zero
    x = torch.zeros((T, K), dtype=torch.bfloat16, device="cuda")
    x[:K] = torch.eye(K, dtype=torch.bfloat16, device="cuda")
    y = bcq.bcq_linear_fwd_grouped(packed_to_dev(packed), to_dev(alpha), x, g, workspace=_workspace(bcq, T, N, K, g, q))
    assert torch.equal(y[:K].cpu(), ref)
    assert not y[K:].any()


@pytest.mark.parametrize("T,N,K,g,q", [(1, 64, 64, 32, 3), (31, 35, 96, 96 // 3, 4), (32, 1056, 1024, 64, 2),
                                       (33, 96, 4128, 32, 4), (64, 33, 2048, 128, 3), (65, 130, 1056, 96, 1),
                                       (81, 70, 1056, 1056, 3), (128, 64, 320, 320, 4), (129, 257, 640, 640, 2),
                                       (512, 40, 1024, 1024, 4), (300, 1500, 32, 32, 1),
                                       (4, 33, 2080, 32, 3), (40, 70, 8224, 8224, 2), (200, 1030, 8192, 8192, 1),
                                       (1, 5, 16384, 64, 4), (100, 161, 3072, 96, 2)])
def test_fused_forward(oracle, T, N, K, g, q):
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, _ = make_case(1, "out", T, N, K, q, "bf16", oracle, extra=T + N, g=g)
    y = bcq.bcq_linear_fwd_grouped(packed_to_dev(packed), to_dev(alpha.reshape(q, N, K // g)), to_dev(x, "bf16"), g,
                                   workspace=_workspace(bcq, T, N, K, g, q))
    ref = oracle.fwd(alpha.reshape(q, N) if g == K else alpha, planes, x)
    assert nmax_err(to_host(y), ref) <= 1e-2


@pytest.mark.parametrize("T,N,K,g,q", [(8, 40, 96, 32, 2), (40, 40, 96, 32, 4), (100, 200, 160, 160, 1), (300, 8200, 160, 160, 3)])
def test_infinite_scale_stays_in_its_row(oracle, T, N, K, g, q):
    """Columns beyond an odd number of words are zero activations: an infinite scale must not meet them."""
    import paper_2210_03858_amd as bcq
    import torch
    _, alpha, _, packed, _, _ = make_case(1, "out", T, N, K, q, "bf16", oracle, g=g)
    packed, alpha = packed.copy(), alpha.reshape(q, N, K // g).copy()
    packed[:, 3], alpha[0, 3] = 0xFFFFFFFF, np.inf
    x = torch.rand((T, K), device="cuda").add_(0.5).bfloat16()
    y = bcq.bcq_linear_fwd_grouped(packed_to_dev(packed), to_dev(alpha), x, g, workspace=_workspace(bcq, T, N, K, g, q))
    assert (y[:, 3] == float("inf")).all()
    assert torch.cat((y[:, :3], y[:, 4:]), dim=1).isfinite().all()
