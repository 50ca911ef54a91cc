"""The one-kernel forward (row-wise scales 81 .. 384 tokens of bf16, group-wise ones from 1 on; q <= 4) at the edges of its
tiles: 32, 64 or 128 tokens to a workgroup, scale tables per row, per pair of words or per word, the contraction whole or
in parts.  Every case checks that this kernel ran: the two-kernel path fills the whole workspace, this one
leaves the end of these.

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
    n = max(bcq.workspace_bytes_grouped(1, T, N, K, g, q, 1), 16)
    return torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda")


def _one_kernel(workspace):
    return bool((workspace[-16:] == 0x5A).all())


@pytest.mark.parametrize("T,N,K,g,q", [(96, 33, 32, 32, 1), (32, 40, 288, 96, 2), (32, 64, 288, 32, 3), (31, 31, 416, 32, 4),
                                       (100, 100, 160, 160, 4), (32, 65, 480, 160, 3), (32, 32, 512, 128, 2),
                                       (16, 1, 256, 64, 4), (64, 70, 512, 128, 2), (64, 2600, 480, 32, 4),
                                       (130, 4095, 320, 32, 2), (100, 8190, 192, 64, 4), (128, 8191, 96, 96, 3),
                                       (300, 800, 480, 480, 4)])
def test_expanded_weights_bit_exact(oracle, T, N, K, g, q):
    import torch
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, _, _ = make_case(1, "out", 1, N, K, q, "bf16", oracle, extra=N + K, g=g)
    alpha = alpha.reshape(q, N, K // g)
    what = np.zeros((N, K), dtype=np.float32)
    for i in range(q):
        what = what + np.repeat(alpha[i], g, axis=1) * planes[i].astype(np.float32)
    ref = torch.from_numpy(what).to(torch.bfloat16).t().contiguous()  # y[t = k][n]
    d_packed, d_alpha, eye = packed_to_dev(packed), to_dev(alpha), torch.eye(K, dtype=torch.bfloat16, device="cuda")
    for k in range(0, K, T):
        rows = min(T, K - k)
        x = torch.zeros((T, K), dtype=torch.bfloat16, device="cuda")
        x[:rows] = eye[k:k + rows]
        ws = _workspace(bcq, T, N, K, g, q)
        y = bcq.bcq_linear_fwd_grouped(d_packed, d_alpha, x, g, workspace=ws)
        assert _one_kernel(ws)
        assert torch.equal(y[:rows].cpu(), ref[k:k + rows])
        assert not y[rows:].any()


@pytest.mark.parametrize("T,N,K,g,q", [(1, 64, 64, 32, 3), (31, 35, 96, 96 // 3, 4), (32, 1056, 1024, 64, 2),
                                       (33, 320, 4128, 32, 4), (64, 65, 2048, 128, 3), (65, 130, 1056, 96, 1),
                                       (81, 70, 1056, 1056, 3), (128, 160, 320, 320, 4), (129, 257, 640, 640, 2),
                                       (384, 416, 1024, 1024, 4), (300, 1500, 32, 32, 1),
                                       (4, 33, 2080, 32, 3), (96, 100, 8224, 8224, 2), (200, 1030, 8192, 8192, 1),
                                       (1, 5, 16384, 64, 4), (100, 400, 3072, 96, 2),
                                       # 128 tokens to a workgroup: group-wise at every q, row-wise at q = 2, 3
                                       (250, 4100, 96, 32, 1), (130, 4095, 320, 32, 2), (140, 4099, 192, 64, 3),
                                       (100, 8190, 192, 64, 4), (100, 2030, 8224, 32, 4), (129, 4100, 96, 96, 2),
                                       (100, 8191, 64, 64, 3)])
def test_fused_forward(oracle, T, N, K, g, q):
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, _ = make_case(1, "out", T, N, K, q, "bf16", oracle, extra=T + N, g=g)
    ws = _workspace(bcq, T, N, K, g, q)
    y = bcq.bcq_linear_fwd_grouped(packed_to_dev(packed), to_dev(alpha.reshape(q, N, K // g)), to_dev(x, "bf16"), g,
                                   workspace=ws)
    assert _one_kernel(ws)
    ref = oracle.fwd(alpha.reshape(q, N) if g == K else alpha, planes, x)
    assert nmax_err(to_host(y), ref) <= 1e-2


@pytest.mark.parametrize("T,N,K,g,q", [(385, 500, 512, 512, 2), (33, 96, 4128, 32, 4), (384, 2560, 256, 64, 4),
                                       (64, 100, 320, 32, 5)])
def test_beyond_the_rule_two_kernels_run(oracle, T, N, K, g, q):
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, _ = make_case(1, "out", T, N, K, q, "bf16", oracle, extra=T + N, g=g)
    ws = _workspace(bcq, T, N, K, g, q)
    y = bcq.bcq_linear_fwd_grouped(packed_to_dev(packed), to_dev(alpha.reshape(q, N, K // g)), to_dev(x, "bf16"), g,
                                   workspace=ws)
    assert not _one_kernel(ws)
    ref = oracle.fwd(alpha.reshape(q, N) if g == K else alpha, planes, x)
    assert nmax_err(to_host(y), ref) <= 1e-2


@pytest.mark.parametrize("T,N,K,q", [(257, 8200, 992, 4), (129, 40100, 1024, 1)])
def test_rows_beyond_the_size_line(oracle, T, N, K, q):
    """Row-wise scales: one token less takes one kernel, and both agree with the oracle (same bound as above)."""
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, _ = make_case(1, "out", T, N, K, q, "bf16", oracle, extra=T + N)
    ref = oracle.fwd(alpha.reshape(q, N), planes, x)
    d_packed, d_alpha, dx = packed_to_dev(packed), to_dev(alpha.reshape(q, N, 1)), to_dev(x, "bf16")
    for tokens in (T, T - 1):
        ws = _workspace(bcq, tokens, N, K, K, q)
        y = bcq.bcq_linear_fwd_grouped(d_packed, d_alpha, dx[:tokens].contiguous(), K, workspace=ws)
        assert _one_kernel(ws) == (tokens < T)
        assert nmax_err(to_host(y), ref[:tokens]) <= 1e-2


@pytest.mark.parametrize("T,N,K,q,one", [(320, 1632, 5056, 4, True), (320, 1664, 5056, 4, False),
                                         (160, 8192, 4896, 2, True), (160, 8224, 4896, 2, False),
                                         (160, 5120, 7840, 1, False), (288, 5120, 8000, 3, False), (130, 25024, 4000, 1, True)])
def test_large_layers_in_one_full_round(T, N, K, q, one):
    """Row-wise scales beyond the size line take one kernel where its workgroups fill one round: 255 against 260 of 64 tokens,
    512 against 514 of 128 tokens, 320 and three tiles of 128 tokens; above 100 million weights always.  Same bound as above,
    against fp32 products."""
    import torch
    import paper_2210_03858_amd as bcq
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    packed = torch.randint(-2**31, 2**31 - 1, (q, N, K // 32), dtype=torch.int32, device="cuda", generator=gen)
    alpha = torch.rand((q, N, 1), device="cuda", generator=gen) + 0.1
    x = torch.randn((T, K), device="cuda", generator=gen).bfloat16()
    bits = torch.arange(32, dtype=torch.int32, device="cuda")
    w = sum((2 * ((packed[i].unsqueeze(-1) >> bits) & 1) - 1).reshape(N, K) * alpha[i] for i in range(q))
    ws = _workspace(bcq, T, N, K, K, q)
    y = bcq.bcq_linear_fwd_grouped(packed, alpha, x, K, workspace=ws)
    assert _one_kernel(ws) == one
    assert nmax_err(to_host(y), (x.float() @ w.t()).cpu().numpy()) <= 1e-2


@pytest.mark.parametrize("T,N,K,g,q", [(8, 40, 96, 32, 2), (40, 40, 96, 32, 1), (100, 200, 160, 160, 1), (300, 8200, 160, 160, 3)])
def test_infinite_scale_stays_in_its_row(oracle, T, N, K, g, q):
    """Columns beyond an odd number of words are zero activations: an infinite scale must not meet them."""
    import paper_2210_03858_amd as bcq
    import torch
    _, alpha, _, packed, _, _ = make_case(1, "out", T, N, K, q, "bf16", oracle, g=g)
    packed, alpha = packed.copy(), alpha.reshape(q, N, K // g).copy()
    packed[:, 3], alpha[0, 3] = 0xFFFFFFFF, np.inf
    x = torch.rand((T, K), device="cuda").add_(0.5).bfloat16()
    ws = _workspace(bcq, T, N, K, g, q)
    y = bcq.bcq_linear_fwd_grouped(packed_to_dev(packed), to_dev(alpha), x, g, workspace=ws)
    assert _one_kernel(ws)
    assert (y[:, 3] == float("inf")).all()
    assert torch.cat((y[:, :3], y[:, 4:]), dim=1).isfinite().all()
