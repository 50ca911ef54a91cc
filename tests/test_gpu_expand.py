"""Expanded weights of the large-token route, bit for bit.

With one-hot rows of activations every element of Y = X W^T and dX = dY W is one weight, rounded once to bf16 when the sum of
the planes is stored and exact from there on.  Sizes are edges of the expansion's blocks: fewer rows than a fragment, rows
that are no multiple of 8 or 32, one word, word counts below and above a block's 8 or 32, scale groups of one word.  The
blocks are in the order of the XCDs that read them in the product at 640 tokens and 1000 or more columns, else in plain order; the
input gradient of five planes and more only where the column words make even eighths (32 and 63, not 33 or 65).
"""
import pytest
import torch

import paper_2210_03858_amd as bcq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("N,K,g,T", [(5, 32, 32, 640), (32, 256, 32, 640), (72, 288, 96, 640), (264, 1056, 1056, 640),
                                     (300, 2080, 32, 640), (264, 1056, 32, 3200), (1000, 96, 32, 640),
                                     (264, 1024, 32, 640), (288, 2016, 32, 640)])
def test_expanded_weights_bit_exact(N, K, g, T, q):
    gen = torch.Generator().manual_seed(N * K + q)
    packed = torch.randint(-2**31, 2**31 - 1, (q, N, K // 32), dtype=torch.int32, generator=gen)
    alpha = torch.rand((q, N, K // g), generator=gen) - 0.3
    bits = (packed.unsqueeze(-1) >> torch.arange(32, dtype=torch.int32)) & 1
    signs = (2 * bits.reshape(q, N, K) - 1).float()
    w = torch.zeros(N, K)
    for i in range(q):  # in plane order, in fp32
        w += signs[i] * alpha[i].repeat_interleave(g, dim=1)
    want = w.bfloat16()
    packed, alpha = packed.cuda(), alpha.cuda()
    twin = bcq.bcq_pack_transposed(packed) if N % 32 == 0 else None

    def rows(n):  # a row of the identity per token, and enough zero rows for the large-token route
        x = torch.zeros((max(n, T), n), dtype=torch.bfloat16, device="cuda")
        x[:n] = torch.eye(n, dtype=torch.bfloat16, device="cuda")
        return x

    x, dy = rows(K), rows(N)
    ws = [torch.empty(bcq.workspace_bytes_grouped(op, t.shape[0], N, K, g, q, 1), dtype=torch.uint8, device="cuda")
          for op, t in ((1, x), (2, dy))]
    y = bcq.bcq_linear_fwd_grouped(packed, alpha, x, g, workspace=ws[0])
    assert torch.equal(y[:K].t().cpu(), want)
    if N % 8:  # dX takes other kernels there, whose sums over planes and rows are not one rounding of a weight
        return
    for t in {twin is not None, False}:
        dx = bcq.bcq_linear_bwd_input_grouped(packed, alpha, dy, g, packed_t=twin if t else None, workspace=ws[1])
        assert torch.equal(dx[:N].cpu(), want)


@pytest.mark.parametrize("contraction", [1056, 1088, 1000, 1032])
def test_infinity_in_the_last_columns_stays_infinite(contraction):
    """Contractions that end inside a K-step (of 64 or of 128 columns): what stands beyond them is zero on both sides, so one
    infinite activation in the last eight columns makes its token's results infinite, not NaN, and no other's."""
    q, T, other, bad = 3, 640, 72 if contraction % 32 else 96, 5
    N, K = (other, contraction) if contraction % 32 == 0 else (contraction, 96)
    gen = torch.Generator().manual_seed(contraction)
    packed = torch.randint(-2**31, 2**31 - 1, (q, N, K // 32), dtype=torch.int32, generator=gen).cuda()
    alpha = (torch.rand((q, N, 1), generator=gen) * torch.tensor([4.0, 2.0, 1.0]).view(q, 1, 1) + 0.01).cuda()
    act = torch.randn((T, contraction), generator=gen).bfloat16().cuda()
    clean = act.clone()
    act[bad, contraction - 3] = float("inf")

    def product(a):
        op = 1 if contraction == K else 2
        ws = torch.empty(bcq.workspace_bytes_grouped(op, T, N, K, K, q, 1), dtype=torch.uint8, device="cuda")
        if op == 1:
            return bcq.bcq_linear_fwd_grouped(packed, alpha, a, K, workspace=ws)
        return bcq.bcq_linear_bwd_input_grouped(packed, alpha, a, K, workspace=ws)

    out, ref = product(act), product(clean)
    assert out[bad].isinf().all()
    keep = torch.arange(T, device="cuda") != bad
    assert torch.equal(out[keep], ref[keep])
