"""Decode-layout forward around the limits of its single-kernel form (one segment per wave, at most four segments, 256
row tiles and 8 tokens; three segments for group-wise scales of three planes and five tokens on, one, row-wise, for more
than four planes), against the oracle at the suite's bf16 tolerance."""
import pytest

from _util import TOL_BF16, make_case, nmax_err, packed_to_dev, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,K,g,q", [(1, 1, 32, 32, 1), (8, 17, 512, 512, 3), (5, 4096, 544, 544, 2),
                                       (8, 4097, 512, 512, 4), (2, 300, 2048, 2048, 8), (3, 100, 2080, 2080, 3),
                                       (9, 64, 1024, 1024, 3), (4, 50, 2048, 512, 4), (7, 33, 1536, 768 * 2, 5),
                                       (3, 48, 480, 480, 6), (8, 20, 512, 512, 8), (8, 33, 1536, 512, 4), (5, 40, 2048, 512, 3),
                                       (2, 24, 1024, 512, 7)])
def test_decode_forward(oracle, T, N, K, g, q):
    import torch
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, _ = make_case(3, "out", T, N, K, q, "bf16", oracle, extra=N, g=g)
    tiled = bcq.bcq_pack_decode(packed_to_dev(packed))
    ws = torch.empty((max(bcq.workspace_bytes_grouped(1, T, N, K, g, q, 1), 16),), dtype=torch.uint8, device="cuda")
    y = bcq.bcq_linear_fwd_decode(tiled, to_dev(alpha.reshape(q, N, K // g)), to_dev(x, "bf16"), g, workspace=ws)
    ref = oracle.fwd(alpha.reshape(q, N) if g == K else alpha, planes, x)
    assert nmax_err(to_host(y), ref) <= TOL_BF16
