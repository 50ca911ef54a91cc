"""Every tile shape of the large-token product at ragged edges, bit for bit.

Scales of 1 and 1/2 and whole activations make every product a whole number of halves below 2^24, so that any order of the
sums is exact and the only rounding is the one of the stored result.  Rows and columns are no multiple of the tile, with and
without output rows of a multiple of 16 bytes, and the contraction ends inside a K-step of 64 and of 128 columns.  The tile is
chosen by an estimate of the time: the profiler names the kernel that ran, so that a retuned estimate cannot move a case.
"""
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2210_03858_amd as bcq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,T,N", [((64, 64), 389, 200), ((64, 64), 413, 1001), ((64, 128), 389, 2312),
                                      ((64, 128), 413, 2509), ((128, 128), 389, 4616), ((128, 128), 909, 2211),
                                      ((128, 160), 909, 4104), ((128, 160), 1300, 3005), ((256, 128), 909, 5128),
                                      ((256, 128), 1300, 3707), ((256, 160), 2501, 3208), ((256, 160), 3001, 2777),
                                      ((256, 192), 2501, 4008), ((256, 192), 3503, 3005), ((256, 256), 2501, 4808),
                                      ((256, 256), 3503, 3707)])
def test_ragged_tiles_are_exact(tile, T, N):
    K, q = 352, 2
    gen = torch.Generator(device="cuda").manual_seed(T + N)
    packed = torch.randint(-2**31, 2**31 - 1, (q, N, K // 32), dtype=torch.int32, device="cuda", generator=gen)
    alpha = torch.tensor([1.0, 0.5], device="cuda").view(q, 1, 1).expand(q, N, 1).contiguous()
    x = torch.randint(-8, 9, (T, K), device="cuda", generator=gen).bfloat16()
    bits = torch.arange(32, dtype=torch.int32, device="cuda")
    w = sum((2 * ((packed[i].unsqueeze(-1) >> bits) & 1) - 1).reshape(N, K) * alpha[i] for i in range(q))
    want = (x.float() @ w.t()).bfloat16()
    ws = torch.empty(bcq.workspace_bytes_grouped(1, T, N, K, K, q, 1), dtype=torch.uint8, device="cuda")
    y = torch.full((T + 1, N), 77.0, dtype=torch.bfloat16, device="cuda")  # a row behind the result stays as it is
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        bcq.bcq_linear_fwd_grouped(packed, alpha, x, K, y=y[:T], workspace=ws)
        torch.cuda.synchronize()
    names = [e.key for e in prof.key_averages()]
    assert any("gemm_kernel<%d, %d>" % tile in n for n in names), names
    assert torch.equal(y[:T], want)
    assert (y[T] == 77.0).all()
