"""The one-kernel forward above 32 tokens: both tile shapes, the contraction whole and in parts, at ragged edges of rows, tokens
and columns (word counts that are no multiple of 4, a last unit of one word, parts beyond the last column).

Scales of 1, 1/2, .. and whole activations make every product a whole number of eighths below 2^24, so that any order of the sums
is exact and the only rounding is the one of the stored result.  The shape is chosen by an estimate of the time: the profiler
names the kernel that ran.
"""
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2210_03858_amd as bcq

pytestmark = pytest.mark.gpu


def _layer(q, N, K, g, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    packed = torch.randint(-2**31, 2**31 - 1, (q, N, K // 32), dtype=torch.int32, device="cuda", generator=gen)
    alpha = (0.5 ** torch.arange(q, device="cuda", dtype=torch.float32)).view(q, 1, 1).expand(q, N, K // g).contiguous()
    alpha[:, :, 1::2] *= 0.5
    bits = torch.arange(32, dtype=torch.int32, device="cuda")
    w = sum((2 * ((packed[i].unsqueeze(-1) >> bits) & 1) - 1).reshape(N, K) * alpha[i].repeat_interleave(g, dim=1) for i in range(q))
    return packed, alpha, w, gen


def _forward(packed, alpha, x, g):
    q, N, _ = packed.shape
    T, K = x.shape
    ws = torch.empty(bcq.workspace_bytes_grouped(1, T, N, K, g, q, 1), dtype=torch.uint8, device="cuda")
    y = torch.full((T + 1, N), 77.0, dtype=torch.bfloat16, device="cuda")  # a row behind the result stays as it is
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        bcq.bcq_linear_fwd_grouped(packed, alpha, x, g, y=y[:T], workspace=ws)
        torch.cuda.synchronize()
    assert (y[T] == 77.0).all()
    return y[:T], [e.key for e in prof.key_averages()]


@pytest.mark.parametrize("form,parts,T,N,K,g,q", [
    ("4, 1", 1, 96, 4200, 1056, 1056, 3), ("4, 1", 1, 90, 131, 96, 96, 1), ("4, 1", 1, 33, 67, 96, 32, 1), ("4, 1", 1, 97, 8200, 1056, 352, 2), ("4, 1", 1, 333, 1500, 1056, 1056, 3),
    ("4, 1", 5, 130, 1030, 8224, 8224, 3), ("4, 1", 6, 95, 1100, 7424, 7424, 2), ("4, 1", 6, 140, 520, 4128, 32, 2),
    ("4, 1", 3, 400, 1312, 5216, 5216, 1), ("4, 1", 2, 450, 1001, 4128, 96, 1), ("4, 1", 4, 100, 2030, 8224, 32, 4),
    ("8, 2", 1, 110, 8448, 2112, 2112, 2), ("8, 2", 1, 128, 9000, 2080, 2080, 4), ("8, 2", 3, 256, 2557, 10272, 10272, 4)])
def test_tile_forward_exact(form, parts, T, N, K, g, q):
    packed, alpha, w, gen = _layer(q, N, K, g, T + N)
    x = torch.randint(-4, 5, (T, K), device="cuda", generator=gen).bfloat16()
    y, names = _forward(packed, alpha, x, g)
    kernel = "tile_fwd_kernel<%d, %s, %s>" % (q, form, "true" if g != K else "false")
    assert any(kernel in n for n in names), names
    assert any("sum_parts_kernel" in n for n in names) == (parts > 1), names
    assert torch.equal(y, (x.double() @ w.double().t()).float().bfloat16())


@pytest.mark.parametrize("one,T,N,K,g,q", [
    (True, 442, 2723, 1536, 256, 1), (False, 452, 3885, 1152, 128, 1), (True, 720, 1805, 3648, 3648, 1), (False, 481, 1154, 1920, 1920, 2),
    (True, 347, 674, 2112, 96, 2), (False, 274, 863, 2688, 32, 4), (True, 218, 3748, 1792, 64, 4), (False, 137, 5977, 768, 256, 4),
    (True, 342, 5061, 1088, 1088, 4), (False, 354, 3191, 1088, 1088, 4)])
def test_clear_estimates_choose_the_route(one, T, N, K, g, q):
    """Both sides of the two lines in the ratio of the estimated times, with row-wise and group-wise scales."""
    packed, alpha, w, gen = _layer(q, N, K, g, T + N)
    x = torch.randint(-4, 5, (T, K), device="cuda", generator=gen).bfloat16()
    y, names = _forward(packed, alpha, x, g)
    assert any("tile_fwd_kernel" in n for n in names) == one, names
    assert torch.equal(y, (x.double() @ w.double().t()).float().bfloat16())


@pytest.mark.parametrize("T,N,K,q", [(96, 300, 1056, 3), (100, 9000, 2080, 4), (130, 1030, 8224, 3)])
def test_infinity_in_the_last_columns_stays_in_its_token(T, N, K, q):
    packed, alpha, _, gen = _layer(q, N, K, K, N)
    x = torch.randn((T, K), device="cuda", generator=gen).bfloat16()
    clean = _forward(packed, alpha, x, K)[0]
    x[5, K - 3] = float("inf")
    y = _forward(packed, alpha, x, K)[0]
    assert y[5].isinf().all()
    keep = torch.arange(T, device="cuda") != 5
    assert torch.equal(y[keep], clean[keep])
