"""The forward of at most 8 tokens in one kernel, from both plane layouts, at the edges of its tiles: row counts of less than a
tile and beyond one, word counts that are no multiple of 4 or 16, one to several segments per wave, row tiles shared by two and three
to a workgroup, groups of one and more segments.

Signs and scales are exact and the activations are bf16 within 2^-13 of their block's largest, so only the fp32 sums and the one
rounding of the result (2^-9 of its value) differ from fp64: 2^-8 of every value and 1e-5 of the largest.  The profiler names the
kernel that ran.
"""
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import paper_2210_03858_amd as bcq

pytestmark = pytest.mark.gpu


def _layer(q, N, K, g, T, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    packed = torch.randint(-2**31, 2**31 - 1, (q, N, K // 32), dtype=torch.int32, device="cuda", generator=gen)
    alpha = torch.rand((q, N, K // g), device="cuda", generator=gen) + 0.1
    x = torch.randn((T, K), device="cuda", generator=gen).bfloat16()
    bits = torch.arange(32, dtype=torch.int32, device="cuda")
    w = sum((2 * ((packed[i].unsqueeze(-1) >> bits) & 1) - 1).reshape(N, K).double() * alpha[i].double().repeat_interleave(g, dim=1)
            for i in range(q))
    return packed, alpha, x, w


def _run(layout, packed, alpha, x, g, kernel="few_fwd_kernel"):
    q, N, _ = packed.shape
    T, K = x.shape
    ws = torch.empty(max(16, bcq.workspace_bytes_grouped(1, T, N, K, g, q, 1)), dtype=torch.uint8, device="cuda")
    y = torch.full((T + 1, N), 77.0, dtype=torch.bfloat16, device="cuda")  # a row behind the result stays as it is
    planes = bcq.bcq_pack_decode(packed) if layout == "decode" else packed
    call = bcq.bcq_linear_fwd_decode if layout == "decode" else bcq.bcq_linear_fwd_grouped
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call(planes, alpha, x, g, y=y[:T], workspace=ws)
        torch.cuda.synchronize()
    assert any(kernel in e.key for e in prof.key_averages())
    assert (y[T] == 77.0).all()
    return y[:T]


@pytest.mark.parametrize("layout,T,N,K,g,q", [
    ("decode", 1, 1024, 1024, 1024, 3), ("decode", 8, 33, 32, 32, 1), ("decode", 5, 1000, 1056, 1056, 4), ("decode", 3, 8208, 544, 544, 2),
    ("decode", 8, 8209, 2528, 2528, 4), ("decode", 2, 200, 12288, 12288, 1), ("decode", 4, 100, 8192, 8192, 3), ("decode", 8, 70, 4096, 4096, 2),
    ("decode", 8, 300, 2048, 512, 4), ("decode", 1, 300, 1536, 512, 3), ("canonical", 1, 1, 160, 160, 2), ("canonical", 7, 5000, 1056, 1056, 2),
    ("canonical", 6, 131, 3104, 3104, 3), ("canonical", 4, 2048, 2048, 512, 3), ("canonical", 1, 35, 1536, 512, 4), ("canonical", 8, 2100, 2560, 512, 1),
    ("canonical", 3, 4200, 1024, 512, 4), ("canonical", 2, 17, 3072, 1536, 2), ("canonical", 8, 8300, 1536, 512, 1), ("canonical", 4, 40, 6144, 512, 1),
    ("canonical", 5, 4100, 2048, 1024, 3), ("canonical", 2, 64, 1024, 512, 4)])
def test_few_tokens_in_one_kernel(layout, T, N, K, g, q):
    packed, alpha, x, w = _layer(q, N, K, g, T, T + N + K)
    y = _run(layout, packed, alpha, x, g).double()
    ref = x.double() @ w.t()
    assert ((y - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max()).all()


@pytest.mark.parametrize("layout,T,N,K,g,q", [
    ("decode", 1, 40, 7168, 7168, 4), ("decode", 1, 40, 7200, 7200, 3), ("decode", 2, 4096, 7712, 7712, 4), ("decode", 2, 4112, 7712, 7712, 4),
    ("decode", 4, 100, 8192, 512, 4), ("canonical", 1, 4112, 4608, 512, 2), ("canonical", 2, 4080, 4608, 512, 1)])
def test_up_to_sixteen_segments_at_a_time(layout, T, N, K, g, q):
    """Both sides of the lines between 8 and 16 waves, and the largest workgroup."""
    test_few_tokens_in_one_kernel(layout, T, N, K, g, q)


@pytest.mark.parametrize("layout,T,N,K,g,q", [("decode", 8, 600, 1056, 1056, 3), ("canonical", 5, 4200, 1024, 512, 2), ("canonical", 4, 100, 1536, 512, 4)])
def test_non_finite_token_and_zero_blocks(layout, T, N, K, g, q):
    """A non-finite activation makes its own token's results NaN; blocks of zeros, a block of subnormals and one of large values
    re-code exactly."""
    packed, alpha, x, w = _layer(q, N, K, g, T, N)
    x[0, 32:64], x[1, 64:96], x[2, :32] = 0.0, 1e-39, 2.0 ** 100
    clean = _run(layout, packed, alpha, x, g)
    ref = x.double() @ w.t()
    assert ((clean.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max(dim=1, keepdim=True).values).all()
    x[3, 5], x[3, K - 1] = float("inf"), float("nan")
    y = _run(layout, packed, alpha, x, g)
    assert y[3].isnan().all()
    keep = torch.arange(T, device="cuda") != 3
    assert torch.equal(y[keep], clean[keep])


@pytest.mark.parametrize("layout,T,N,K,g,q", [
    ("decode", 7, 8208, 2048, 2048, 3), ("decode", 7, 12288, 1312, 1312, 3), ("decode", 8, 12304, 2048, 2048, 1), ("canonical", 6, 7150, 4096, 4096, 1),
    ("canonical", 5, 4096, 4096, 4096, 1), ("canonical", 8, 600, 3584, 512, 4), ("canonical", 6, 2032, 4096, 512, 4)])
def test_row_tiles_that_share(layout, T, N, K, g, q):
    """Both sides of the lines between one, two and three row tiles to a workgroup, and groups of one segment beyond the line of the others."""
    test_few_tokens_in_one_kernel(layout, T, N, K, g, q)


@pytest.mark.parametrize("layout,T,N,K,g,q", [
    ("canonical", 6, 9822, 3072, 1536, 4), ("decode", 6, 8208, 3072, 3072, 3), ("canonical", 3, 300, 7168, 7168, 4), ("canonical", 2, 40, 8192, 1024, 3),
    ("canonical", 8, 300, 3072, 1536, 4), ("decode", 3, 164, 9216, 1536, 2), ("decode", 8, 80, 3584, 512, 1)])
def test_beyond_the_lines_two_kernels_run(layout, T, N, K, g, q):
    """Calls of which this kernel would take more than one round, or whose contraction is too long for it: same bound."""
    packed, alpha, x, w = _layer(q, N, K, g, T, T + N + K)
    y = _run(layout, packed, alpha, x, g, kernel="stream_kernel").double()
    ref = x.double() @ w.t()
    assert ((y - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max()).all()


@pytest.mark.parametrize("layout,T,N,K,g,q,kernel", [("decode", 4, 100, 1056, 1056, 3, "few_fwd_kernel"), ("canonical", 4, 40, 2048, 1024, 2, "few_fwd_kernel"),
                                                     ("canonical", 4, 300, 9216, 9216, 2, "stream_kernel"), ("canonical", 4, 70, 640, 640, 6, "stream_fused_kernel")])
def test_largest_magnitudes(layout, T, N, K, g, q, kernel):
    """1.75 x 2^127 is multiplied like any other activation; from 3.0e38 on a token counts as non-finite, and no other token does."""
    packed, alpha, x, w = _layer(q, N, K, g, T, N)
    alpha, w = alpha * 2.0 ** -10, w * 2.0 ** -10
    x[1, 7], x[2, 9] = 1.75 * 2.0 ** 127, 3.2e38
    y = _run(layout, packed, alpha, x, g, kernel=kernel).double()
    ref = x.double() @ w.t()
    ok = torch.tensor([0, 1, 3], device="cuda")
    assert ((y - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max(dim=1, keepdim=True).values)[ok].all()
    assert y[2].isnan().all()
