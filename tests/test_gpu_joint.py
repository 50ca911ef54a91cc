"""The training step's joined launches (scales of two tensors in one expansion, the scale gradient's reduction beside the
input gradient's expansion) against the separate entry points, bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


# groups of whole tiles and of 32-column runs, both orders of the expansions' blocks, row counts with and without a twin, more
# than four planes, calls of other kernels (few tokens, rows of no whole 16 bytes, fp32)
@pytest.mark.parametrize("T,N,K,g,q,q_train,dtype", [
    (4096, 1024, 1024, 1024, 4, 1, "bf16"), (1500, 768, 2560, 2560, 3, 2, "bf16"), (2100, 1280, 1280, 256, 2, 1, "bf16"),
    (900, 1000, 1056, 96, 4, 3, "bf16"), (800, 3072, 1024, 64, 2, 1, "bf16"), (770, 2048, 2048, 2048, 1, 1, "bf16"),
    (1030, 520, 544, 32, 3, 1, "bf16"), (1024, 640, 640, 640, 6, 2, "bf16"), (333, 1500, 1056, 1056, 3, 1, "bf16"),
    (100, 512, 512, 128, 3, 1, "bf16"), (20, 256, 512, 512, 2, 1, "bf16"), (3, 96, 128, 64, 4, 2, "bf16"),
    (33, 200, 96, 32, 2, 1, "f32")])
def test_step_equals_separate_calls(T, N, K, g, q, q_train, dtype):
    import torch
    import paper_2210_03858_amd as bcq
    from paper_2210_03858_amd.autograd import BCQLinear
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(T + N)
    layer = BCQLinear.from_weight(torch.randn((N, K), generator=gen, device="cuda"), q, g=g, q_train=q_train, grad_scale=1.0 / g)
    x = torch.randn((T, K), generator=gen, device="cuda").to(dt).requires_grad_(True)
    dy = torch.randn((T, N), generator=gen, device="cuda").to(dt)
    alpha = torch.cat([layer.alpha_train] + ([layer.alpha_frozen] if q_train < q else [])).detach().contiguous()
    packed, twin = layer._layer.packed, layer._layer.twin
    scratch = lambda op: layer._layer.workspace(op, T, bcq.binding.BCQ_BF16 if dtype == "bf16" else bcq.binding.BCQ_F32)
    want = (bcq.bcq_linear_fwd_grouped(packed, alpha, x.detach(), g, workspace=scratch(1)),
            bcq.bcq_linear_bwd_input_grouped(packed, alpha, dy, g, packed_t=twin, workspace=scratch(2)),
            bcq.bcq_linear_bwd_alpha_grouped(packed, x.detach(), dy, g, q_train=q_train, grad_scale=1.0 / g, workspace=scratch(3)))
    y = layer(x)
    both = torch.autograd.grad(y, (x, layer.alpha_train), dy, retain_graph=True)
    only_x, = torch.autograd.grad(y, (x,), dy)
    only_alpha, = torch.autograd.grad(layer(x.detach()), (layer.alpha_train,), dy)
    for got, ref in zip((y.detach(),) + both + (only_x, only_alpha), want + want[1:]):
        assert torch.equal(got, ref)


# unaligned rows, more than four planes, few tokens: nothing is joined, and the second call's scratch may not be held beside the first's
@pytest.mark.parametrize("T,N,K,g,q", [(1500, 5002, 1056, 1056, 3), (2048, 1024, 2048, 2048, 6), (40, 4096, 2048, 128, 2), (3000, 2001, 2048, 64, 4)])
def test_separate_gradients_hold_one_scratch_at_a_time(T, N, K, g, q):
    import torch
    import paper_2210_03858_amd as bcq
    from paper_2210_03858_amd.autograd import BCQLinear
    layer = BCQLinear.from_weight(torch.randn((N, K), device="cuda"), q, g=g)
    x = torch.randn((T, K), device="cuda").bfloat16().requires_grad_(True)
    dy = torch.randn((T, N), device="cuda").bfloat16()
    y = layer(x)
    torch.autograd.grad(y, (x, layer.alpha_train), dy, retain_graph=True)
    sizes = [max(bcq.workspace_bytes_grouped(op, T, N, K, g, q, bcq.binding.BCQ_BF16), 16) for op in (2, 3)]
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    grads = torch.autograd.grad(y, (x, layer.alpha_train), dy)
    peak = torch.cuda.max_memory_allocated() - before
    assert min(sizes) > 1 << 20
    assert peak < max(sizes) + sum(t.numel() * t.element_size() for t in grads) + min(sizes) // 2


# where the scales are joined: by the expansion, by a kernel of its own, or nothing to join; where the scale gradient is reduced: beside the
# expansion, by a kernel of its own, or without partial sums
@pytest.mark.parametrize("T,N,K,g,q,q_train,dtype,join,reduction", [
    (4096, 1024, 1024, 1024, 4, 1, "bf16", "expansion", "expansion"), (2100, 1280, 1280, 256, 2, 1, "bf16", "expansion", "expansion"),
    (900, 1000, 1056, 96, 4, 3, "bf16", "expansion", "expansion"), (770, 2048, 2048, 2048, 1, 1, "bf16", None, "expansion"),
    (1024, 640, 640, 640, 6, 2, "bf16", "expansion", "kernel"), (333, 1500, 1056, 1056, 3, 1, "bf16", "kernel", "kernel"),
    (100, 512, 512, 128, 3, 1, "bf16", "kernel", "expansion"), (3, 96, 128, 64, 4, 2, "bf16", "kernel", "kernel"),
    (20, 256, 512, 512, 2, 1, "bf16", "kernel", "kernel"), (12, 256, 512, 512, 2, 1, "bf16", "kernel", None), (33, 200, 96, 32, 2, 1, "f32", "kernel", None)])
def test_where_scales_are_joined_and_reduced(T, N, K, g, q, q_train, dtype, join, reduction):
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_2210_03858_amd.autograd import BCQLinear
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    layer = BCQLinear.from_weight(torch.randn((N, K), device="cuda"), q, g=g, q_train=q_train)
    x = torch.randn((T, K), device="cuda").to(dt).requires_grad_(True)
    dy = torch.randn((T, N), device="cuda").to(dt)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        torch.autograd.grad(layer(x), (x, layer.alpha_train), dy)
        torch.cuda.synchronize()
    ran = lambda name: any(name in e.key for e in prof.key_averages())
    assert ran("join_scales_kernel") == (join == "kernel")
    assert ran("expand_fwd_kernel") or join != "expansion"
    assert not ran("CatArray")
    assert ran("dalpha_reduce_kernel") == (reduction == "kernel")
    assert ran("expand_bwd_rows_kernel") or reduction != "expansion"
