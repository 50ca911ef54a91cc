"""The any-shape kernels (fp64; fp32 activations, or bf16 without a workspace) at the edges of their tiles.

All sums are fp64, so a result differs from the oracle's fp64 value by its own rounding: half a unit in
the last place, 2^-24 of the value for fp32 outputs (24 significant bits) and 2^-8 for bf16 ones (8 significant bits;
they are rounded to fp32 first, hence the 1 %); the normalised error divides by the largest value, which
can only make it smaller."""
import pytest

from _util import make_case, nmax_err, packed_to_dev, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = {"f32": 1.05 * 2.0 ** -24, "bf16": 1.01 * 2.0 ** -8}

# T, N, K, g, q, q_train
EDGES = [
    (1, 1, 32, 32, 1, 1),          # smallest of everything: seven of eight waves without work
    (15, 17, 96, 32, 8, 5),        # one row beyond a tile, three groups
    (16, 16, 256, 256, 2, 2),      # whole tiles, one word per wave
    (17, 31, 288, 96, 3, 3),       # nine words over eight waves, groups of three words
    (32, 1001, 512, 32, 4, 4),     # more groups (16) than waves, odd row count
    (33, 33, 1056, 352, 3, 1),     # groups over two waves each
    (100, 1100, 64, 64, 3, 3),     # two token tiles per workgroup in the forward
    (130, 4100, 32, 32, 2, 1),     # four token tiles per workgroup in the forward
    (70, 40, 3072, 3072, 1, 1),    # two token tiles x a whole word in the input gradient
    (8, 72, 2560, 64, 4, 2),       # forty groups, one wave each
]
# Few tokens or rows: the vector ALU forms
FEW = [
    (1, 5, 384, 384, 8, 8),        # twelve words; the last workgroup's waves without a row
    (4, 1499, 2080, 2080, 2, 2),   # a wave per row, 65 words; scale gradient on the matrix cores
    (2, 6, 16384, 2048, 3, 3),     # four waves per row, eight groups
    (5, 1000, 4128, 96, 5, 3),     # a second, ragged token tile
    (8, 600, 1056, 1056, 4, 1),    # scale gradient of eight tokens
    (3, 10000, 2048, 512, 8, 8),   # all of eight planes, groups too short for the row form of the scale gradient
    (1, 9999, 800, 32, 3, 2),
    (2, 700, 512, 512, 3, 3),      # the longest calls that rows of 16 words take
    (8, 500, 1056, 1056, 2, 2),    # two whole token tiles
    (1, 5, 352, 352, 3, 3),        # too short for the row forms
    (700, 7, 1056, 352, 4, 4),     # input gradient by columns, ragged last tile of tokens and of columns
    (2100, 33, 4096, 4096, 1, 1),
    (70, 1, 544, 32, 2, 2),
    (333, 16, 4096, 128, 8, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,N,K,g,q,q_train", EDGES + FEW)
def test_generic_kernels_are_correctly_rounded(oracle, dtype, T, N, K, g, q, q_train):
    import torch
    import paper_2210_03858_amd as bcq
    _, alpha, planes, packed, x, dy = make_case(1, "out", T, N, K, q, dtype, oracle, extra=T + N, g=g)
    d_packed, d_alpha = packed_to_dev(packed), to_dev(alpha.reshape(q, N, K // g))
    d_x, d_dy = to_dev(x, dtype), to_dev(dy, dtype)
    rowwise_small = dtype == "bf16" and g == K and T < 32  # kernels of their own without a workspace
    a_or = alpha.reshape(q, N) if g == K else alpha
    dx = bcq.bcq_linear_bwd_input_grouped(d_packed, d_alpha, d_dy, g)
    assert nmax_err(to_host(dx), oracle.bwd_input(a_or, planes, dy)) <= TOL[dtype]
    if not rowwise_small:
        y = bcq.bcq_linear_fwd_grouped(d_packed, d_alpha, d_x, g)
        da = bcq.bcq_linear_bwd_alpha_grouped(d_packed, d_x, d_dy, g, q_train=q_train)
        assert nmax_err(to_host(y), oracle.fwd(a_or, planes, x)) <= TOL[dtype]
        ref = oracle.bwd_alpha(planes, x, dy, q_train=q_train, grad_scale=1.0, g=g)
        assert nmax_err(to_host(da).reshape(ref.shape), ref) <= TOL["f32"]
    torch.cuda.synchronize()
