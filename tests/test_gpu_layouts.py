"""Transposed twin and decode layout around the tile and grid limits of their kernels, bit for bit against numpy."""
import numpy as np
import pytest

from _util import decode_layout, packed_to_dev, packed_to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,N,K", [(1, 32, 32), (3, 288, 256), (2, 256, 288), (1, 4096, 8224), (4, 2080, 4096),
                                   (8, 33 * 32, 1056), (1, 17, 2080), (2, 5, 16384), (2, 64, 512), (3, 65, 32),
                                   (1, 33, 544), (2, 47, 1024), (8, 31, 96)])
def test_twin_and_decode_layout(q, N, K):
    import paper_2210_03858_amd as bcq
    rng = np.random.default_rng(N + K)
    packed = rng.integers(0, 2 ** 32, (q, N, K // 32), dtype=np.uint32)
    dev = packed_to_dev(packed)
    assert np.array_equal(packed_to_host(bcq.bcq_pack_decode(dev)), decode_layout(packed))
    if N % 32 == 0:
        bits = np.unpackbits(packed.view(np.uint8), axis=2, bitorder="little")           # [q][N][K]
        twin = np.packbits(bits.transpose(0, 2, 1).copy(), axis=2, bitorder="little").view(np.uint32)
        assert np.array_equal(packed_to_host(bcq.bcq_pack_transposed(dev)), twin)


@pytest.mark.parametrize("q,N,K", [(1, 128, 32), (3, 512, 512), (5, 640, 544), (2, 544, 1056), (7, 1152, 480), (1, 32, 16384),
                                   (2, 16384, 32)])
def test_twin_and_decode_layout_around_one_tile(q, N, K):
    """Tiles of 16 x 16 words, whole and in part, rows of packed_t of whole 16-byte units and others, odd plane counts."""
    test_twin_and_decode_layout(q, N, K)
