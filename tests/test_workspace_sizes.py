"""Scratch that the unaligned backward products ask for: bounded by a constant for any number of tokens (host only)."""
import pytest

import paper_2210_03858_amd as bcq


@pytest.mark.parametrize("op", [2, 3])
@pytest.mark.parametrize("T", [4096, 1 << 14, 1 << 17, 1 << 20])
def test_unaligned_backward_scratch_is_bounded(op, T):
    """A 50257-row output layer: 1.6 GB for the input gradient (4096 tokens and the weights in three bf16 terms each), 512 MiB
    and 1 % of dy's size in partial sums for the scale gradient."""
    need = bcq.workspace_bytes_grouped(op, T, 50257, 1024, 1024, 3, 1)
    assert need <= (1.6e9 if op == 2 else (1 << 29) + 2e7 + 0.01 * 2 * T * 50257)
