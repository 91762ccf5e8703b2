"""Causal decoder layers whose three convolutions run in one launch: strips of a multiple of four rows, whose first rows are
computed twice, so lengths around multiples of four, strips of one and of many steps, several sequences per round of blocks,
sequences that end inside a strip, and every number of channels and columns the kernel is built for."""
import pytest

import tests.test_gpu_decoder as base

pytestmark = pytest.mark.gpu

CASES = [
    base._wl("chain_4_heads_64_columns", 1, 4, 64, 64, 64, 8),
    base._wl("chain_4_heads_128_columns", 3, 4, 131, 64, 128, 8, pad_frac=0.4),
    base._wl("chain_8_heads_64_columns", 2, 8, 97, 64, 64, 8, pad_frac=0.4),
    base._wl("chain_8_heads_128_columns", 1, 8, 130, 64, 128, 8),
    base._wl("chain_12_heads_64_columns", 2, 12, 257, 64, 64, 8, pad_frac=0.4),
    base._wl("chain_12_heads_128_columns", 1, 12, 129, 64, 128, 8),
    base._wl("chain_long_strips", 20, 4, 399, 64, 64, 8),
    base._wl("chain_more_sequences_than_blocks", 260, 4, 66, 64, 64, 8, pad_frac=0.3),
]


@pytest.fixture(scope="module")
def sea():
    from paper_2310_01777_amd import binding
    return binding


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_decoder_sizes(sea, wl):
    base.test_decoder_matches_oracle(sea, wl)
