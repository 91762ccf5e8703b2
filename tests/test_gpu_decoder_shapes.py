"""The decoder's kernels at the sizes where their tiles, slabs and dispatch change: channel counts up to and
past the 64 the resident-weight convolutions take, image rows up to and past 128 stored pixels, more outputs
of nu than one slab, token counts around the 64-token chunks of the Performer step."""
import pytest

import tests.test_gpu_decoder as base

pytestmark = pytest.mark.gpu

CASES = [
    base._wl("dec_64_channels", 1, 16, 130, 64, 64, 8),
    base._wl("dec_72_channels", 1, 18, 90, 64, 32, 8),
    base._wl("dec_56_channels_bidir", 1, 14, 129, 64, 64, 8, causal=False),
    base._wl("dec_two_slabs", 1, 2, 300, 64, 256, 16),
    base._wl("dec_wide_rows", 1, 2, 520, 64, 512, 8),
    base._wl("dec_odd_columns_bidir_pad", 2, 12, 193, 128, 62, 16, causal=False, pad_frac=0.3),
    base._wl("dec_one_chunk", 2, 4, 64, 128, 32, 8),
    base._wl("dec_one_token_over", 1, 4, 65, 256, 32, 8, causal=False),
    base._wl("dec_segments_pad", 2, 2, 1030, 64, 16, 4, pad_frac=0.4),
]


@pytest.fixture(scope="module")
def sea():
    from paper_2310_01777_amd import binding
    return binding


@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_decoder_sizes(sea, wl):
    base.test_decoder_matches_oracle(sea, wl)
