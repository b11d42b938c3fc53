"""The products on tiles smaller than 256x256: every tile configuration, with the adapter
product as tile columns of its own or riding on the backbone's, and the adapter gradient formed inside the
input-gradient tiles, on exact-integer data (fp32 outputs bit for bit)."""
import pytest

from test_gpu_layer import _exact_integer_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n,m,r", [
    (10, 16, 16, 16),             # one K-step of 16
    (12, 1040, 4112, 64),         # 32-token tiles, K tail
    (32, 128, 2064, 256),         # ... the largest rank in columns of its own, a single K-step
    (33, 896, 272, 48),           # two tile rows, the second with one token; seven K-steps
    (65, 1024, 528, 32),          # eight K-steps (the ring's depth)
    (100, 1152, 144, 96),         # nine
    (256, 640, 512, 16),          # five
    (777, 784, 2000, 48),         # 64 x 128 tiles forward, 64 x 64 backward, ragged everywhere
    (512, 272, 4096, 64),         # 256 tiles: adapter rows ride on two tile columns
    (500, 400, 4112, 256),        # ... on eight, ragged
    (512, 1040, 4000, 80),        # ... on three, the last with 16 ranks
    (1024, 400, 4096, 64),        # 128 x 128 tiles, adapter rows riding
    (1000, 4112, 400, 16),        # 128 x 128 tiles in the input gradient
    (1500, 272, 4112, 128),       # more than one round of tiles
    (9000, 272, 144, 256),        # more than 64 tile rows: the adapter gradient in a launch of its own
])
def test_exact_integer_layer_is_bit_exact(T, n, m, r):
    _exact_integer_layer(T, n, m, r)


@pytest.mark.parametrize("T,n,m,r", [
    (2048, 400, 4096, 64),        # 128-row tiles, exactly one round, one rank block per wave through the LDS
    (2000, 128, 4112, 128),       # ... two rank blocks, ragged, a single K-step
    (1900, 272, 4352, 256),       # ... the largest rank, three K-steps
    (1500, 144, 2560, 256),       # ... four rank blocks per wave, read from memory
    (2000, 400, 4064, 16),        # ... adapter columns inside the last tile column
    (3000, 400, 4080, 48),        # 192-row tiles, ragged tokens and columns
    (2900, 1040, 4096, 32),       # ... two rank blocks
    (1900, 4096, 400, 64),        # input gradient: 128-row tiles, dB over groups of 256 tokens, the last one short
    (2900, 4080, 528, 48),        # ... 192-row tiles, groups of 384 tokens
    (1700, 4352, 272, 128),       # ... rank above the side job's: dB in a launch of its own
])
def test_tiles_of_128_and_192_rows_exact_integer_layer_is_bit_exact(T, n, m, r):
    _exact_integer_layer(T, n, m, r)
