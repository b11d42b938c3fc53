"""The adapter gradient on workgroups of its own beside small input-gradient tiles, and inside the tiles where these leave no
CU for it, on exact-integer data (fp32 outputs bit for bit)."""
import pytest

from test_gpu_layer import _exact_integer_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n,m,r", [
    (17, 272, 1040, 16),          # 32 x 64 tiles; fewer tokens than one step of the gradient's tiles
    (129, 304, 2064, 256),        # ... four rank tiles, ragged features, one token in the second step
    (200, 1040, 3984, 48),        # 64-row tiles
    (513, 272, 4112, 96),         # a second group of tokens with one of them
    (777, 1040, 2000, 48),
    (700, 1296, 528, 128),        # two splits of the tokens
    (2298, 640, 464, 96),         # several, ragged
    (3898, 736, 416, 64),         # 128 x 128 tiles, many splits
    (2500, 368, 144, 208),        # the last rank tile 16 wide
    (500, 4080, 1040, 48),        # inside: every CU has a tile
    (60, 8208, 400, 256),         # ... 32 x 64 tiles, more than one round
])
def test_exact_integer_layer_is_bit_exact(T, n, m, r):
    print(T, n, m, r, flush=True)
    _exact_integer_layer(T, n, m, r)
