"""The products on tiles smaller than 256x256: every tile configuration, with the adapter
product as tile columns of its own or riding on the backbone's, and the adapter gradient formed inside the
input-gradient tiles, on exact-integer data (fp32 outputs bit for bit)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_24061_amd as fq
from gpu_common import np_of
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
    (9000, 272, 144, 256),        # the adapter gradient in a launch of its own
    (4000, 1024, 512, 256),       # ... beside an input gradient on 128 x 128 tiles, two per CU
    (5000, 144, 1008, 16),        # adapter columns inside the last column of 128 x 128 tiles
    (5000, 4112, 1024, 112),      # two rounds of 128 x 128 tiles, adapter columns of their own inside the second
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
    (1700, 4352, 272, 128),       # ... rank 128: two chunks of ranks per feature step
    (2300, 4096, 400, 208),       # ... four chunks, the last one 16 wide, 256-row tiles
    (1100, 4352, 4240, 256),      # ... four chunks and more feature steps than a workgroup takes: tiles of their own for dB
])
def test_tiles_of_128_and_192_rows_exact_integer_layer_is_bit_exact(T, n, m, r):
    _exact_integer_layer(T, n, m, r)


@pytest.mark.parametrize("T,n,m,r", [
    (20, 8208, 144, 32),          # 32 x 64 tiles, rows one chunk of 16 bytes further into their lines each
    (33, 8288, 272, 48),          # ... six chunks, two tile rows
    (250, 5152, 4000, 64),        # 64 x 64, two chunks
    (512, 1552, 4096, 64),        # 64 x 128, adapter rows riding, one chunk
    (500, 1600, 3984, 48),        # ... four chunks, ragged
    (500, 1648, 4080, 256),       # ... seven chunks, the largest rank
    (1024, 1584, 4000, 96),       # 128 x 128, three chunks
    (1500, 1616, 2000, 16),       # ... five chunks, adapter columns of their own
])
def test_long_rows_across_cache_lines_exact_integer_layer_is_bit_exact(T, n, m, r):
    _exact_integer_layer(T, n, m, r)


@pytest.mark.parametrize("M,N,K,a_at,b_at", [
    (20, 144, 8192, 16, 0),       # rows of whole lines that begin inside one
    (256, 2048, 5120, 0, 112),
    (512, 4096, 1536, 64, 48),
    (1000, 4000, 1552, 96, 32),
    (1, 64, 8200 // 16 * 16, 80, 16),
])
@pytest.mark.parametrize("a_fmt", [fq.E4M3, fq.E5M2])
def test_operands_that_begin_inside_a_cache_line(M, N, K, a_at, b_at, a_fmt):
    """Codes of integers up to 4 in size: sums below 2^24 are exact in fp32 in any order."""
    g = torch.Generator().manual_seed(M + N + K)
    kind = torch.float8_e4m3fn if a_fmt == fq.E4M3 else torch.float8_e5m2
    a = torch.randint(-4, 5, (M, K), generator=g).float()
    b = torch.randint(-4, 5, (N, K), generator=g).float()

    def placed(codes, at):
        buf = torch.full((codes.numel() + at + 16,), 0x7f, dtype=torch.uint8, device="cuda")     # NaN around the operand
        view = buf[at:at + codes.numel()].view(codes.shape)
        view.copy_(codes.view(torch.uint8))
        return view

    one = torch.ones(1, device="cuda")
    c = torch.empty(M, N, device="cuda")
    fq.fp8_gemm(placed(a.to(kind), a_at), a_fmt, placed(b.to(torch.float8_e4m3fn), b_at), False, one, one, c)
    assert torch.equal(c.cpu(), a @ b.T)


@pytest.mark.parametrize("T,n,m,r", [(512, 1024, 1040, 64), (1900, 4096, 8208, 48)])
def test_backward_also_works_in_the_smallest_workspace(T, n, m, r):
    """A workspace without room for the partial sums that the small or 128- and 192-row tiles would leave: the call
    takes the launches that need less.  Same dX; dB up to the order of fp32 sums."""
    g = torch.Generator().manual_seed(T)
    layer = fq.MeldedLinear(T, n, m, r, 8)
    layer.init_weights(torch.randn(m, n, generator=g).cuda() * 0.02, torch.randn(r, n, generator=g).cuda() / r)
    layer.forward(torch.randn(T, n, generator=g).bfloat16().cuda())
    dy = torch.randn(T, m, generator=g).bfloat16().cuda()
    layer.backward(dy, accumulate=False)
    dx, d_b = layer.dx.clone(), layer.d_b.clone()
    lo, hi, full = 0, layer.ws.numel(), layer.ws
    while hi - lo > 256:                           # the smallest workspace that the call accepts
        mid = (lo + hi) // 2 // 256 * 256
        layer.ws = full[:mid]
        try:
            layer.backward(dy, accumulate=False)
            hi = mid
        except fq.FalqonError:
            lo = mid
    assert hi < full.numel()
    layer.ws = torch.empty(hi, dtype=torch.uint8, device="cuda")
    layer.dx.zero_(), layer.d_b.zero_()
    layer.backward(dy, accumulate=False)
    assert torch.equal(layer.dx, dx)
    assert float((layer.d_b - d_b).norm() / d_b.norm()) < 1e-4      # fp32 matrix-core sums: 2e-5 of the result


@pytest.mark.parametrize("M,N,K", [
    (40, 64, 144),                # 32 x 64 tiles
    (500, 1040, 272),             # 64 x 64
    (500, 2064, 272),             # 64 x 128
    (3900, 1008, 144),            # 128 x 128, two workgroups per CU: short K, no room in one round for smaller tiles
    (5990, 784, 400),             # ... more than 256 of them
    (2600, 1040, 6160),           # 128 x 128 on a deep ring: long K
    (2600, 1552, 6160),           # 128 x 256: long K and more than 256 tiles of 128 x 128
])
@pytest.mark.parametrize("kn", [False, True])
@pytest.mark.parametrize("fmt", [fq.E4M3, fq.E5M2])
def test_plain_product_of_integers_is_exact_on_every_kind_of_tile(M, N, K, kn, fmt):
    g = np.random.default_rng(M + N)
    ai, bi = (g.integers(-v, v + 1, size=s).astype(np.float32) for v, s in ((4, (M, K)), (8, (K, N) if kn else (N, K))))
    c = torch.empty(M, N, dtype=torch.float32, device="cuda")
    scale = [torch.tensor([v], device="cuda") for v in (2.0, 0.5)]
    fq.fp8_gemm(torch.from_numpy(oracle.fp8_encode(ai, fmt)).cuda(), fmt, torch.from_numpy(oracle.fp8_encode(bi, fq.E4M3)).cuda(),
                kn, *scale, c)
    want = ai.astype(np.float64) @ (bi if kn else bi.T).astype(np.float64)
    assert np.max(np.abs(want)) < 2.0 ** 24 and np.array_equal(np_of(c).astype(np.float64), want)
