"""Forward of up to 16 tokens in one launch: every split of its workgroups (16 to 64 columns, two to eight shares of the
K-steps), ragged tokens, columns and K, ranks up to 64 in it and beyond it, on exact-integer data (fp32 outputs bit for
bit) and against the same call on codes quantized beforehand, which takes other launches."""
import pytest
import torch

import paper_2510_24061_amd as fq
from gpu_common import relf, np_of
from test_gpu_layer import _exact_integer_layer

pytestmark = pytest.mark.gpu

SHAPES = [(1, 16, 16, 16), (1, 4096, 4096, 64), (2, 144, 272, 48), (7, 1040, 4080, 64), (8, 2064, 4096, 16), (8, 4096, 528, 64),
          (15, 2064, 8160, 32), (16, 2048, 8176, 64), (9, 2048, 12240, 64), (3, 272, 12256, 48), (10, 3264, 144, 64), (13, 400, 16400, 16),
          (17, 400, 528, 64), (7, 4112, 144, 32), (5, 1024, 1040, 80)]


@pytest.mark.parametrize("T,n,m,r", [s for s in SHAPES if s[0] >= 10] + [(10, 16, 16, 16), (10, 3008, 4080, 64), (12, 272, 12256, 48)])
def test_exact_integer_layer_is_bit_exact(T, n, m, r):
    _exact_integer_layer(T, n, m, r)


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,n,m,r", SHAPES[:12])
def test_matches_the_call_on_quantized_input(T, n, m, r, out_dtype):
    g = torch.Generator().manual_seed(T + n)
    layer = fq.MeldedLinear(T, n, m, r, 8, out_dtype=out_dtype)
    layer.init_weights((torch.randn(m, n, generator=g) * 0.02).cuda(), (torch.randn(r, n, generator=g) / r).cuda())
    x = torch.randn(T, n, generator=g).to(torch.bfloat16)
    x[T - 1, n - 1] = -9.0
    for b in (layer.y, layer.o_a):
        b.fill_(7.0)
    layer.forward(x.cuda())
    y, o_a, amax = layer.y.clone(), layer.o_a.clone(), layer.amax_oa.clone()
    xq, s = torch.empty_like(layer.xq), torch.zeros(1, device="cuda")
    fq.quantize(x.cuda(), fq.E4M3, xq, s, layer.ws)
    torch.cuda.synchronize()
    assert torch.equal(xq, layer.xq) and torch.equal(s, layer.s_x)                # bit for bit the quantizer's
    assert float(amax) == float(o_a.float().abs().max())
    fq.melded_fwd(None, layer.wq, layer.s_w, m, r, xq, s, layer.y, layer.o_a, layer.amax_oa, layer.ws)
    torch.cuda.synchronize()
    # sums in another order: fp32 rounding of up to n terms, or half a unit of bf16 on either side of a tie
    assert relf(np_of(y), np_of(layer.y)) <= (1e-5 if out_dtype == torch.float32 else 1e-3)
    assert relf(np_of(o_a), np_of(layer.o_a)) <= 1e-3


def _bits(x, values):
    """x (bf16) with the given positions set to the given bit patterns"""
    u = x.view(torch.int16)
    for (t, j), b in values.items():
        u[t, j] = b - 65536 if b > 32767 else b
    return x


# A maximum is that of the values that are not NaN, as in the quantizer; positions beside and far from one another, so
# that values of one thread and of several are concerned
@pytest.mark.parametrize("name", ["beside the largest", "a token", "all", "infinite", "infinite and NaN", "smallest NaNs", "zeros and NaN"])
@pytest.mark.parametrize("T,n,m,r", [(8, 4096, 272, 64), (1, 4096, 144, 16), (5, 272, 528, 48), (16, 2048, 400, 64), (16, 16, 16, 16)])
def test_not_finite_inputs_have_the_quantizers_codes(T, n, m, r, name):
    g = torch.Generator().manual_seed(T + n)
    layer = fq.MeldedLinear(T, n, m, r, 8)
    layer.init_weights((torch.randn(m, n, generator=g) * 0.02).cuda(), (torch.randn(r, n, generator=g) / r).cuda())
    x = torch.full((T, n), 0.5).to(torch.bfloat16) if name == "beside the largest" else torch.randn(T, n, generator=g).to(torch.bfloat16)
    at, other = (T - 1, n - 12), (0, 3)
    bad = set()
    if name == "beside the largest":
        x[at[0], at[1] + 2] = 50.0
        _bits(x, {at: 0x7fc0, (at[0], at[1] + 3): 0xffc0})
        bad = {T - 1}
    elif name == "a token":
        _bits(x, {(T - 1, j): 0x7fc0 for j in range(n)})
        bad = {T - 1}
    elif name == "all":
        x.fill_(float("nan"))
        bad = set(range(T))
    elif name == "infinite":
        x[at], x[other] = float("inf"), float("-inf")
    elif name == "infinite and NaN":
        _bits(x, {at: 0x7f80, other: 0x7fff, (0, 4): 0xff80})
    elif name == "smallest NaNs":
        _bits(x, {at: 0x7f81, other: 0xff81})
        bad = {T - 1, 0}
    else:
        x.zero_()
        _bits(x, {other: 0x7fc0, at: 0x8000})
        bad = {0}
    for b in (layer.y, layer.o_a):
        b.fill_(7.0)
    layer.forward(x.cuda())
    xq, s = torch.empty_like(layer.xq), torch.zeros(1, device="cuda")
    fq.quantize(x.cuda(), fq.E4M3, xq, s, layer.ws)
    torch.cuda.synchronize()
    assert torch.equal(s, layer.s_x) and torch.equal(xq, layer.xq)
    if "infinite" in name:
        return                                                                    # (a scale of zero)
    y, o_a = layer.y.clone(), layer.o_a.clone()
    fq.melded_fwd(None, layer.wq, layer.s_w, m, r, xq, s, layer.y, layer.o_a, layer.amax_oa, layer.ws)
    torch.cuda.synchronize()
    rows = [t for t in range(T) if t not in bad]                                  # the other tokens are what they were
    assert relf(np_of(y)[rows], np_of(layer.y)[rows]) <= 1e-3 and relf(np_of(o_a)[rows], np_of(layer.o_a)[rows]) <= 1e-3


@pytest.mark.parametrize("T,n,m", [(8, 4096, 4096), (16, 256, 32000), (3, 1008, 20000), (1, 4096, 8192)])
def test_outputs_may_lie_over_the_input(T, n, m):
    """The input is read by the quantizer alone, before anything else is written: y, or O_A, may take its memory."""
    r, g = 64, torch.Generator().manual_seed(T)
    layer = fq.MeldedLinear(T, n, m, r, 8)
    layer.init_weights((torch.randn(m, n, generator=g) * 0.02).cuda(), (torch.randn(r, n, generator=g) / r).cuda())
    x = torch.randn(T, n, generator=g).to(torch.bfloat16)
    memory = torch.empty(T * (n + m), dtype=torch.bfloat16, device="cuda")
    for first, o_a in [(0, layer.o_a), (T * n // 2 // 8 * 8, layer.o_a), (T * n, memory[:T * r].view(T, r))]:
        memory.fill_(3.0)
        memory[:T * n] = x.flatten().cuda()
        xin, y = memory[:T * n].view(T, n), memory[first:first + T * m].view(T, m)
        fq.melded_fwd(xin, layer.wq, layer.s_w, m, r, layer.xq, layer.s_x, y, o_a, layer.amax_oa, layer.ws)
        torch.cuda.synchronize()
        y, o_a = y.clone(), o_a.clone()
        fq.quantize(x.cuda(), fq.E4M3, layer.xq, layer.s_x, layer.ws)
        fq.melded_fwd(None, layer.wq, layer.s_w, m, r, layer.xq, layer.s_x, layer.y, layer.o_a, layer.amax_oa, layer.ws)
        torch.cuda.synchronize()
        assert relf(np_of(y), np_of(layer.y)) <= 1e-3 and relf(np_of(o_a), np_of(layer.o_a)) <= 1e-3, first


# one round of workgroups of 64 columns, two up to n = 1024, and the first sizes beyond
@pytest.mark.parametrize("T,n,m,r", [(2, 4096, 16320, 64), (2, 4096, 16336, 64), (3, 1040, 16336, 16), (16, 1024, 32704, 64), (5, 1024, 32720, 48)])
def test_at_the_most_columns(T, n, m, r):
    test_matches_the_call_on_quantized_input(T, n, m, r, torch.bfloat16)
