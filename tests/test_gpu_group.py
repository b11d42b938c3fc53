"""Layers that read one activation: the forward that quantizes it once, and the input gradient added inside the product."""
import pytest
import torch

import paper_2510_24061_amd as fq
from paper_2510_24061_amd import binding as b

pytestmark = pytest.mark.gpu


def _layer(T, n, m, r, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    wq = torch.empty(m + r, n, dtype=torch.uint8, device="cuda")
    s_w, s_tmp = torch.empty(1, device="cuda"), torch.empty(1, device="cuda")
    ws = torch.empty(fq.workspace_bytes(T, n, m, r), dtype=torch.uint8, device="cuda")
    b.quantize(torch.randn(m, n, device="cuda", generator=g).mul_(0.02), b.E4M3, wq[:m], s_w, ws)
    b.quantize(torch.randn(r, n, device="cuda", generator=g) / r, b.E4M3, wq[m:], s_tmp, ws, scale_in=s_w)
    return wq, s_w, ws, g


# the kernels that add, by a trace of this list: small tiles of 32 x 64, 64 x 128 and 128 x 128 with dB inside, of 32 x 64, 64 x 64,
# 64 x 128 and 128 x 128 with dB beside them, of 64 x 128 with dB apart; 128, 192 and 256 rows of 256 columns with dB in the tiles;
# 256 x 256 with dB in workgroups of its own; 128 x 256 and 128 x 128 two to a CU with dB apart; ragged in rows and columns
@pytest.mark.parametrize("T,n,m,r", [(17, 272, 144, 16), (200, 1040, 528, 32), (512, 4096, 1024, 64), (777, 1040, 2000, 48),
                                     (1000, 2064, 512, 256), (1024, 4096, 128, 16), (2048, 4096, 512, 64), (1999, 5120, 400, 32),
                                     (4096, 4112, 272, 64), (4000, 4096, 256, 256), (5000, 1008, 96, 16),
                                     (285, 4736, 1600, 64), (636, 2688, 9168, 256), (3900, 4096, 2048, 64), (2048, 4096, 4240, 256),
                                     (2041, 4112, 9168, 128), (5000, 1008, 4240, 64), (3354, 912, 6096, 128)])
def test_input_gradient_added_in_the_product_is_the_sum_of_the_tensors(T, n, m, r):
    wq, s_w, ws, g = _layer(T, n, m, r, 5)
    dy = torch.randn(T, m, device="cuda", generator=g).mul_(1e-3).to(torch.bfloat16)
    o_a = torch.randn(T, r, device="cuda", generator=g).to(torch.bfloat16)
    amax = o_a.abs().max().float().reshape(1)
    held = torch.randn(T, n, device="cuda", generator=g).mul_(1e-3).to(torch.bfloat16)
    outs = []
    for call, dx in ((b.melded_bwd, torch.empty_like(held)), (b.melded_bwd_add, torch.cat([held, held[:1]])[:T])):
        dyq, s_dy = torch.empty(T, m, dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")
        d_b, buf = torch.empty(m, r, device="cuda"), torch.zeros(m, r, device="cuda")
        print(T, n, m, r, call.__name__, flush=True)
        call(dy, wq, s_w, o_a, amax, n, r, dyq, s_dy, dx, d_b, buf, 0.1, ws)
        outs.append((dx, dyq, s_dy, d_b, buf))
    torch.cuda.synchronize()
    plain, added = outs
    assert torch.equal(added[0], held + plain[0])                       # the same two roundings
    for p, a in zip(plain[1:], added[1:]):
        assert torch.equal(p, a)
    with pytest.raises(TypeError):
        b.melded_bwd_add(dy, wq, s_w, o_a, amax, n, r, dyq, s_dy, added[0].float(), d_b, buf, 0.1, ws)


@pytest.mark.parametrize("T,n,widths,r,dt", [(5, 256, (256, 64, 64), 16, torch.bfloat16), (300, 528, (1040, 272), 48, torch.float32),
                                             (2048, 4096, (4096, 1024, 1024), 64, torch.bfloat16), (700, 1024, (4096,), 128, torch.bfloat16)])
def test_group_forward_equals_the_layers_on_the_same_codes(T, n, widths, r, dt):
    layers = [_layer(T, n, m, r, 10 + i) for i, m in enumerate(widths)]
    x = torch.randn(T, n, device="cuda", generator=layers[0][3]).to(torch.bfloat16)

    def outputs():
        return (torch.empty(T, n, dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda"),
                torch.full((len(widths),), 7e9, device="cuda"), [torch.empty(T, m, dtype=dt, device="cuda") for m in widths],
                [torch.empty(T, r, dtype=torch.bfloat16, device="cuda") for _ in widths])

    xq, s_x, amax, ys, oas = outputs()
    b.quantize(x, b.E4M3, xq, s_x, layers[0][2])
    for i, (wq, s_w, ws, _) in enumerate(layers):
        b.melded_fwd(None, wq, s_w, widths[i], r, xq, s_x, ys[i], oas[i], amax[i:i + 1], ws)
    xq2, s_x2, amax2, ys2, oas2 = outputs()
    b.melded_fwd_group(x, [(wq, s_w, m, r, y, o_a, ws) for (wq, s_w, ws, _), m, y, o_a in zip(layers, widths, ys2, oas2)],
                       xq2, s_x2, amax2)
    torch.cuda.synchronize()
    assert torch.equal(xq, xq2) and torch.equal(s_x, s_x2) and torch.equal(amax, amax2)
    for p, q in zip(ys + oas, ys2 + oas2):
        assert torch.equal(p, q)


def test_group_of_more_layers_than_a_call_takes():
    """Layers beyond the first 256 run on the same codes in calls of their own."""
    from paper_2510_24061_amd.nn import MeldedGroup, MeldedLoRALinear
    T, n, m, r, count = 24, 64, 48, 16, b.GROUP_MAX + 3
    g = torch.Generator(device="cuda").manual_seed(2)
    layers = []
    for _ in range(count):
        layers.append(MeldedLoRALinear(n, m, r, 4))
        layers[-1].load_weights(torch.randn(m, n, device="cuda", generator=g).mul_(0.05), torch.randn(r, n, device="cuda", generator=g) / r)
    x = torch.randn(T, n, device="cuda", generator=g).to(torch.bfloat16)
    one, all_of_them = x.clone().requires_grad_(True), x.clone().requires_grad_(True)
    outs = MeldedGroup(*layers)(all_of_them)
    dys = [torch.randn(T, m, device="cuda", generator=g).mul_(1e-2).to(torch.bfloat16) for _ in range(count)]
    torch.autograd.backward(outs, dys)
    d_bs = [layer.d_b.clone() for layer in layers]
    total = None
    for layer, y, dy, d_b in zip(layers, outs, dys, d_bs):
        one.grad = None
        alone = layer(one)
        alone.backward(dy)
        total = one.grad.clone() if total is None else total.add_(one.grad)
        assert torch.equal(alone, y) and torch.equal(layer.d_b, d_b)
    assert torch.equal(total, all_of_them.grad)
