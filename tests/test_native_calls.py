"""The extension that takes a step's calls refuses what the binding has always refused, before anything is launched (this
machine may have no GPU)."""
import pytest
import torch

from paper_2510_24061_amd import binding as b


@pytest.fixture(autouse=True)
def _no_device(monkeypatch):
    monkeypatch.setattr(b, "_stream", lambda: 0)


def test_tensors_off_the_gpu_are_refused():
    t = torch.zeros(16, 16)
    with pytest.raises(ValueError, match="contiguous GPU"):
        b.melded_fwd(t, t, t, 16, 16, t, t, t, t, t, t)
    with pytest.raises(ValueError, match="contiguous GPU"):
        b.melded_bwd(t, t, t, t, t, 16, 16, t, t, None, t, None, 0.1, t)
    with pytest.raises(ValueError, match="contiguous GPU"):
        b.melded_bwd_add(t, t, t, t, t, 16, 16, t, t, t.to(torch.bfloat16), t, None, 0.1, t)
    with pytest.raises(ValueError, match="contiguous GPU"):
        b.proxy_update(t, t, 16, 16, 4, t, t)
    with pytest.raises(ValueError, match="contiguous GPU"):
        b.grad_sqnorm(t, t, t)
    with pytest.raises(ValueError, match="contiguous GPU"):
        b.adamw_delta(t, t, t, t, 1)


def test_what_is_no_tensor_and_what_has_no_shape():
    n = b._native()
    with pytest.raises(TypeError):
        n.grad_sqnorm([1.0], None, None, 0)
    with pytest.raises(TypeError):
        n.grad_sqnorm(None, None)                                     # too few
    with pytest.raises(AttributeError):
        b.proxy_update(None, None, 16, 16, 4, None, None)
    with pytest.raises(AttributeError):
        b.grad_sqnorm(None, None, None)
    with pytest.raises(TypeError):
        b.workspace_bytes(16, 64.5, 64, 16)
    with pytest.raises(OverflowError):
        b.workspace_bytes(16, 1 << 70, 64, 16)
    assert b.workspace_bytes(16, 64, 64, 16) == b.lib().falqon_workspace_bytes(16, 64, 64, 16) > 0


def test_rates_are_what_float_takes(monkeypatch):
    """A rate read from a file of settings may be text ("2e-4" is a string to YAML)."""
    rates = []

    class Calls:
        @staticmethod
        def melded_bwd(*args):
            rates.append(args[12])
            return 0
        melded_bwd_add = melded_bwd

    monkeypatch.setattr(b, "_native", lambda: Calls)
    t = [None] * 5
    b.melded_bwd(*t, 16, 16, None, None, None, None, None, "2e-4", None)
    b.melded_bwd_add(*t, 16, 16, None, None, None, None, None, torch.tensor(0.5), None)
    assert rates == [2e-4, 0.5] and all(type(r) is float for r in rates)


@pytest.mark.gpu
def test_update_takes_the_width_of_a_weight_of_more_dimensions():
    m, r, n, k = 32, 16, 64, 4
    buf = torch.randn(m, r, device="cuda", generator=torch.Generator(device="cuda").manual_seed(0))
    outs = []
    for shape in [(m + r, n), (m + r, n, 1)]:
        wq = torch.full(shape, 0x30, dtype=torch.uint8, device="cuda")
        idx = torch.empty(k, dtype=torch.int32, device="cuda")
        ws = torch.empty(b.workspace_bytes(16, n, m, r), dtype=torch.uint8, device="cuda")
        b.proxy_update(buf.clone(), wq, m, r, k, idx, ws)
        torch.cuda.synchronize()
        outs.append((wq.reshape(m + r, n), idx))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    with pytest.raises(ValueError):
        b.proxy_update(buf, wq.reshape(-1), m, r, k, idx, ws)
