"""Selection of the proxy update, with the requantize in one launch and in two, at the edges of its paths: register counts
(1024, 4096, 11264 and 16384 rows), k on both sides of the limit, long runs of equal scores, scores that share all but a few
neighbouring or separate bits, rows that are nearly alike (with and without a few far larger ones), large rows
that all sit in a few threads, and infinite and zero rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_24061_amd as fq
from gpu_common import layer_on_gpu, np_of

pytestmark = pytest.mark.gpu


def _buffer(kind, m, r, g):
    if kind == "spread":
        return (g.normal(size=(m, r)) * np.exp(1.5 * g.normal(size=(m, 1)))).astype(np.float32)
    buf = np.zeros((m, r), np.float32)
    if kind == "few":                              # fewer rows than k carry anything
        buf[g.choice(m, size=3, replace=False), 0] = [1.0, 2.0, 2.0]
    elif kind == "equal":                          # one value everywhere, a few larger
        buf[:, 1] = 0.5
        buf[g.choice(m, size=5, replace=False), 2] = 1.0
    elif kind == "last bits":                      # scores that share all but their last bits
        buf[:, 0] = 1.0
        buf[:, 1] = (g.integers(0, 4, size=m) * 2.0 ** -50).astype(np.float32)
    elif kind.startswith("bits"):                  # ... that differ in single bits of the fp64 pattern, none adjacent
        buf[:, 0] = 1.0
        for bit in kind.split()[1:]:
            buf[:, 1] += (g.integers(0, 2, size=m) * 2.0 ** (int(bit) - 52)).astype(np.float32)
    elif kind in ("alike", "outliers"):            # as the first step of AdamW leaves them; a few far larger
        buf[:] = 2e-4 * (1.0 + 1e-5 * g.normal(size=(m, r)))
        if kind == "outliers":
            buf[g.choice(m, size=5, replace=False)] *= 1e6
    elif kind == "clustered":                      # all that is large in the first 16 of every 256 rows
        buf[:, 0] = 0.5
        top = np.arange(m) % 256 < 16
        buf[top] = 1.0 + np.abs(g.normal(size=(int(top.sum()), r)))
    elif kind == "infinite":
        buf[:] = g.normal(size=(m, r))
        buf[7, 3] = np.inf
    elif kind == "half infinite":
        buf[:] = g.normal(size=(m, r))
        buf[1::2, 3] = np.inf
    elif kind == "last":                           # the largest at the end
        buf[:] = g.normal(size=(m, r)) + 4.0 * np.arange(m)[:, None] / m
    return buf


@pytest.mark.parametrize("m,k", [(16, 16), (1024, 8), (1040, 96), (4096, 97), (4112, 32), (11264, 64), (11280, 33), (16384, 96),
                                 (16400, 20)])
@pytest.mark.parametrize("kind", ["spread", "few", "equal", "last bits", "bits 2 0", "bits 40 38 31", "alike", "outliers",
                                  "clustered", "infinite", "half infinite"])
def test_rows_and_order_are_the_oracles(m, k, kind):
    n, r = 64, 16
    g = np.random.default_rng(m + k)
    buf = _buffer(kind, m, r, g)
    wcat = oracle.fp8_encode(g.integers(-8, 9, size=(m + r, n)).astype(np.float32), oracle.E4M3)
    layer = layer_on_gpu(4, n, m, r, k, wcat, np.float32(1.0))
    layer.delta_buf.copy_(torch.from_numpy(buf))
    layer.update()
    torch.cuda.synchronize()
    score = np.abs(buf.astype(np.float64)).sum(1)
    want = np.lexsort((np.arange(m), -score))[:k]
    assert np.array_equal(np_of(layer.idx), want)
    left = buf.copy()
    left[want] = 0.0
    assert np.array_equal(np_of(layer.delta_buf), left)
    if "infinite" not in kind:                      # non-finite values: selection and buffer only
        idx_ref, w_ref, buf_ref = oracle.proxy_update(buf, wcat, m, r, k, True)
        assert np.array_equal(idx_ref, want) and np.array_equal(np_of(layer.wq), w_ref)


# one launch up to 256 workgroups of 512, 1024 or 2048 columns and 128 KB of A~ each; beyond, two launches
@pytest.mark.parametrize("m,n,r,k", [(304, 16, 16, 8), (1024, 528, 16, 96), (1040, 512, 48, 32), (96, 4096, 16, 32), (4096, 4112, 64, 28),
                                     (704, 4096, 64, 64), (704, 4096, 64, 65), (512, 13824, 48, 36), (512, 13824, 64, 37), (400, 6160, 128, 40),
                                     (272, 2064, 256, 50), (272, 2064, 256, 52), (272, 4096, 256, 33), (11280, 1040, 32, 9), (96, 8192, 16, 32)])
def test_folded_rows_over_several_workgroups(m, n, r, k):
    g = np.random.default_rng(m + n + r + k)
    wcat = oracle.fp8_encode(g.integers(-8, 9, size=(m + r, n)).astype(np.float32), oracle.E4M3)
    buf = (g.normal(size=(m, r)) * np.exp(1.5 * g.normal(size=(m, 1)))).astype(np.float32)
    layer = layer_on_gpu(4, n, m, r, k, wcat, np.float32(1.0))
    layer.ws.fill_(0x7f)
    w, b = wcat, buf
    for clear in (True, False, True):              # the second update sees what the first one has left
        layer.delta_buf.copy_(torch.from_numpy(b))
        layer.update(clear_selected=clear)
        torch.cuda.synchronize()
        idx_ref, w, left = oracle.proxy_update(b, w, m, r, k, clear)
        assert np.array_equal(np_of(layer.idx), idx_ref)
        assert np.array_equal(np_of(layer.wq), w)
        assert np.array_equal(np_of(layer.delta_buf), left)
        b = np.where(left == 0, np.float32(0.25), left)


# never one launch: 128 KB of A~ have room for 512 columns, of which 96 rows would take 288 workgroups
@pytest.mark.parametrize("m", [112, 272, 1040, 4096, 4112, 11264, 11280, 13824, 16384])
@pytest.mark.parametrize("kind", ["spread", "few", "equal", "last bits", "alike", "outliers", "clustered", "infinite", "half infinite", "last"])
def test_rows_and_order_in_two_launches(m, kind):
    n, r, k = 1040, 256, 96
    g = np.random.default_rng(m + k)
    buf = _buffer(kind, m, r, g)
    wcat = oracle.fp8_encode(g.integers(-8, 9, size=(m + r, n)).astype(np.float32), oracle.E4M3)
    want = np.lexsort((np.arange(m), -oracle.row_scores(buf)))[:k]
    left = buf.copy()
    left[want] = 0.0
    w_ref = None
    if "infinite" not in kind:
        idx_ref, w_ref, _ = oracle.proxy_update(buf, wcat, m, r, k, True)
        assert np.array_equal(idx_ref, want)
    layer = layer_on_gpu(1, n, m, r, k, wcat, np.float32(1.0))
    for static in (False, True):
        layer.wq.copy_(torch.from_numpy(wcat))
        layer.delta_buf.copy_(torch.from_numpy(buf))
        layer.idx.fill_(-1)
        if static:
            fq.proxy_update_static(layer.delta_buf, layer.wq, m, r, k, layer.idx)
        else:
            layer.update()
        torch.cuda.synchronize()
        assert np.array_equal(np_of(layer.idx), want), static
        assert np.array_equal(np_of(layer.delta_buf), left), static
        assert w_ref is None or np.array_equal(np_of(layer.wq), w_ref), static


# up to 512 rows are spread over 128 groups of four threads
@pytest.mark.parametrize("m,k", [(32, 20), (112, 30), (128, 40), (144, 48), (208, 64), (240, 96), (272, 80), (304, 96), (384, 96), (496, 96),
                                 (512, 96), (528, 96)])
@pytest.mark.parametrize("kind", ["spread", "few", "equal", "last bits", "alike", "clustered", "infinite", "half infinite", "last"])
def test_rows_and_order_of_small_buffers(m, k, kind):
    test_rows_and_order_are_the_oracles(m, k, kind)
