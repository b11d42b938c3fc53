"""GPU parity of the initialization steps against the CPU oracle.

The residual is bit-exact.  The rank-r factor is the result of an iteration whose limit (the
truncated SVD) is unique only as a subspace and only up to the sign of each vector, so what is
compared is what is unique: the projector on the row space, the singular values and the energy
captured, with the exact SVD of the oracle as reference; what is not unique is checked for
validity (orthogonal rows, squared norms equal to the Ritz values, Ritz values = |E v|).

Tolerances.  With a spectral gap the subspace iteration converges at (sigma_{l+1}/sigma_r)^(2q+1);
the planted cases have a gap of 10^2 or more, so after q = 3 rounds what remains is fp32 rounding
of products over n terms: 1e-4 on projector and singular values.  Quantization residuals have no
gap; there the r Ritz values must capture at least 90 % of the energy of the best rank-r factor."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_24061_amd as fq
from gpu_common import np_of

pytestmark = pytest.mark.gpu


def _factor(e: np.ndarray, r: int, iters: int, seed: int = 0):
    m, n = e.shape
    g = torch.Generator().manual_seed(seed)
    omega = torch.randn(r + 8, n, generator=g).cuda()
    a = torch.empty(r, n, dtype=torch.float32, device="cuda")
    sig = torch.empty(r, dtype=torch.float32, device="cuda")
    ws = torch.empty(fq.svd_workspace_bytes(m, n, r), dtype=torch.uint8, device="cuda")
    fq.svd_right_factor(torch.from_numpy(e).cuda(), r, omega, iters, a, sig, ws)
    torch.cuda.synchronize()
    return np_of(a).astype(np.float64), np_of(sig).astype(np.float64)


def _projector(a):
    q, _ = np.linalg.qr(a.T)
    return q @ q.T


@pytest.mark.parametrize("m,n", [(64, 128), (300, 400), (1000, 520), (4096, 1024)])
def test_residual_bit_exact(m, n):
    w = (np.random.default_rng(m).normal(size=(m, n)) * 0.02).astype(np.float32)
    w[0, :4] = [0.0, -0.0, 1e-9, 0.09]
    wq, s_w, _ = oracle.quantize(w, oracle.E4M3)
    ref = oracle.init_residual(w, wq, s_w)
    e = torch.empty(m, n, dtype=torch.float32, device="cuda")
    fq.init_residual(torch.from_numpy(w).cuda(), torch.from_numpy(wq).cuda(), torch.tensor([s_w], device="cuda"), e)
    torch.cuda.synchronize()
    assert np_of(e).tobytes() == ref.tobytes()


@pytest.mark.parametrize("m,n,r", [(300, 400, 16), (520, 272, 24), (1024, 2048, 64), (200, 1000, 120)])
def test_factor_of_a_matrix_with_a_spectral_gap(m, n, r):
    g = np.random.default_rng(m + n)
    u, _ = np.linalg.qr(g.normal(size=(m, r)))
    v, _ = np.linalg.qr(g.normal(size=(n, r)))
    s = np.linspace(10.0, 2.0, r)                                   # distinct, well separated from the noise
    e = ((u * s) @ v.T + 1e-3 * g.normal(size=(m, n)) / np.sqrt(max(m, n))).astype(np.float32)
    print(f"gap case m={m} n={n} r={r}", flush=True)
    a, sig = _factor(e, r, iters=3, seed=r)
    a_ref, sv = oracle.svd_right_factor(e, r)
    assert np.max(np.abs(sig - sv[:r])) <= 1e-4 * sv[0]
    assert np.all(np.diff(sig) <= 0)
    gram = a @ a.T
    assert np.max(np.abs(gram - np.diag(sig))) <= 1e-4 * sig[0]     # orthogonal rows, squared norms sigma_i
    assert np.linalg.norm(_projector(a) - _projector(a_ref)) <= 1e-3
    # each row is +/- the oracle's row (distinct singular values): compare up to sign
    for i in range(r):
        c = float(a[i] @ a_ref[i]) / (np.linalg.norm(a[i]) * np.linalg.norm(a_ref[i]))
        assert abs(abs(c) - 1.0) <= 1e-4, (i, c)
    # Ritz values are |E v_i|
    ev = e.astype(np.float64) @ (a / np.sqrt(sig)[:, None]).T
    assert np.max(np.abs(np.linalg.norm(ev, axis=0) - sig)) <= 1e-4 * sig[0]


def test_factor_of_a_quantization_residual_and_the_layer_it_initializes():
    """Initialization algorithm end to end on the GPU: Q(W), residual, rank-r factor, cast with s_w."""
    m, n, r, k = 1024, 768, 32, 8
    g = np.random.default_rng(11)
    w = (g.normal(size=(m, n)) * 0.02).astype(np.float32)
    ref = oracle.init_adapter(w, r)
    layer = fq.MeldedLinear(64, n, m, r, k)
    wg = torch.from_numpy(w).cuda()
    fq.quantize(wg, fq.E4M3, layer.wq[:m], layer.s_w, layer.ws)
    e = torch.empty(m, n, dtype=torch.float32, device="cuda")
    fq.init_residual(wg, layer.wq[:m], layer.s_w, e)
    torch.cuda.synchronize()
    assert np.array_equal(np_of(layer.wq[:m]), ref["wq"]) and np_of(e).tobytes() == ref["e"].tobytes()
    a, sig = _factor(ref["e"], r, iters=8, seed=5)
    sv = ref["sv"]
    assert np.all(sig <= sv[:r] * (1 + 1e-4))                        # Ritz values approach from below
    captured, best = float(np.sum(sig ** 2)), float(np.sum(sv[:r] ** 2))
    print(f"captured {captured / best:.4f} of the best rank-{r} energy", flush=True)
    assert captured >= 0.90 * best
    gram = a @ a.T
    assert np.max(np.abs(gram - np.diag(sig))) <= 1e-4 * sig[0]
    ev = ref["e"].astype(np.float64) @ (a / np.sqrt(sig)[:, None]).T
    assert np.max(np.abs(np.linalg.norm(ev, axis=0) - sig)) <= 1e-4 * sig[0]
    # last step of the initialization: the cast of A^ with the backbone's scale equals the oracle's cast of the same A^
    a32 = torch.from_numpy(a.astype(np.float32)).cuda()
    s_tmp = torch.zeros(1, device="cuda")
    fq.quantize(a32, fq.E4M3, layer.wq[m:], s_tmp, layer.ws, scale_in=layer.s_w)
    torch.cuda.synchronize()
    aq_ref, _, _ = oracle.quantize(a.astype(np.float32), oracle.E4M3, scale_in=ref["s_w"])
    assert np.array_equal(np_of(layer.wq[m:]), aq_ref)
    # and the layer it initializes runs: O_A = A~ x
    x = torch.randn(64, n, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    layer.forward(x.cuda())
    torch.cuda.synchronize()
    f = oracle.layer_fwd(x.float().numpy(), np_of(layer.wq), ref["s_w"], m, r)
    assert np.linalg.norm(np_of(layer.o_a) - f["o_a"]) <= 1e-3 * np.linalg.norm(f["o_a"])


@pytest.mark.parametrize("m,n,r", [(272, 400, 88), (272, 400, 96)])      # eigenvectors just inside the LDS, and in memory
def test_largest_subspaces(m, n, r):
    g = np.random.default_rng(r)
    e = g.normal(size=(m, n)).astype(np.float32) * np.linspace(3.0, 0.01, n, dtype=np.float32) ** 4
    a, sig = _factor(e, r, iters=4, seed=r)
    sv = np.linalg.svd(e.astype(np.float64), compute_uv=False)
    assert np.all(sig <= sv[:r] * (1 + 1e-4)) and np.sum(sig ** 2) >= 0.97 * np.sum(sv[:r] ** 2)
    assert np.max(np.abs(a @ a.T - np.diag(sig))) <= 1e-4 * sig[0]


@pytest.mark.parametrize("r,scale", [(16, 1.0), (32, 1e30), (48, 1.0), (64, 1.0), (64, 1e-33), (80, 1e-20), (96, 1.0), (112, 1.0), (120, 1.0)])
def test_products_of_many_steps_against_64_bits(r, scale):
    """Every number of vector blocks, on a matrix whose products take several steps per wave and end inside one, against the
    same iteration in fp64.  A product of fp32 rounding error moves Ritz values by at most its relative size, which for
    sums of 2500 terms of random sign is about 1e-6 at the very worst (2500 roundings of 6e-8 adding up as a random walk
    over sums of 2500 terms: 6e-8)."""
    m, n, iters = 2500, 2420, 1
    e = np.random.default_rng(r).normal(size=(m, n)).astype(np.float32) * np.float32(scale)
    a, sig = _factor(e, r, iters=iters, seed=r)
    e64 = e.astype(np.float64) / scale
    z = np.linalg.qr(torch.randn(r + 8, n, generator=torch.Generator().manual_seed(r)).numpy().astype(np.float64).T)[0]
    for _ in range(iters):
        z = np.linalg.qr(e64.T @ np.linalg.qr(e64 @ z)[0])[0]
    want = np.linalg.svd(e64 @ z, compute_uv=False)[:r]
    assert np.max(np.abs(sig / scale - want)) <= 1e-6 * want[0]
    assert np.max(np.abs((a / scale) @ a.T - np.diag(sig / scale))) <= 1e-5 * want[0]


@pytest.mark.parametrize("rank", [0, 5])
def test_matrix_of_lower_rank_than_asked_for(rank):
    """Vectors in the span of the others drop out (all of them for a zero matrix); nothing becomes NaN."""
    g = np.random.default_rng(3)
    e = (g.normal(size=(200, rank)) @ g.normal(size=(rank, 320))).astype(np.float32)
    a, sig = _factor(e, 16, iters=2, seed=1)
    assert np.all(np.isfinite(a)) and np.all(np.isfinite(sig))
    sv = np.linalg.svd(e.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(sig - sv[:16])) <= 1e-4 * max(sv[0], 1e-30)


@pytest.mark.parametrize("r", [16, 96])                                   # eigenvectors in the LDS, and in memory
def test_matrix_that_is_not_finite_leaves_the_next_one_alone(r):
    """What comes out for it is unspecified; no index is formed from it, and the same workspace serves the next matrix."""
    g = np.random.default_rng(r)
    m, n = 200, 320
    e = g.normal(size=(m, n)).astype(np.float32)
    bad = e.copy()
    bad[3, 5], bad[7, 11] = np.nan, np.inf
    omega = torch.randn(r + 8, n, generator=torch.Generator().manual_seed(r)).cuda()
    a, sig = torch.empty(r, n, device="cuda"), torch.empty(r, device="cuda")
    ws = torch.full((fq.svd_workspace_bytes(m, n, r),), 0x7f, dtype=torch.uint8, device="cuda")
    fq.svd_right_factor(torch.from_numpy(bad).cuda(), r, omega, 1, a, sig, ws)
    torch.cuda.synchronize()
    fq.svd_right_factor(torch.from_numpy(e).cuda(), r, omega, 4, a, sig, ws)
    torch.cuda.synchronize()
    sv = np.linalg.svd(e.astype(np.float64), compute_uv=False)
    sig = np_of(sig).astype(np.float64)
    assert np.all(sig <= sv[:r] * (1 + 1e-4)) and np.sum(sig ** 2) >= 0.9 * np.sum(sv[:r] ** 2)


@pytest.mark.parametrize("r", range(16, 121, 8))
def test_every_subspace_size_on_ragged_matrices(r):
    """Each number of vectors has kernels of its own; sizes around the 16 and 64 of their tiles, the smallest included.
    A = sum of s_i u_i v_i^T with a gap of 10^3 behind the r-th: both factors against the known ones.  Bounds: what is
    left of the gap after q = 3 rounds is below 1e-18, so fp32 products remain, as in the gap cases above."""
    for m, n in [(r + 8, r + 12), (r + 8 + 4 * (r // 8), 4 * r + 4 * (r // 8 % 5) + 36)]:
        g = np.random.default_rng(m * n)
        u, _ = np.linalg.qr(g.normal(size=(m, r)))
        v, _ = np.linalg.qr(g.normal(size=(n, r)))
        s = np.linspace(9.0, 2.0, r)
        e = ((u * s) @ v.T + 2e-3 * g.normal(size=(m, n)) / np.sqrt(m + n)).astype(np.float32)
        omega = torch.randn(r + 8, n, generator=torch.Generator().manual_seed(r)).cuda()
        a, bt = torch.full((r, n), 7.0, device="cuda"), torch.full((r, m), 7.0, device="cuda")
        sig = torch.empty(r, device="cuda")
        ws = torch.full((fq.svd_workspace_bytes(m, n, r),), 0x7f, dtype=torch.uint8, device="cuda")
        fq.svd_right_factor(torch.from_numpy(e).cuda(), r, omega, 3, a, sig, ws, bt_out=bt)
        torch.cuda.synchronize()
        sv = np.linalg.svd(e.astype(np.float64), compute_uv=False)
        a, bt, sig = np_of(a).astype(np.float64), np_of(bt).astype(np.float64), np_of(sig).astype(np.float64)
        assert np.max(np.abs(sig - sv[:r])) <= 1e-4 * sv[0], (m, n)
        assert np.max(np.abs(a @ a.T - np.diag(sig))) <= 1e-4 * sig[0], (m, n)
        assert np.linalg.norm(bt.T @ a - (u * s) @ v.T) <= 2e-3 * np.linalg.norm(s), (m, n)


def _factors(e, r, omega, iters):
    m, n = e.shape
    a, bt, sig = torch.empty(r, n, device="cuda"), torch.empty(r, m, device="cuda"), torch.empty(r, device="cuda")
    ws = torch.full((fq.svd_workspace_bytes(m, n, r),), 0x7f, dtype=torch.uint8, device="cuda")
    fq.svd_right_factor(torch.from_numpy(e).cuda(), r, torch.from_numpy(omega).cuda(), iters, a, sig, ws, bt_out=bt)
    torch.cuda.synchronize()
    return (np_of(x).astype(np.float64) for x in (a, bt, sig))


@pytest.mark.parametrize("r", [16, 32, 64, 120])
@pytest.mark.parametrize("decades", [3, 7, 9, 20])
def test_steep_spectrum_without_an_iteration(r, decades):
    """The first basis is random, so H = (Z E^T)(Z E^T)^T has entries of one size and eigenvalues over the whole range of
    fp64: the eigenvectors have to be orthogonal to one another all the same, and both factors those of E Z^T Z.  Bounds:
    Z and the product are exact to some 1e-7 of the largest singular value, and H to l 1e-16 of its square."""
    g = np.random.default_rng(r + decades)
    m, n, rank = 200, 300, 160
    u, _ = np.linalg.qr(g.normal(size=(m, rank)))
    v, _ = np.linalg.qr(g.normal(size=(n, rank)))
    e = ((u * np.logspace(0, -decades, rank)) @ v.T).astype(np.float32)
    omega = g.normal(size=(r + 8, n)).astype(np.float32)
    a, bt, sig = _factors(e, r, omega, 0)
    q, _ = np.linalg.qr(omega.T.astype(np.float64))
    uu, ss, vv = np.linalg.svd(e.astype(np.float64) @ q, full_matrices=False)
    assert np.all(np.diff(sig) <= 0) and np.max(np.abs(sig - ss[:r])) <= 1e-6 * ss[0]
    assert np.max(np.abs(a @ a.T - np.diag(sig))) <= 1e-6 * ss[0]
    assert np.linalg.norm(bt.T @ a - (uu[:, :r] * ss[:r]) @ vv[:r] @ q.T) <= 1e-5 * ss[0]


@pytest.mark.parametrize("seed", [5, 6, 7])
def test_small_singular_values_of_rows_apart_from_the_large(seed):
    """Two blocks without common rows and columns: what is small beside the other one, here 1e-8 of it, keeps a precision
    of its own.  (The small block has no gap: its Ritz values come within a few per cent, from below.)"""
    g = np.random.default_rng(seed)
    e = np.zeros((400, 600), np.float32)
    e[:16, :16] = g.normal(size=(16, 16)) + 4.0 * np.eye(16)
    e[100:, 300:] = 1e-8 * g.normal(size=(300, 300)) * 0.4
    a, bt, sig = _factors(e, 32, g.normal(size=(40, 600)).astype(np.float32), 6)
    sv = np.linalg.svd(e.astype(np.float64), compute_uv=False)[:32]
    assert np.all(np.diff(sig) <= 0) and np.max(np.abs(sig[:16] / sv[:16] - 1.0)) <= 1e-4
    assert np.all(sig[16:] <= sv[16:] * 1.001) and np.all(sig[16:] >= 0.9 * sv[16:])
    small = (bt.T @ a)[100:, 300:]
    assert np.linalg.norm(small, 2) <= sv[16] * 1.01 and np.linalg.norm(small) >= 0.9 * np.linalg.norm(sv[16:])


@pytest.mark.parametrize("m,n,r,rank,iters", [(128, 128, 120, 100, 0), (92, 64, 56, 40, 1), (128, 192, 120, 70, 4), (104, 156, 96, 90, 2)])
def test_both_factors_where_the_rank_is_lower_than_asked_for(m, n, r, rank, iters):
    """What is left of the matrix there is rounding: its rows have to be as small, and as orthogonal, in either factor.
    Bound: 16 roundings of fp32 of the largest value."""
    g = np.random.default_rng(m + n)
    u, _ = np.linalg.qr(g.normal(size=(m, rank)))
    v, _ = np.linalg.qr(g.normal(size=(n, rank)))
    e = ((u * g.uniform(0.1, 1.0, rank)) @ v.T).astype(np.float32)
    a, bt, sig = _factors(e, r, g.normal(size=(r + 8, n)).astype(np.float32), iters)
    assert np.all(np.diff(sig) <= 0)
    for f in (a, bt):
        assert np.max(np.abs(f @ f.T - np.diag(sig))) <= 1e-6 * sig[0]
    if iters:
        assert np.linalg.norm(bt.T @ a - e) <= 1e-6 * np.linalg.norm(e) * np.sqrt(rank)


@pytest.mark.parametrize("largest", [3.3999e38, 1.3e36, 1e-3, 8e-33, 1.7e-36])
def test_entries_at_the_ends_of_the_range(largest):
    """The products take elements in parts of 8 bits, which hold numbers up to 3.39e38 and, to all their bits, down to 1.5e-33:
    beyond that the elements have to be taken whole.  Twenty entries in rows and columns of their own are the singular values,
    and all of them are in a subspace of 24.  Bound: 16 roundings of fp32."""
    g = np.random.default_rng(1)
    m, n = 200, 324
    values = np.sort(largest * g.uniform(0.2, 1.0, 20).astype(np.float32))[::-1].astype(np.float32)
    values[0] = np.float32(largest)
    e = np.zeros((m, n), np.float32)
    e[g.permutation(m)[:20], g.permutation(n)[:20]] = values
    a, bt, sig = _factors(e, 16, g.normal(size=(24, n)).astype(np.float32), 2)
    assert np.max(np.abs(sig / values[:16] - 1.0)) <= 1e-6
    assert np.max(np.abs((a / sig[0]) @ a.T - np.diag(sig / sig[0]))) <= 1e-6
    assert np.max(np.abs((bt.T / sig[0]) @ a - np.where(e >= values[15], e / sig[0], 0.0))) <= 1e-6


@pytest.mark.parametrize("r", [16, 32, 40, 64, 80, 88, 104, 120])
@pytest.mark.parametrize("scale", [1e-34, 1e36])
def test_products_of_whole_elements_against_64_bits(r, scale):
    """Every number of vector blocks with elements beyond the range of the parts, on sizes that end inside steps and tiles.
    Bounds as in the products of many steps above."""
    m, n = 300, 412
    e = np.random.default_rng(r).normal(size=(m, n)).astype(np.float32) * np.float32(scale)
    a, sig = _factor(e, r, iters=1, seed=r)
    e64 = e.astype(np.float64) / scale
    z = np.linalg.qr(torch.randn(r + 8, n, generator=torch.Generator().manual_seed(r)).numpy().astype(np.float64).T)[0]
    z = np.linalg.qr(e64.T @ np.linalg.qr(e64 @ z)[0])[0]
    want = np.linalg.svd(e64 @ z, compute_uv=False)[:r]
    assert np.max(np.abs(sig / scale - want)) <= 1e-6 * want[0]
    assert np.max(np.abs((a / scale) @ a.T - np.diag(sig / scale))) <= 1e-5 * want[0]
