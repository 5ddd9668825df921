"""The gather kernels of apply_H: blocks of at most 4 MiB, and dense blocks up to 2^22.

Random Pauli sums (complex coefficients, so both phases occur) against the oracle's matrix-free
rows, at the edges of the kernels' amplitude tiles (64 to 512 amplitudes), of their launch rules
(2^14 to 2^19 amplitudes) and of the term slices (fewer terms or masks than slices).
Tolerance per row: a sum of M products accumulates at most M roundings, each within u of the
running sum of |c x|, so |err| <= M u sum |c x| with M = 2 K + 20 (real and imaginary part of
each coefficient, the sums over slices, the rounding of c).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402
from oracle import matfree, pauli  # noqa: E402
from tests import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def _check(L, x, z, c, dt, nrows=500):
    h = syk.Operator(L, x, z, c).to_hamiltonian()
    n = 1 << L
    cd = torch.complex64 if dt == syk.C64 else torch.complex128
    xd = torch.from_numpy(inputs.complex_vector(n, L + len(x))[0]).to(dtype=cd, device="cuda")
    yd = torch.full_like(xd, float("nan"))
    syk.apply_H(h, 0, xd, yd)
    y, xr = yd.cpu().numpy().astype(np.complex128), xd.cpu().numpy().astype(np.complex128)
    rows = inputs.row_sample(n, nrows, 3)
    strings = [(pauli.from_xz(L, int(a), int(b)), v) for a, b, v in zip(x, z, c)]
    terms = [(labels, v * 1j ** p) for (labels, p), v in strings]
    yref = matfree.apply_rows(terms, lambda i: xr[i.astype(np.int64)], rows)
    mag = sum(abs(v) * np.abs(xr[(rows ^ np.uint64(a)).astype(np.int64)]) for a, v in zip(x, c))
    u = 2.0 ** -53 if dt == syk.C128 else 2.0 ** -24
    assert np.all(np.abs(y[rows.astype(np.int64)] - yref) <= (2 * len(x) + 20) * u * mag)
    assert np.isfinite(y).all()


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("L,K", [(2, 3), (5, 1), (6, 9), (7, 40), (13, 17), (14, 60), (16, 33), (17, 5), (17, 70),
                                 (18, 33), (19, 21)])
def test_sparse_gather(L, K, dt):
    rng = np.random.default_rng(100 * L + K)
    x = rng.integers(0, 1 << L, K).astype(np.uint64)
    z = rng.integers(0, 1 << L, K).astype(np.uint64)
    _check(L, x, z, rng.standard_normal(K) + 1j * rng.standard_normal(K), dt)


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("L,masks,per", [(6, 7, 8), (7, 33, 6), (8, 1, 5), (8, 20, 9), (9, 3, 4), (15, 40, 7), (16, 17, 23), (17, 2, 31),
                                        (18, 5, 6), (19, 33, 8)])
def test_grouped_gather(L, masks, per, dt):
    rng = np.random.default_rng(100 * L + masks)
    m = rng.choice(1 << L, masks, replace=False).astype(np.uint64)
    m[0] = 0                                             # a diagonal group
    # groups of unequal size (not multiples of four), one of them with a single phase
    sizes = [max(1, per + int(rng.integers(-2, 3))) + (per if g == 0 else 2) for g in range(masks)]
    x = np.concatenate([np.full(s, a, dtype=np.uint64) for a, s in zip(m, sizes)])
    z = np.concatenate([rng.choice(min(1 << L, 4096), s, replace=False).astype(np.uint64) * np.uint64((1 << L) // min(
        1 << L, 4096)) ^ np.uint64(g % 5) for g, s in enumerate(sizes)])
    c = rng.standard_normal(x.size) + 1j * rng.standard_normal(x.size)
    c[:sizes[0]] = c[:sizes[0]].real
    h = syk.Operator(L, x, z, c).to_hamiltonian()
    if L < 18:
        assert syk.plan_describe(h, 0, dt, -1)["n_groups"] == masks
    _check(L, x, z, c, dt)


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("N,dense", [(10, False), (20, False), (34, False), (20, True)])
def test_many_vectors_and_full_space_bitwise(N, dense, dt):
    """Vectors at a ragged stride and both blocks in one launch give, bit for bit, what single
    vectors and blocks give, and leave the padding alone."""
    k = (N - 1) * (N - 2) * (N - 3) / 24.0 if dense else 4
    h = syk.create_hamiltonian(N, 4, k, 5, syk.BERNOULLI if dense else syk.EXACT_K)
    n = 1 << (N // 2 - 1)
    nvec, ld = 3, 2 * n + 5
    cd = torch.complex64 if dt == syk.C64 else torch.complex128
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn(nvec, ld, dtype=cd, device="cuda", generator=g)
    y = torch.full_like(x, 3.0)
    syk.apply_H(h, syk.FULL, x, y, nvec=nvec, ld=ld)
    one = torch.empty(n, dtype=cd, device="cuda")
    for v in range(nvec):
        for b in (0, 1):
            syk.apply_H(h, b, x[v, b * n:(b + 1) * n].clone(), one)
            assert torch.equal(y[v, b * n:(b + 1) * n], one)
    assert torch.all(y[:, 2 * n:] == 3.0)


@pytest.mark.parametrize("N,dense,dt", [(38, True, syk.C128), (38, False, syk.C128), (38, False, syk.C64),
                                        (40, False, syk.C64)])
def test_gathered_block_pinned_to_a_tiled_variant_matches(N, dense, dt):
    """A dense block above the tiled size, or a block that fits an L2, runs the gather kernels unless a
    tiled variant is pinned; the two agree within twice the term-by-term accumulation bound."""
    k = (N - 1) * (N - 2) * (N - 3) / 24.0 if dense else 4
    h = syk.create_hamiltonian(N, 4, k, 2, syk.BERNOULLI if dense else syk.EXACT_K)
    n = 1 << (N // 2 - 1)
    cd = torch.complex64 if dt == syk.C64 else torch.complex128
    x = torch.randn(n, dtype=cd, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    a, b = torch.empty_like(x), torch.empty_like(x)
    syk.apply_H(h, 0, x, a)
    syk.select_variant(h, dt, 11)
    syk.apply_H(h, 0, x, b)
    u = 2.0 ** -53 if dt == syk.C128 else 2.0 ** -24
    bound = 2 * h.info()["K"] * u * float(np.abs(0.25 * h.terms()["J"]).sum()) * float(x.abs().max())
    assert float((a - b).abs().max()) <= bound
    assert not torch.equal(a, b)                          # not the same kernel
