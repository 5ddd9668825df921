"""The grouped gather kernel from 2^19 to 2^22 amplitudes, the largest it serves: applies against sampled
oracle rows, and the fused Lanczos steps, whose partial sums there are too many for the next pass
to add (launches of their own), against full reorthogonalisation.  Few terms on few x masks."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402
from tests.test_gpu_gather import _check  # noqa: E402

pytestmark = pytest.mark.gpu


def _terms(L, masks, per, seed):
    """`per` or more distinct z masks on each of `masks` x masks, the diagonal among them."""
    rng = np.random.default_rng(seed)
    m = np.unique(np.concatenate([[0], rng.integers(0, 1 << L, masks - 1)])).astype(np.uint64)
    x = np.repeat(m, per)
    z = np.concatenate([rng.choice(1 << 16, per, replace=False).astype(np.uint64) << np.uint64(L - 16) ^ np.uint64(g)
                        for g in range(m.size)])
    return x, z, rng


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("L,masks,per", [(19, 6, 5), (20, 5, 4), (21, 3, 17), (22, 4, 6)])
def test_rows(L, masks, per, dt):
    x, z, rng = _terms(L, masks, per, L)
    c = rng.standard_normal(x.size) + 1j * rng.standard_normal(x.size)
    # complex coefficients are two terms each
    assert syk.apply_kernel(syk.Operator(L, x, z, c).to_hamiltonian(), dt) == syk.KERNEL_GROUPED
    _check(L, x, z, c, dt, nrows=1500)


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("L", [19, 20, 21, 22])
def test_propagation(L, dt):
    x, z, rng = _terms(L, 4, 6, 50 + L)
    odd = np.array([bin(int(a & b)).count("1") & 1 for a, b in zip(x, z)])
    h = syk.Operator(L, x, z, rng.standard_normal(x.size) / 5.0 * np.where(odd, 1j, 1.0)).to_hamiltonian()
    assert syk.apply_kernel(h, dt) == syk.KERNEL_GROUPED
    cd = torch.complex64 if dt == syk.C64 else torch.complex128
    v = torch.randn(1 << L, dtype=cd, device="cuda", generator=torch.Generator(device="cuda").manual_seed(L))
    v /= torch.linalg.vector_norm(v)
    a, b = torch.empty_like(v), torch.empty_like(v)
    for w, m in ((-0.4 + 0.9j, 30), (1.2j, 8)):            # the second in several sub-steps
        syk.krylov_expm(h, 0, w, v, a, m=m)
        syk.krylov_expm(h, 0, w, v, b, m=30, reorth=2)
        err = float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))
        assert err <= (1e-10 if dt == syk.C128 else 1e-5)
