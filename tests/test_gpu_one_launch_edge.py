"""One launch per Lanczos step up to 16 MB of further reads (2 K 2^L amplitudes), two above: both sides of the
rule in both precisions, with the Krylov dimension ending the steps before the next error check.
"""
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k,dt,one", [(26, 4, syk.C128, True), (26, 5, syk.C128, False), (28, 4, syk.C64, True),
                                        (28, 5, syk.C64, False)])
@pytest.mark.parametrize("m", [4, 5, 9, 30])
def test_both_sides_of_the_rule(N, k, dt, one, m):
    """Tolerance: the accepted errors sum to at most tol, and each sub-step rounds its applies and its
    result (8 units), as in the tests of small Krylov dimensions."""
    n = 1 << (N // 2 - 1)
    assert (2 * round(k * N) * n * (16 if dt == syk.C128 else 8) <= 16e6) == one
    h = syk.create_hamiltonian(N, 4, k, 3)
    x = torch.randn(n, dtype=torch.complex64 if dt == syk.C64 else torch.complex128, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(7))
    x /= torch.linalg.vector_norm(x)
    out, ref = torch.empty_like(x), torch.empty_like(x)
    z = 0.02j if m < 30 else 0.3j
    st = syk.krylov_expm(h, 0, z, x, out, m=m, tol=1e-5)
    syk.krylov_expm(h, 0, z, x, ref, m=40, reorth=2)
    assert st["matvecs"] <= m * st["substeps"]
    u = 2.0 ** -24 if dt == syk.C64 else 2.0 ** -53
    assert float(torch.linalg.vector_norm(out - ref)) <= 1e-5 + st["substeps"] * 8 * u
