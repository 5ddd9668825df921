"""The kernel that serves a block, where a GPU decides: pinned variants and autotuning."""
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402

pytestmark = pytest.mark.gpu


def _cd(dt):
    return torch.complex64 if dt == syk.C64 else torch.complex128


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
def test_autotune_forgets_a_pinned_variant(dt):
    """A 2^18 block pinned to the tiled kernel is gathered again after syk_autotune, in that precision
    only, and gives the gather kernel's result bit for bit; a tiled block stays tiled."""
    h = syk.create_hamiltonian(38, 4, 2, 4)
    x = torch.randn(1 << 18, dtype=_cd(dt), device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    y, z = torch.empty_like(x), torch.empty_like(x)
    syk.apply_H(h, 0, x, y)
    for d in (syk.C64, syk.C128):
        syk.select_variant(h, d, 11)
        assert syk.apply_kernel(h, d) == syk.KERNEL_TILED
    syk.autotune(h, dt)
    assert syk.apply_kernel(h, dt) == syk.KERNEL_GATHER
    assert syk.apply_kernel(h, syk.C64 + syk.C128 - dt) == syk.KERNEL_TILED
    syk.apply_H(h, 0, x, z)
    assert torch.equal(y, z)
    big = syk.create_hamiltonian(42, 4, 2, 4)
    syk.select_variant(big, dt, 9)
    syk.autotune(big, dt)
    assert syk.apply_kernel(big, dt) == syk.KERNEL_TILED
