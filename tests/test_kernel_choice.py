"""Which kernel serves a block (syk_apply_kernel), by size, precision and terms per x mask; without a GPU."""
import pytest

import paper_2311_00639_amd as syk


def _ham(N, k=2):
    dense = k == "dense"
    return syk.create_hamiltonian(N, 4, (N - 1) * (N - 2) * (N - 3) / 24.0 if dense else k, 2,
                                  syk.BERNOULLI if dense else syk.EXACT_K)


@pytest.mark.parametrize("N,c64,c128", [(6, syk.KERNEL_GATHER, syk.KERNEL_GATHER), (36, syk.KERNEL_GATHER, syk.KERNEL_GATHER),
                                        (38, syk.KERNEL_GATHER, syk.KERNEL_GATHER), (40, syk.KERNEL_GATHER, syk.KERNEL_TILED),
                                        (42, syk.KERNEL_TILED, syk.KERNEL_TILED), (56, syk.KERNEL_TILED, syk.KERNEL_TILED)])
def test_sparse_blocks(N, c64, c128):
    """Blocks of at most 4 MiB are gathered: 2^19 amplitudes in complex64, 2^18 in complex128."""
    h = _ham(N)
    assert (syk.apply_kernel(h, syk.C64), syk.apply_kernel(h, syk.C128)) == (c64, c128)
    assert syk.plan_describe(h, 0, syk.C64)["tiled"] == (N >= 38)         # the plan exists either way


@pytest.mark.parametrize("N,kernel", [(12, syk.KERNEL_GATHER), (14, syk.KERNEL_GROUPED), (30, syk.KERNEL_GROUPED),
                                      (38, syk.KERNEL_GROUPED), (46, syk.KERNEL_GROUPED), (48, syk.KERNEL_TILED)])
def test_dense_blocks(N, kernel):
    """From one 64-amplitude tile (L = 6) to 2^22 amplitudes."""
    h = _ham(N, "dense")
    assert syk.apply_kernel(h, syk.C64) == syk.apply_kernel(h, syk.C128) == kernel


def test_a_pinned_variant_is_tiled_in_its_precision():
    h = _ham(38, "dense")
    syk.select_variant(h, syk.C64, 9)
    assert syk.apply_kernel(h, syk.C64) == syk.KERNEL_TILED and syk.apply_kernel(h, syk.C128) == syk.KERNEL_GROUPED
    small = _ham(36)
    syk.select_variant(small, syk.C64, 9)                                  # below the tiled size
    assert syk.apply_kernel(small, syk.C64) == syk.KERNEL_GATHER


def test_refuses_an_unknown_precision():
    with pytest.raises(syk.SykError) as e:
        syk.apply_kernel(_ham(12), 2)
    assert e.value.status == 1
