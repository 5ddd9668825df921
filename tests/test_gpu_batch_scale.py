"""The scale of a propagation's start vector in the batched OTOC: formed in 64 bits, one rounding per
amplitude.  A scale rounded to 32 bits would multiply the whole result of every propagation.

At beta = 1e-3 and t = 0 the propagators are the identity up to 1e-3, so what is left of the error of
F(0) against the complex128 run on the same Haar vectors is the rounding of the stored vectors: at
most 12 roundings of each amplitude (Haar state, r0, r2, r4, r6, the Majorana strings exact; bra and
ket), each at most u = 2^-24 relative and independent between amplitudes.  Their mean over the 2^(L+1)
amplitudes, weighted by |psi|^2 (a factor sqrt 2 for Gaussian amplitudes), has a standard deviation of
at most sqrt(12) sqrt(2) u / sqrt(3 2^(L+1)); the bound is six of them, 17 u / sqrt(2^(L+1)).
"""
import math

import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,variant", [(18, 2), (20, 1), (24, 0), (28, 1), (30, 2), (32, 0)])
def test_start_vector_is_scaled_in_64_bits(N, variant):
    torch.cuda.set_device(0)
    items = [(N, 4, 300 + r, N - 1, N - 2, 900 + r) for r in range(16)]
    raw = syk.otoc_batch(items, 1e-3, [0.0], nvec=1, variant=variant)[0]
    bound = 17.0 * 2.0 ** -24 / math.sqrt(2.0 ** (N // 2))
    for r, it in enumerate(items):
        h = syk.create_hamiltonian(N, 4, it[1], it[2])
        ref = syk.otoc(h, N - 1, N - 2, 1e-3, [0.0], nvec=1, state_seed=it[5], dtype=syk.C128)[0]
        assert abs(raw[r][0] - ref[0]) <= bound * abs(ref[0]), r
