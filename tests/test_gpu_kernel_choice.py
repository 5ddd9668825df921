"""The kernel that serves a block, where a GPU decides: pinned variants, autotuning, vector layouts."""
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


@pytest.mark.parametrize("N,dt", [(38, syk.C64), (38, syk.C128), (40, syk.C64), (42, syk.C64), (42, syk.C128)])
def test_otoc_in_an_explicit_layout_runs_in_the_tiled_kernel(N, dt):
    """Blocks that are gathered by default (2^18, and 2^19 in complex64) and tiled ones: a rotated layout is
    the tiled kernel's, bit for bit what a handle pinned to it gives.  All agree within the bound of the
    precision's correlators in the parity tests."""
    h, pinned = (syk.create_hamiltonian(N, 4, 2, 7) for _ in range(2))
    syk.select_variant(pinned, dt, syk.plan_describe(h, 0, dt)["variant"])
    gathered = syk.apply_kernel(h, dt) == syk.KERNEL_GATHER
    assert gathered == (N == 38 or (N == 40 and dt == syk.C64))
    ts = [0.0, 1.0]

    def run(ham, layout):
        return syk.otoc(ham, N - 1, N - 2, 2.0, ts, nvec=1, state_seed=3, dtype=dt, layout=layout, autotune=False)[0]

    ref = run(h, 0)
    tol = 1e-9 if dt == syk.C128 else 1e-5
    rotated = [(run(h, r), run(pinned, r)) for r in (1, 7, N // 2 - 2)]
    for a, b in rotated + [(run(h, -1), ref), (run(pinned, 0), ref)]:
        assert abs(a - ref).max() <= tol * max(1.0, abs(ref).max())
    for a, b in rotated:
        assert (a == b).all()
    assert any((a != ref).any() for a, b in rotated)      # another order of sums, so not the kernel of `ref`
    if gathered:
        assert (run(h, -1) == ref).all()


def test_a_run_keeps_its_kernel_while_another_thread_pins_and_tunes():
    """A dense block of 2^22 amplitudes: the two kernels leave their partial sums to be added by different
    launches, so a run may not change kernels half way.  Results of both kernels agree within the Krylov
    bound, whichever a run began with."""
    import threading

    import numpy as np
    L, rng = 22, np.random.default_rng(5)
    x = np.repeat(np.array([0, 5, 77, 1 << 21], dtype=np.uint64), 5)
    z = (np.arange(20, dtype=np.uint64) * np.uint64(7919)) % np.uint64(1 << L)
    odd = np.array([bin(int(a & b)).count("1") & 1 for a, b in zip(x, z)])
    h = syk.Operator(L, x, z, rng.standard_normal(20) / 5.0 * np.where(odd, 1j, 1.0)).to_hamiltonian()
    v = torch.randn(1 << L, dtype=torch.complex64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    v /= torch.linalg.vector_norm(v)
    ref = torch.empty_like(v)
    syk.krylov_expm(h, 0, -0.4 + 0.9j, v, ref, reorth=2)
    torch.cuda.synchronize()
    stop, errors = threading.Event(), []

    def flip():
        try:
            s = torch.cuda.Stream()
            while not stop.is_set():
                syk.select_variant(h, syk.C64, 10)
                stop.wait(0.002)
                syk.autotune(h, syk.C64, stream=s)
            syk.release_workspace()
        except Exception as e:                            # reported by the test's thread
            errors.append(e)

    t = threading.Thread(target=flip)
    t.start()
    try:
        out = torch.empty_like(v)
        for _ in range(60):
            syk.krylov_expm(h, 0, -0.4 + 0.9j, v, out)
            assert float(torch.linalg.vector_norm(out - ref)) <= 1e-5
    finally:
        stop.set()
        t.join()
    assert not errors
