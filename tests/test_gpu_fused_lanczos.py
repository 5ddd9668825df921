"""The fused Lanczos steps of krylov_expm (reorth = 0) against the unfused, fully
reorthogonalised run of the same propagation.

Sizes: the gather kernels' tiles and launch rules (2^2 ... 2^17 amplitudes, sparse and dense), a dense
block above the tiled size, and the tiled kernel on both sides of the change from summing the
partials in the next pass to launches of their own (2^21 and 2^22 amplitudes).  Both runs meet the
requested tolerance (1e-12 in complex128, 1e-7 in complex64) per propagation; the bounds are the
Krylov bounds of the parity tests, 1e-10 and 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402

pytestmark = pytest.mark.gpu


def _state(n, dt, seed):
    cd = torch.complex64 if dt == syk.C64 else torch.complex128
    x = torch.randn(n, dtype=cd, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed))
    return x / torch.linalg.vector_norm(x)


def _ham(N, k, seed=3):
    dense = k == "dense"
    return syk.create_hamiltonian(N, 4, (N - 1) * (N - 2) * (N - 3) / 24.0 if dense else k, seed,
                                  syk.BERNOULLI if dense else syk.EXACT_K)


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("N,k", [(6, 1), (12, 3), (14, 4), (16, 4), (18, "dense"), (28, 4), (30, 4), (32, "dense"),
                                (34, 4), (34, "dense"), (36, 2), (38, "dense"), (44, 2), (46, 2)])
def test_fused_steps_vs_reorthogonalised(N, k, dt):
    h = _ham(N, k)
    x = _state(1 << (N // 2 - 1), dt, N)
    z = -0.4 + 0.9j
    out, ref = torch.full_like(x, float("nan")), torch.empty_like(x)
    st = syk.krylov_expm(h, 1, z, x, out)
    syk.krylov_expm(h, 1, z, x, ref, reorth=2)
    err = float(torch.linalg.vector_norm(out - ref) / torch.linalg.vector_norm(ref))
    assert err <= (1e-10 if dt == syk.C128 else 1e-5)
    assert st["substeps"] == 1 and st["matvecs"] >= 2
    again = torch.empty_like(x)
    st2 = syk.krylov_expm(h, 1, z, x, again)
    assert torch.equal(out, again) and st == st2           # what runs ahead does not show
    y = x.clone()
    syk.krylov_expm(h, 1, z, y, y)                          # in place
    assert torch.equal(y, out)


@pytest.mark.parametrize("N", [16, 34, 40])
def test_restarts(N):
    """A Krylov dimension too small for z: several sub-steps of bisected length."""
    h = _ham(N, 4)
    x = _state(1 << (N // 2 - 1), syk.C128, 5)
    out, ref = torch.empty_like(x), torch.empty_like(x)
    st = syk.krylov_expm(h, 0, 1.5j, x, out, m=6)
    syk.krylov_expm(h, 0, 1.5j, x, ref, m=60, reorth=2)
    assert st["substeps"] > 2 and st["matvecs"] <= 6 * st["substeps"]
    assert float(torch.linalg.vector_norm(out - ref)) <= 1e-10
    with pytest.raises(syk.SykError) as e:
        syk.krylov_expm(h, 0, 1.5j, x, out, m=6, max_substeps=1)
    assert e.value.status == 5


@pytest.mark.parametrize("N", [16, 34, 40])
def test_zero_and_non_finite_vectors(N):
    h = _ham(N, 4)
    x = torch.zeros(1 << (N // 2 - 1), dtype=torch.complex128, device="cuda")
    out = torch.full_like(x, 7.0)
    syk.krylov_expm(h, 0, -0.5 + 1j, x, out)
    assert torch.equal(out, x)
    for bad in (float("nan"), float("inf")):
        x[3] = bad
        with pytest.raises(syk.SykError) as e:
            syk.krylov_expm(h, 0, -0.5 + 1j, x, out)
        assert e.value.status == 6
    y = _state(x.numel(), syk.C128, 1)                      # the next run is not disturbed
    a = torch.empty_like(y)
    syk.krylov_expm(h, 0, -0.5 + 1j, y, a)
    assert np.isfinite(float(torch.linalg.vector_norm(a)))


def test_threads_and_streams_share_nothing():
    """Runs of several threads, each on its own stream, give what they give alone."""
    import threading
    cases = [(16, 1), (24, 2), (34, 3), (40, 4)]
    hams = [_ham(N, 4, s) for N, s in cases]
    xs = [_state(1 << (N // 2 - 1), syk.C64, s) for N, s in cases]
    alone = []
    for h, x in zip(hams, xs):
        alone.append(torch.empty_like(x))
        syk.krylov_expm(h, 0, -0.3 + 0.7j, x, alone[-1])
    torch.cuda.synchronize()
    outs = [[torch.empty_like(x) for _ in range(5)] for x in xs]

    def work(i):
        s = torch.cuda.Stream()
        for o in outs[i]:
            syk.krylov_expm(hams[i], 0, -0.3 + 0.7j, xs[i], o, stream=s)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for o, a in zip(outs, alone):
        assert all(torch.equal(v, a) for v in o)


@pytest.mark.parametrize("dt", [syk.C128, syk.C64])
@pytest.mark.parametrize("N,m", [(8, 2), (16, 2), (16, 3), (16, 5), (24, 7), (28, 4)])
def test_small_krylov_dimensions(N, m, dt):
    """The dimension ends the steps before the next error check, with one launch per step (N <= 28 here)
    and its two spare slots: the accepted errors sum to at most tol, and each sub-step rounds its applies and
    its result (8 units).  With m = 2 the estimate falls only linearly with the sub-step, so that no sub-step
    meets a tolerance proportional to it: refused on every path."""
    h = _ham(N, 2 if N == 8 else 4)
    x = _state(1 << (N // 2 - 1), dt, 7)
    out, ref = torch.empty_like(x), torch.empty_like(x)
    if m == 2:
        for reorth in (0, 2):
            with pytest.raises(syk.SykError) as e:
                syk.krylov_expm(h, 0, 0.02j, x, out, m=m, tol=1e-5, reorth=reorth)
            assert e.value.status == 5
        return
    st = syk.krylov_expm(h, 0, 0.02j, x, out, m=m, tol=1e-5)
    syk.krylov_expm(h, 0, 0.02j, x, ref, m=40, reorth=2)
    assert st["matvecs"] <= m * st["substeps"]
    assert float(torch.linalg.vector_norm(out - ref)) <= 1e-5 + st["substeps"] * 8 * (2.0 ** -24 if dt == syk.C64 else 2.0 ** -53)
