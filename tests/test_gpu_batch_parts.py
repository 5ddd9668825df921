"""The cut of batched jobs into parts (one block's chain over a range of t points): results, matvec
counts and the sub-step limit do not depend on it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402

pytestmark = pytest.mark.gpu


def _items(N, count):
    return [(N, (2, 4, 8)[r % 3], 300 + r, N - 1, N - 2, 900 + r) for r in range(count)]


@pytest.mark.parametrize("N,variant,ts", [(18, 2, [0.0, 0.3, 0.3, 1.0]), (20, 1, [0.4]), (24, 0, [0.0, 0.5, 1.0, 2.0, 4.0]),
                                          (28, 1, [0.25, 0.5]), (32, 0, [0.0, 0.5])])
def test_cut_jobs_equal_whole_jobs_bitwise(N, variant, ts):
    """An item alone is cut at its t points to fill the chip; among many it runs whole."""
    torch.cuda.set_device(0)
    count = 600 if N <= 24 else 40
    many = syk.otoc_batch(_items(N, count), 4.0, ts, nvec=2, variant=variant)
    total = 0
    for r in (0, 1, count - 1):
        one = syk.otoc_batch(_items(N, count)[r:r + 1], 4.0, ts, nvec=2, variant=variant)
        for a, b in zip(one[:3], many[:3]):
            assert np.array_equal(a[0], b[r])
        total += one[3]["matvecs"]
    three = syk.otoc_batch([_items(N, count)[r] for r in (0, 1, count - 1)], 4.0, ts, nvec=2, variant=variant)
    assert three[3]["matvecs"] == total and three[3]["n_jobs"] == 6


def test_substep_limit_is_per_job():
    torch.cuda.set_device(0)
    item, ts = _items(20, 1), [0.0, 1.0, 2.0]
    # m = 4 needs several sub-steps per propagation, and a job has 2 (2 + 2 + 4 + 4) propagations
    with pytest.raises(syk.SykError) as e:
        syk.otoc_batch(item, 2.0, ts, m=4, max_substeps=28)
    assert e.value.status == 5
    raw = syk.otoc_batch(item, 2.0, ts, m=4)[0]
    ref = syk.otoc_batch(item, 2.0, ts, m=30)[0]
    assert np.abs(raw - ref).max() <= 1e-5 * abs(ref[0][0])
