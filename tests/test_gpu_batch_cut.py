"""Parts and slots of the batched OTOC.  Jobs are cut so that a lone item fills more workgroups than its
whole jobs would, and a large batch is not.  A job is an (item, vector) pair of two parity-block chains; a
part is a range of one chain's t points."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2311_00639_amd as syk  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,variant,ts", [(18, 2, [0.0, 0.3, 0.3, 1.0]), (24, 0, [0.0, 0.5, 1.0, 2.0, 4.0]),
                                          (28, 1, [0.25, 0.5]), (32, 0, [0.0, 0.5])])
def test_a_lone_item_is_cut_at_its_t_points(N, variant, ts):
    """nvec = 2: four whole chains, one slot each at most if nothing were cut.  The cut repeats the
    incremental propagations, so results and counts equal those of the whole jobs, which an item has
    among many equal ones."""
    torch.cuda.set_device(0)
    item = (N, 4, 300, N - 1, N - 2, 900)
    one = syk.otoc_batch([item], 4.0, ts, nvec=2, variant=variant)
    assert one[3]["slots"] > 4 and one[3]["n_jobs"] == 2
    # at most one part per chain and t point (t = 0 is prepended where the grid lacks it)
    assert one[3]["slots"] <= 4 * (len(ts) + (ts[0] != 0.0))
    slots = torch.cuda.get_device_properties(0).multi_processor_count * (1, 2, 4)[variant]
    count = slots                                          # 4 chains per slot: the longest is below half the mean
    many = syk.otoc_batch([item] * count, 4.0, ts, nvec=2, variant=variant) if N <= 24 else None
    if many is not None:
        assert many[3]["slots"] == slots
        assert many[3]["matvecs"] == count * one[3]["matvecs"]
        for a, b in zip(one[:3], many[:3]):
            assert all(np.array_equal(a[0], row) for row in b)


def test_short_of_memory_runs_with_fewer_slots():
    """With about 3 GiB left, fewer slots than one per CU (4.4 GB of vectors) serve an item's parts, with the same
    result."""
    torch.cuda.set_device(0)
    item, ts = [(32, 2, 300, 31, 30, 900)], [0.02 * k for k in range(40)]
    full = syk.otoc_batch(item, 0.5, ts, nvec=4, m=60)
    assert full[3]["slots"] >= 240
    syk.release_workspace()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    hold = torch.empty(free - (3 << 30), dtype=torch.uint8, device="cuda")
    try:
        few = syk.otoc_batch(item, 0.5, ts, nvec=4, m=60)
    finally:
        del hold
        torch.cuda.empty_cache()
        syk.release_workspace()
    assert 1 <= few[3]["slots"] < 240
    for a, b in zip(full[:3], few[:3]):
        assert np.array_equal(a, b)
