"""Host code of the compute calls, on a device that only notes what is launched on it (tests/fake_device)."""
import pytest

import fake_device


@pytest.fixture(scope="module")
def device(tmp_path_factory):
    return fake_device.build(tmp_path_factory.mktemp("fake"))


def test_simulation_calls_go_through_when_host_memory_is_out(device):
    """No C++ exception leaves the C entry points, and a simulation call needs no host memory at all: whole histogram and
    strata, strata that fit in bins and strata that do not."""
    out = fake_device.run(device, """
cum, ends = W.length_histogram_piecewise_uniform(), W.LENGTH_STRATUM_END
sums = 4096
with lbs.Dataset(cum, ends, device=0) as ds:
    for gpn, batch in ((8, 16), (4, 64), (1, 3)):
        quota = [int(x) for x in W.stratum_quota(cum, ends, batch)]
        for call in [lambda m=m: ds.lbs_simulate(m, batch, gpn, 8 * gpn, quota, 1, 100, sums) for m in range(5)] + [
                lambda: ds.lbs_simulate_all(batch, gpn, 8 * gpn, quota, 1, 100, sums)]:
            fake.fake_fail_host_allocations(1)
            try:
                call()
            finally:
                fake.fake_fail_host_allocations(0)
            names = [k for k, _ in kernels()]
            assert names[0] in ("k_lbs_clear", "k_lbs_clear_all") and len(names) >= 2, names
    # nor does one that refuses the call
    fake.fake_fail_host_allocations(1)
    for call in (lambda: ds.lbs_simulate(7, 16, 8, 64, [6, 3, 2, 5], 1, 100, sums), lambda: ds.lbs_simulate(3, 16, 8, 60, [6, 3, 2, 5], 1, 100, sums),
                 lambda: ds.lbs_simulate_all(16, 8, 64, [6, 3, 2, 4], 1, 100, sums)):
        try:
            call()
        except lbs.LbsError as e:
            refused = e
        fake.fake_fail_host_allocations(0)
        assert refused is not None
        refused = None
        fake.fake_fail_host_allocations(1)
    fake.fake_fail_host_allocations(0)
print("went through")
""")
    assert "went through" in out
