"""Host code of the compute calls, on a device that only notes what is launched on it (tests/fake_device)."""
import numpy as np
import pytest
import torch

import fake_device
import paper_2402_02447_amd as B
import workloads as W


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


def test_lamb_goes_in_two_sweeps_where_the_parameters_do_not_lie_for_one_pass(device):
    """Which kernels lamb_step and bucket_clip_lamb enqueue: by the share of the elements in tensors whose p, m and v start
    alike but off 16 bytes, and after a second bind that mends or spoils the placement."""
    fake_device.run(device, """
MI, hp = 1 << 20, B.AdamHyper()
def bind(plan, sizes, off):                     # off: per tensor, the element offsets of g, p, m, v
    base = [[(1 << 40) + (k << 36) + (t << 26) + 4 * o[k] for t, o in enumerate(off)] for k in range(4)]
    plan.bind(*base)
def forms(plan):
    plan.lamb_step(hp, 1, 64)
    a = [k for k, _ in kernels()]
    plan.bucket_clip_lamb(64, hp, 1, 0, 64, 64, 64, 64)
    b = [k for k, _ in kernels()]
    one = (a == ["k_lamb", "k_lamb_tail"], b == ["k_lamb", "k_lamb_late", "k_lamb_tail"])
    two = (a == ["k_lamb_moments", "k_lamb_trust", "k_lamb_update"] * len(plan.lamb_runs()),
           b == ["k_step", "k_finish", "k_lamb_trust", "k_lamb_update"])
    assert one[0] != two[0] and one[1] != two[1], (a, b)
    assert (plan.n_lamb_items(False) > 0, plan.n_lamb_items(True) > 0) == one
    return one

aligned, packed, grads, mutual = (0, 0, 0, 0), (1, 1, 1, 1), (1, 0, 0, 0), (0, 1, 2, 3)
sizes = [MI] * 16
plan = B.Plan.from_layout(W.layout_flat_split(sizes, 2 * MI), B.BCA_GRAD_F32)
for n_off in (0, 1, 2, 3, 16):                  # an eighth of the elements is the limit
    bind(plan, sizes, [packed] * n_off + [aligned] * (16 - n_off))
    assert forms(plan) == ((n_off <= 2,) * 2), n_off
for off in (aligned, grads, mutual, (3, 2, 2, 1)):      # these are no obstacle
    bind(plan, sizes, [off] * 16)
    assert forms(plan) == (True, True), off
for off in (packed, (0, 3, 3, 3), (0, 2, 2, 2), (1, 5, 1, 9)):
    bind(plan, sizes, [off] * 16)
    assert forms(plan) == (False, False), off
bind(plan, sizes, [aligned] * 16)
assert forms(plan) == (True, True)
plan.close()
""")


def test_lamb_goes_in_two_sweeps_where_slots_would_idle():
    """Tensors cut into items of few elements, by buckets that end inside them or by their own size, and tensors that take more
    than half the slots with too little beside them: the form of a host-only
    plan (which lies as one whose tensors start on 16 bytes)."""
    MI = 1 << 20
    for sizes, cap, want in [
            ([MI] * 16, 1 << 40, (1, 1)), ([MI] * 16, 50_000, (1, 1)), ([MI] * 16, 20_000, (0, 0)), ([MI] * 16, 5_000, (0, 0)), ([MI] * 16, 1_000, (0, 0)),
            ([1_000] * 16_000, 4 * MI, (1, 1)), ([1_000] * 8_000, 4 * MI, (1, 1)), ([1_500] * 11_000, 4 * MI, (0, 0)), ([2_000] * 8_000, 4 * MI, (0, 0)), ([3_000] * 6_000, 4 * MI, (1, 1)),
            ([9_000] * 2_000, 4 * MI, (1, 1)), ([9_000] * 700, 4 * MI, (0, 1)), ([12_300] * 600, 4 * MI, (0, 1)), ([12_300] * 1_100, 4 * MI, (1, 1)), ([5_000] * 1_100, 4 * MI, (1, 1)),
            ([100_000] * 63, 4 * MI, (1, 1)), ([512 * 12_288] * 6, 1 << 40, (1, 1)), ([513 * 12_288] * 6, 1 << 40, (0, 0)),
            ([8 * MI] * 3 + [MI] * 8, 1 << 40, (1, 1)), ([8 * MI] * 3 + [MI] * 7, 1 << 40, (0, 0)), ([MI] * 14 + [1_500] * 1_200, 1 << 40, (1, 1)), ([MI] * 14 + [1_500] * 1_500, 1 << 40, (0, 0))]:
        lay = W.layout_flat_split(sizes, cap)
        with B.Plan.from_layout(lay, B.BCA_GRAD_F32, device=-1) as plan:
            got = tuple(int(plan.n_lamb_items(clip) > 0) for clip in (False, True))
            assert got == want, (len(sizes), sizes[0], cap, got)
            for clip in (False, True):          # the list, where there is one, has every chunk of the tensor-major table once
                if plan.n_lamb_items(clip) and len(sizes) < 100:
                    seen = np.zeros(plan.n_chunks(B.BCA_TABLE_LAMB), int)
                    for kind, first, count, _, _ in plan.lamb_items(clip):
                        if kind == 1:
                            seen[first:first + count] += 1
                    assert (seen == 1).all()


def test_the_listed_items_of_lamb_are_those_of_the_kernel(device):
    """k_lamb's own item table: every chunk is in it once and at its address, also where workgroups share a run of chunks, and the chunks that
    wait on the chip are those that the plan lists as held.  Tensors that are held, and ones of which only the end is, which begins at an item's
    distance from the last one, wherever that is in a run."""
    fake_device.run(device, """
SPREAD, HELD, ALONE, STATE = 32, 4, 16, np.dtype([("tab", "u8"), ("items", "u8"), ("rest", "u8", 6), ("n", "u4", 4)])
ITEM = np.dtype([("at", "u8", 4), ("first", "u4"), ("count", "u4"), ("tensor", "u4"), ("bucket", "u4"), ("flags", "u4"), ("items", "u4"), ("chunks", "u4", 2)])
fake.fake_watch(b"k_lambI", 1, STATE.itemsize)
split = 0
for sizes, cap in [([n] + [4 << 20] * 8, 1 << 40) for n in (22_050_000, 22_100_000, 22_150_000, 30_000_000)] + [
        ([96 * 1024 * k + r for k in (1, 2, 11, 40) for r in (-1, 0, 1, 60_000)], 3 * 96 * 1024), ([1 << 20] * 20, 300_000)]:
    lay = W.layout_flat_split(sizes, cap)
    plan = B.Plan.from_layout(lay, B.BCA_GRAD_F32)
    base = [[(k + 1 << 44) + (t << 32) for t in range(len(sizes))] for k in range(4)]
    plan.bind(*base)
    chunks = [plan.chunk_info(i, B.BCA_TABLE_LAMB) for i in range(plan.n_chunks(B.BCA_TABLE_LAMB))]
    for clip in (False, True):
        kernels()
        plan.bucket_clip_lamb(64, B.AdamHyper(), 1, 0, 64, 64, 64, 64) if clip else plan.lamb_step(B.AdamHyper(), 1, 64)
        st = np.frombuffer(ctypes.string_at(fake.fake_launch_arg(0), STATE.itemsize), STATE)[0]
        items = np.frombuffer(ctypes.string_at(int(st["items"]), int(st["n"][0]) * ITEM.itemsize), ITEM)
        held, listed = np.full(len(chunks), -1), np.full(len(chunks), -1)
        for it in items:
            stride = 8 if it["flags"] & SPREAD else 1
            split += stride == 8
            for j in range(it["count"]):
                i = int(it["first"]) + j * stride
                assert held[i] == -1 and chunks[i][0] == it["tensor"] and chunks[i][3] == it["bucket"]
                held[i] = (it["flags"] & (HELD if clip else HELD | ALONE)) != 0
            t, begin = chunks[it["first"]][:2]
            assert [int(x) for x in it["at"]] == [base[k][t] + 4 * begin for k in range(4)]
        for kind, first, count, tensor, h in plan.lamb_items(clip):
            if kind == 1:
                assert (listed[first:first + count] == -1).all()
                listed[first:first + count] = h
        assert (held >= 0).all() and (held == listed).all(), (sizes[0], clip, int((held != listed).sum()))
    plan.close()
assert split > 1000
""")


def test_adam_sweeps_of_up_to_two_rounds_of_chunks_start_at_once(device):
    """LDS that the sweeps of adam_step and of the whole-gradient step reserve: 36 KiB, four workgroups a compute unit, but none where the chunks
    are one and an eighth to two rounds of those; what the caller asks for, always."""
    fake_device.run(device, """
def reserved(chunks, **tuning):
    with B.Plan.from_layout(W.layout_flat_split([1024 * chunks - 5], 1 << 40), B.BCA_GRAD_F32, **tuning) as plan:
        plan.bind(*[[k << 40] for k in (1, 2, 3, 4)])
        kernels()
        plan.adam_step(B.AdamHyper(), 1)
        plan.bucket_clip_adam(64, B.AdamHyper(), 1, B.BCA_CLIP_WHOLE_GRADIENT, 64, 64, 64)
        lds = [fake.fake_launch_lds(i) for i in range(fake.fake_num_launches()) if b"k_adam" in fake.fake_launch_name(i)]
        assert len(lds) == 2 and lds[0] == lds[1], lds
        return lds[0]
for cus in (256, 64):
    fake.fake_set_cus(cus)
    for sixteenths, want in ((1, 36), (16, 36), (18, 36), (19, 0), (25, 0), (32, 0), (33, 36), (200, 36)):
        assert reserved(cus * sixteenths // 4) == want << 10, (cus, sixteenths)
    assert reserved(cus * 4 + cus // 2 + 1) == 0 and reserved(cus * 8 + 1) == 36 << 10
    for asked, got in ((1, 0), (20 << 10, 20 << 10), (36 << 10, 36 << 10)):
        assert reserved(cus * 6, adam_lds_reserve=asked) == got
    assert reserved(cus * 6, grid_apply=cus) == 36 << 10 and reserved(cus * 3, chunk_apply=2048) == 36 << 10
""")


def test_runs_by_xcd_are_for_one_workgroup_a_chunk(device):
    """The order that adam_step's sweep is given: runs in plans of 144 Ki chunks and more in the library's own cut; in smaller ones, on a grid
    that the caller gives, and behind whole-gradient norms the table's."""
    fake_device.run(device, """
fake.fake_watch(b"k_adam", 6, 4)
def order(chunks, whole=False, **tuning):
    with B.Plan.from_layout(W.layout_flat_split([1024 * chunks - 5], 1 << 40), B.BCA_GRAD_F32, **tuning) as plan:
        plan.bind(*[[k << 40] for k in (1, 2, 3, 4)])
        kernels()
        if whole:
            plan.bucket_clip_adam(64, B.AdamHyper(), 1, B.BCA_CLIP_WHOLE_GRADIENT, 64, 64, 64)
        else:
            plan.adam_step(B.AdamHyper(), 1)
        i = fake.fake_num_launches() - 1
        assert b"k_adam" in fake.fake_launch_name(i)
        return int.from_bytes(ctypes.string_at(fake.fake_launch_arg(i), 4), "little")
RUNS = 144 << 10
assert [order(n) for n in (1, RUNS - 1, RUNS, RUNS + 5)] == [0, 0, 1, 1]
assert order(RUNS, grid_apply=512) == order(RUNS, grid_apply=500) == order(RUNS, chunk_apply=2048) == order(2 * RUNS, chunk_apply=2048) == 0
assert order(RUNS, whole=True) == order(1, whole=True) == 0
""")


def test_norms_of_a_small_plan_in_one_launch(device):
    """Up to 64 squared-norm chunks and 1 024 buckets, all but a few of them without elements."""
    fake_device.run(device, """
K = 16384
def forms(lay):
    out = []
    with B.Plan.from_layout(lay, B.BCA_GRAD_F32) as plan:
        plan.bind(*[[k << 40] * lay.n_tensors for k in (1, 2, 3, 4)])
        for flags in (B.BCA_CLIP_WHOLE_GRADIENT, B.BCA_CLIP_WHOLE_GRADIENT | B.BCA_SKIP_STEP_ON_NONFINITE, B.BCA_SKIP_STEP_ON_NONFINITE):
            kernels()
            plan.bucket_clip_adam(64, B.AdamHyper(), 1, flags, 64, 64, 64)
            names = [k for k, _ in kernels()]
            assert names in (["k_norms", "k_adam"], ["k_sqnorm", "k_finalize"] + ["k_whole_coef"] * (flags != B.BCA_SKIP_STEP_ON_NONFINITE) + ["k_adam"]), names
            out.append(int(names[0] == "k_norms"))
    return out
flat, each = W.layout_flat_split, W.layout_one_tensor_per_bucket
for lay, want in ((flat([5], 10), 1), (flat([64 * K], 1 << 40), 1), (flat([64 * K + 1], 1 << 40), 0), (each([9000] * 32 + [0] * 992), 1),
                  (each([9000] * 32 + [0] * 993), 0), (each([9000] * 50 + [0] * 20_000), 0)):
    assert forms(lay) == [want] * 3, (lay.n_buckets, want, forms(lay))
""")


def test_lamb_in_one_pass_costs_a_plan_one_allocation(device):
    """Every plan of some size has its tables, also where only Adam is called: they are one block, given back with the plan."""
    fake_device.run(device, """
def allocations(n, **tuning):
    before = fake.fake_device_allocations()
    with B.Plan.from_layout(W.layout_flat_split([1 << 20] * n, 1 << 21), B.BCA_GRAD_F32, **tuning) as plan:
        one = plan.n_lamb_items(True) > 0
    assert fake.fake_device_allocations() - fake.fake_device_frees() == 0
    return fake.fake_device_allocations() - before, one
(small, a), (large, b), (multi, c) = allocations(2), allocations(16), allocations(16, tune_flags=B.BCA_TUNE_MULTI_LAUNCH)
assert (a, b, c) == (False, True, False)
assert large == small + 1 == multi + 1, (small, large, multi)
""")


def test_the_form_whose_table_lies_at_address_zero_is_taken_only_where_it_does(device):
    """All five methods, nodes of 8 in full bins: k_lbs_nodes addresses its first table as if nothing lay in front of it, so a kernel with LDS
    of its own is not launched; one method alone has no such table."""
    fake_device.run(device, """
cum, ends, quota = W.length_histogram_piecewise_uniform(), W.LENGTH_STRATUM_END, [6, 3, 2, 5]
for own, want in ((0, "k_lbs_nodes"), (16, "k_lbs_bins"), (0, "k_lbs_nodes")):
    fake.fake_set_static_lds(own)
    with lbs.Dataset(cum, ends, device=0) as ds:
        kernels()
        ds.lbs_simulate_all(16, 8, 1024, quota, 1, 5000, 4096)
        assert [k for k, _ in kernels()] == ["k_lbs_clear_all", want], own
        ds.lbs_simulate(lbs.LBS_LOCAL_SNAKE, 16, 8, 1024, quota, 1, 5000, 4096)
        assert [k for k, _ in kernels()] == ["k_lbs_clear", "k_lbs_nodes"], own
""")


def test_the_gpu_tests_run_every_form_of_nodes_and_bins(device, monkeypatch):
    """What the GPU tests of the simulation ask for, noted instead of carried out and put to the host code: each k_lbs_nodes and k_lbs_bins
    that the library holds has to be among the kernels that it picks."""
    import test_gpu_lbs_bins as T
    calls = []

    def note(method):
        return lambda cum, ends, *rest, n, seed, first=0: calls.append((cum is T.SPIKE, *((None,) if method else ()), *rest, n))
    monkeypatch.setattr(T, "check", note(False))
    monkeypatch.setattr(T, "check_all", note(True))
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda device: type("Properties", (), {"multi_processor_count": 256}))
    for test in (T.test_quotas_that_fit_in_bins_and_quotas_that_do_not, T.test_full_bins_by_number_of_nodes, T.test_forms_of_full_bins):
        names, values = test.pytestmark[0].args
        for row in values:
            test(**dict(zip(names.split(","), row)))
    out = fake_device.run(device, f"""
plain, spike, picked = W.length_histogram_piecewise_uniform(), np.array({T.SPIKE.tolist()}, np.uint32), set()
for searched, method, batch, gpn, gpus, quota, n in {calls!r}:
    with lbs.Dataset(spike if searched else plain, W.LENGTH_STRATUM_END, device=0) as ds:
        kernels()
        if method is None:
            ds.lbs_simulate_all(batch, gpn, gpus, quota, 1, n, 4096)
        else:
            ds.lbs_simulate(method, batch, gpn, gpus, quota, 1, n, 4096)
        picked |= set(fake.fake_launch_name(i) for i in range(fake.fake_num_launches()))
held = set(fake.fake_kernel_name(i) for i in range(fake.fake_num_kernels()))
for kind, n in ((b"k_lbs_nodes", 20), (b"k_lbs_bins", 12)):
    forms = set(k for k in held if kind in k)
    assert len(forms) == n, (kind, len(forms))
    print(sorted(forms - picked))
""")
    assert out.split() == ["[]", "[]"], out


def test_the_form_of_a_run_is_not_one_that_was_measured_slower(device):
    """Nodes of 4 and 8 on 256 compute units, full bins and a histogram whose cells have to be searched: sizes at which the forms differ, most by a
    tenth and more (us beside them)."""
    out = fake_device.run(device, """
ends, quota = W.LENGTH_STRATUM_END, {(8, 16): [6, 3, 2, 5], (8, 8): [3, 2, 1, 2], (4, 16): [5, 2, 3, 6], (4, 32): [12, 6, 4, 10]}
plain, searched = W.length_histogram_piecewise_uniform(), np.concatenate([[0], np.cumsum((1e6 / (1 + np.arange(512.)) ** 2 + 1).astype(np.int64))])
for cum, cases in ((searched, [
        (8, 8, 30, 12000, False, ["bins 0"]),                   # 154; columns 172
        (8, 16, 16, 12000, False, ["bins 0"]),                  # 156; columns 173
        (8, 16, 64, 12000, False, ["bins 3"])]), (plain, [      # 347; 354
        (4, 16, 30, 30000, True, ["bins 2"]),                   # 116; one node at a time 136, 16 registers 140
        (4, 16, 30, 1700, True, ["bins 0", "bins 2"]),          # 30, 28; 33
        (4, 16, 64, 1700, True, ["bins 2"]),                    # 29; 33, 34
        (4, 16, 64, 16000, True, ["bins 2"]),                   # 111; 128, 125
        (4, 16, 64, 100000, True, ["nodes 4"]),                 # 511; 713, columns 613
        (8, 16, 30, 16000, True, ["bins 3", "nodes 3"]),        # 115, 113; 123, 16 registers 128
        (8, 8, 60, 16000, True, ["bins 3", "nodes 3"]),
        (8, 16, 128, 1000, True, ["nodes 4", "nodes 5"]),       # 26, 23; columns 31
        (8, 16, 20, 1100, False, ["bins 0", "nodes 3"]),        # 25; columns 30
        (8, 8, 30, 1200, False, ["bins 0", "nodes 3"]),
        (8, 16, 128, 100000, False, ["nodes 5"])])):             # 1770; 16 registers 2006
    with lbs.Dataset(cum, ends, device=0) as ds:
      for gpn, batch, nodes, n, alone, good in cases:
        kernels()
        if alone:
            ds.lbs_simulate(lbs.LBS_LOCAL_SNAKE, batch, gpn, gpn * nodes, quota[gpn, batch], 1, n, 4096)
        else:
            ds.lbs_simulate_all(batch, gpn, gpn * nodes, quota[gpn, batch], 1, n, 4096)
        kind, lg = re.search(r"k_lbs_(bins|nodes)ILi(\\d)", fake.fake_launch_name(1).decode()).groups()
        if f"{kind} {lg}" not in good:
            print(gpn, batch, nodes, n, alone, kind, lg)
""")
    assert out == "", out
