"""The fused step with and without a finish kernel behind it: the smallest plans, plans on both sides of the limit (8192 work
items), and waits that all expire, call after call against separate launches, bit for bit."""
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

HP = B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)


def _plan(sizes, cap, seed, **tuning):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = [[torch.randn(n, generator=gen, device="cuda") * s for n in sizes] for s in (1e-2, 0.02, 3e-4)]
    state.append([(torch.rand(n, generator=gen, device="cuda") + 0.5) * 1e-6 for n in sizes])
    lay = W.layout_flat_split(sizes, cap)
    plan = B.Plan.from_layout(lay, B.BCA_GRAD_F32, **tuning)
    plan.bind(*state)
    out = [torch.zeros(lay.n_buckets, device="cuda") for _ in range(2)] + [torch.full((1,), -1, dtype=torch.int32, device="cuda")]
    return plan, state, out, torch.full((lay.n_buckets,), 0.5, device="cuda")


@pytest.mark.parametrize("sizes,cap", [([1], 10), ([0, 3], 10), ([63 * 1024], 1024), ([64 * 1024, 5], 4096), ([70_001, 1000, 1], 3000),
                                       ([7_800_000, 11], 262_144), ([9_000_000, 11], 262_144)])
@pytest.mark.parametrize("flags", [0, B.BCA_WRITE_BACK_GRADS])
@pytest.mark.parametrize("spin_limit", [0, 1])
def test_same_bits_as_separate_launches(sizes, cap, flags, spin_limit):
    plan, state, out, thr = _plan(sizes, cap, 1, spin_limit=spin_limit)
    ref, rstate, rout, _ = _plan(sizes, cap, 1, tune_flags=B.BCA_TUNE_MULTI_LAUNCH)
    if sizes[0] > 1_000_000:
        n = len(plan.work_items())
        assert (n <= 8192) == (sizes[0] < 8_000_000)
    for step in range(1, 6):
        plan.bucket_clip_adam(thr, HP, step, flags, *out)
        ref.bucket_clip_adam(thr, HP, step, flags, *rout)
        torch.cuda.synchronize()
        for a, b in zip([x for ts in state for x in ts] + out[:2], [x for ts in rstate for x in ts] + rout[:2]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
        assert int(rout[2].item()) == 0
        assert int(out[2].item()) in ((0,) if spin_limit == 0 else (0, B.BCA_STATUS_TIMEOUT))
    plan.close()
    ref.close()


def test_status_bits_reach_the_caller_and_do_not_stay():
    plan, state, out, thr = _plan([5000, 70_000], 20_000, 2)
    state[0][1][17] = float("inf")
    plan.bucket_clip_adam(thr, HP, 1, 0, *out)
    assert int(out[2].item()) == B.BCA_STATUS_NONFINITE
    state[0][1][17] = 0.0
    plan.bucket_clip_adam(thr, HP, 2, 0, *out)
    assert int(out[2].item()) == 0
    thr[0] = -1.0
    plan.bucket_clip_adam(thr, HP, 3, 0, *out)
    assert int(out[2].item()) == B.BCA_STATUS_BAD_THRESHOLD
    plan.close()


@pytest.mark.parametrize("dtype,gdt", [(torch.float16, B.BCA_GRAD_F16), (torch.bfloat16, B.BCA_GRAD_BF16), (torch.float32, B.BCA_GRAD_F32)])
@pytest.mark.parametrize("sizes,cap", [([1023, 1024, 2049], 2000), ([300_001, 77], 65_536), ([30_000_000, 5], 1_048_576), ([33_000_000, 5], 1_048_576)])
@pytest.mark.parametrize("flags", [0, B.BCA_WRITE_BACK_GRADS])
def test_items_that_load_before_they_wait(dtype, gdt, sizes, cap, flags):
    """Full and ragged chunks, arrays off the vectors' alignment, exempt tensors, and both sides of the number of work items
    up to which such items exist."""
    gen = torch.Generator(device="cuda").manual_seed(7)
    lay = W.layout_flat_split(sizes, cap)
    thr = torch.full((lay.n_buckets,), 0.5, device="cuda")
    runs = []
    for tuning in ({}, {"tune_flags": B.BCA_TUNE_MULTI_LAUNCH}):
        gen.manual_seed(7)
        state = [[(torch.randn(n + 3, generator=gen, device="cuda") * s)[o:o + n] for n in sizes] for s, o in ((1e-2, 0), (0.02, 1), (3e-4, 2))]
        state.append([(torch.rand(n + 3, generator=gen, device="cuda").add_(0.5) * 1e-6)[:n] for n in sizes])
        state[0] = [torch.cat([x[:1], x]).to(dtype)[1:] for x in state[0]]
        plan = B.Plan.from_layout(lay, gdt, **tuning)
        plan.set_decay_mask([i % 2 for i in range(len(sizes))])
        plan.bind(*state)
        out = [torch.zeros(lay.n_buckets, device="cuda") for _ in range(2)] + [torch.full((1,), -1, dtype=torch.int32, device="cuda")]
        if sizes[0] > 20_000_000:
            assert (len(plan.work_items()) <= 32768) == (sizes[0] == 30_000_000)
        for step in range(1, 4):
            plan.bucket_clip_adam(thr, HP, step, flags, *out)
        torch.cuda.synchronize()
        assert int(out[2].item()) == 0
        runs.append(([x.clone() for ts in state for x in ts] + out[:2], plan))
    for a, b in zip(runs[0][0], runs[1][0]):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    for _, plan in runs:
        plan.close()


@pytest.mark.parametrize("sizes,cap,items", [([120 * 1024], 1 << 30, 128), ([121 * 1024], 1 << 30, 129), ([16_384, 1], 16_384, None), ([16_385], 1 << 30, None),
                                             ([16_383, 0, 5], 16_383, None), ([40_000, 16_384, 3], 16_384, None), ([1, 1, 1], 1, 6)])
@pytest.mark.parametrize("spin_limit", [0, 1])
def test_buckets_of_one_chunk_and_launches_of_few_items(sizes, cap, items, spin_limit):
    """Buckets of one squared-norm chunk (16 384 elements), one more, one less; launches on both sides of 128 work items."""
    plan, state, out, thr = _plan(sizes, cap, 3, spin_limit=spin_limit)
    ref, rstate, rout, _ = _plan(sizes, cap, 3, tune_flags=B.BCA_TUNE_MULTI_LAUNCH)
    assert items is None or len(plan.work_items()) == items
    for step in range(1, 6):
        plan.bucket_clip_adam(thr, HP, step, 0, *out)
        ref.bucket_clip_adam(thr, HP, step, 0, *rout)
        if step == 3:      # the next calls: a threshold that is none, a gradient that is infinite
            thr[-1] = 0.0
            for s in (state, rstate):
                s[0][0][0] = float("inf")
        torch.cuda.synchronize()
        for a, b in zip([x for ts in state for x in ts] + out[:2], [x for ts in rstate for x in ts] + rout[:2]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
        want = int(rout[2].item())
        assert want == (0 if step <= 3 else B.BCA_STATUS_NONFINITE | B.BCA_STATUS_BAD_THRESHOLD)
        assert int(out[2].item()) in ((want,) if spin_limit == 0 else (want, want | B.BCA_STATUS_TIMEOUT))
    plan.close()
    ref.close()


@pytest.mark.parametrize("sizes,cap", [([1000, 17_000], 8192), ([120 * 1024], 1 << 30), ([118 * 1024 + 5], 1 << 30), ([300_001, 77], 65_536),
                                       ([8_500_000, 3], 1_048_576), ([33_000_000], 1_048_576)])
@pytest.mark.parametrize("flags", [0, B.BCA_WRITE_BACK_GRADS])
@pytest.mark.parametrize("spin_limit", [0, 1])
def test_hyper_parameters_in_device_memory_with_items_that_load_early(sizes, cap, flags, spin_limit):
    """Hyper-parameters in device memory, changed between replays of a captured step, against separate launches with k_hyper in front."""
    plan, state, out, thr = _plan(sizes, cap, 4, spin_limit=spin_limit)
    ref, rstate, rout, _ = _plan(sizes, cap, 4, tune_flags=B.BCA_TUNE_MULTI_LAUNCH)
    dev = torch.frombuffer(bytearray(B.pack_device_hyper(HP, 1)), dtype=torch.int64).cuda()
    for p in (plan, ref):
        p.set_device_hyper(dev)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.bucket_clip_adam(thr, None, 0, flags, *out, stream=torch.cuda.current_stream())
    for step in range(1, 7):
        hp = B.AdamHyper(1e-3 / step, 0.9 - 0.1 * (step % 2), 0.999, 1e-6, 0.01 * step)
        dev.copy_(torch.frombuffer(bytearray(B.pack_device_hyper(hp, 3 * step)), dtype=torch.int64))
        if step % 3:
            graph.replay()
        else:
            plan.bucket_clip_adam(thr, None, 0, flags, *out)
        ref.bucket_clip_adam(thr, None, 0, flags, *rout)
        torch.cuda.synchronize()
        for a, b in zip([x for ts in state for x in ts] + out[:2], [x for ts in rstate for x in ts] + rout[:2]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), step
        assert int(out[2].item()) in ((0,) if spin_limit == 0 else (0, B.BCA_STATUS_TIMEOUT))
    plan.adam_step(None, 0)                       # and a call that has the constants derived in front of it
    ref.adam_step(None, 0)
    torch.cuda.synchronize()
    for a, b in zip([x for ts in state for x in ts], [x for ts in rstate for x in ts]):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    plan.close()
    ref.close()
