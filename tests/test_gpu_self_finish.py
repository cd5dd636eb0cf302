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
