"""bucket_clip and bucket_clip_flat on buckets of at most one chunk (16 384 elements), which take one launch, and of a little more, which take
two: against separate launches, bit for bit, call after call."""
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _memory_given_back():
    """Uninitialised memory of later tests is not this file's random bits read as another type."""
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


TYPES = [(torch.float32, B.BCA_GRAD_F32), (torch.float16, B.BCA_GRAD_F16), (torch.bfloat16, B.BCA_GRAD_BF16)]


@pytest.mark.parametrize("dtype,gdt", TYPES)
@pytest.mark.parametrize("n", [1, 3, 8, 255, 1024, 2049, 8192, 16_383, 16_384, 16_385])
@pytest.mark.parametrize("offset", [0, 1, 6])
@pytest.mark.parametrize("threshold", [1e-3, 1e9, -1.0])
def test_same_bits_as_separate_launches(dtype, gdt, n, offset, threshold):
    gen = torch.Generator(device="cuda").manual_seed(n)
    base = (torch.randn(n + 16, generator=gen, device="cuda") * 1e-2).to(dtype)
    lay = W.layout_flat_split([n], 1 << 30)
    results = []
    for kind in ("separate", "bucket_clip", "flat"):
        buf = base.clone()
        g = buf[offset:offset + n]
        rest = [[torch.zeros(n, device="cuda")] for _ in range(3)]
        out, status = torch.full((2,), -1.0, device="cuda"), torch.full((1,), -1, dtype=torch.int32, device="cuda")
        thr = torch.full((1,), threshold, device="cuda")
        plan = B.Plan.from_layout(lay, gdt, **(dict(tune_flags=B.BCA_TUNE_MULTI_LAUNCH) if kind == "separate" else {}))
        plan.bind([g], *rest)
        for _ in range(2):
            thr.mul_(0.5)
            if kind == "flat":
                B.bucket_clip_flat(g, n, gdt, thr, out[0:1], out[1:2], status)
            else:
                plan.bucket_clip(0, 1, thr, out[0:1], out[1:2], status)
            torch.cuda.synchronize()
            results.append([buf.clone(), out.clone(), status.clone()])
        plan.close()
    for other in (results[2:4], results[4:6]):
        for one, two in zip(results[:2], other):
            for a, b in zip(one, two):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def test_one_bucket_among_others_and_none():
    """Buckets of one chunk in the middle of a plan; a range of several goes by two launches."""
    lay = W.layout_one_tensor_per_bucket([5000, 16_384, 0, 40_000, 12])
    results = []
    for tuning in ({}, dict(tune_flags=B.BCA_TUNE_MULTI_LAUNCH)):
        gen = torch.Generator(device="cuda").manual_seed(1)
        state = [[torch.randn(int(n), generator=gen, device="cuda") for n in lay.tensor_numel] for _ in range(4)]
        plan = B.Plan.from_layout(lay, B.BCA_GRAD_F32, **tuning)
        plan.bind(*state)
        norms, coefs, status = torch.zeros(5, device="cuda"), torch.zeros(5, device="cuda"), torch.zeros(5, dtype=torch.int32, device="cuda")
        thr = torch.tensor([1.0, 2.0, 3.0, 4.0, -1.0], device="cuda")
        for b in range(5):
            plan.bucket_clip(b, b + 1, thr, norms, coefs, status[b:b + 1])
        plan.bucket_clip(0, 2, thr, norms, coefs, status[0:1])
        torch.cuda.synchronize()
        results.append(state[0] + [norms, coefs, status])
        plan.close()
    for a, b in zip(*results):
        assert torch.equal(a, b)
    assert results[0][-1].tolist() == [0, 0, 0, 0, B.BCA_STATUS_BAD_THRESHOLD]
