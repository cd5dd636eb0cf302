"""Calls that need every norm before any update, in plans small enough for one launch of norms and just too large for it, call after call
against separate launches, bit for bit: values, status words, and what is left in the plan."""
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

HP = B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)
K = 16384                      # elements of a squared-norm chunk
WHOLE, SKIP, WB = B.BCA_CLIP_WHOLE_GRADIENT, B.BCA_SKIP_STEP_ON_NONFINITE, B.BCA_WRITE_BACK_GRADS


def _run(lay, gdt, dtype, flags, spoil, **tuning):
    gen = torch.Generator(device="cuda").manual_seed(7)
    sizes = [int(n) for n in lay.tensor_numel]
    g = [(torch.randn(n, generator=gen, device="cuda") * 1e-2).to(dtype) for n in sizes]
    p, m = ([torch.randn(n, generator=gen, device="cuda") * s for n in sizes] for s in (0.02, 3e-4))
    v = [(torch.rand(n, generator=gen, device="cuda") + 0.5) * 1e-6 for n in sizes]
    plan = B.Plan.from_layout(lay, gdt, **tuning)
    plan.bind(g, p, m, v)
    nb = lay.n_buckets
    norms, coefs, status = torch.zeros(nb + 1, device="cuda"), torch.zeros(nb, device="cuda"), torch.full((1,), -1, dtype=torch.int32, device="cuda")
    thr = torch.full((1 if flags & WHOLE else nb,), 0.5, device="cuda")
    seen = []
    for step in range(1, 6):
        big = max(range(len(sizes)), key=lambda t: sizes[t])
        if spoil and step == 3:
            g[big][sizes[big] // 2] = float("inf")
        if spoil and step == 4:
            g[big][sizes[big] // 2] = 0.01
            thr[-1] = -1.0
        if spoil and step == 5:
            thr[-1] = 0.5
        plan.bucket_clip_adam(thr, HP, step, flags, norms, coefs, status)
        torch.cuda.synchronize()
        seen += [norms.clone(), coefs.clone(), status.clone()]
    plan.close()
    return seen + g + p + m + v


@pytest.mark.parametrize("gdt,dtype", [(B.BCA_GRAD_F32, torch.float32), (B.BCA_GRAD_F16, torch.float16), (B.BCA_GRAD_BF16, torch.bfloat16)])
@pytest.mark.parametrize("flags", [WHOLE, SKIP, WHOLE | SKIP, WHOLE | WB])
@pytest.mark.parametrize("sizes,cap", [([1], 10), ([0, 3], 10), ([5, 0, K, K + 1], 3000), ([64 * K], 1 << 30), ([63 * K, 7], 2 * K + 5), ([64 * K, 1], 1 << 30), ([300_000, 1], 1 << 30)])
def test_same_bits_as_separate_launches(gdt, dtype, flags, sizes, cap):
    lay = W.layout_flat_split(sizes, cap)
    spoil = sizes[0] > 1
    for a, b in zip(_run(lay, gdt, dtype, flags, spoil), _run(lay, gdt, dtype, flags, spoil, tune_flags=B.BCA_TUNE_MULTI_LAUNCH)):
        assert torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


@pytest.mark.parametrize("flags", [WHOLE, SKIP])
def test_buckets_and_plans_without_elements(flags):
    for sizes in ([0, 5, 0, 40_000, 0], [0] * 511 + [9_000, 40_000] + [0] * 511, [0] * 511 + [9_000, 40_000] + [0] * 512):
        lay = W.layout_one_tensor_per_bucket(sizes)
        for a, b in zip(_run(lay, B.BCA_GRAD_F32, torch.float32, flags, False), _run(lay, B.BCA_GRAD_F32, torch.float32, flags, False, tune_flags=B.BCA_TUNE_MULTI_LAUNCH)):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    lay = W.layout_one_tensor_per_bucket([0, 0])
    norms, status = _run(lay, B.BCA_GRAD_F32, torch.float32, flags, False)[0:3:2]
    assert not norms.any() and int(status.item()) == 0


def test_captured_and_replayed():
    lay = W.layout_flat_split([70_001, 5, 33_000], 20_000)
    results = []
    for captured in (False, True):
        gen = torch.Generator(device="cuda").manual_seed(9)
        state = [[torch.randn(int(n), generator=gen, device="cuda") * s for n in lay.tensor_numel] for s in (1e-2, 0.02, 0.0, 0.0)]
        plan = B.Plan.from_layout(lay, B.BCA_GRAD_F32)
        plan.bind(*state)
        norms, coefs, status = torch.zeros(lay.n_buckets + 1, device="cuda"), torch.zeros(lay.n_buckets, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        thr = torch.full((1,), 0.5, device="cuda")
        graph = torch.cuda.CUDAGraph()
        if captured:
            with torch.cuda.graph(graph):
                plan.bucket_clip_adam(thr, HP, 3, WHOLE, norms, coefs, status, stream=torch.cuda.current_stream())
        for _ in range(4):
            graph.replay() if captured else plan.bucket_clip_adam(thr, HP, 3, WHOLE, norms, coefs, status)
            torch.cuda.synchronize()
            results.append([norms.clone(), coefs.clone(), status.clone()] + [x.clone() for ts in state for x in ts])
        plan.close()
    for one, two in zip(results[:4], results[4:]):
        for a, b in zip(one, two):
            assert torch.equal(a, b)
