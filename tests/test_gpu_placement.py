"""Arrays that start anywhere: every combination of element offsets gives the bits of arrays that start on
16-byte boundaries, where the arithmetic is element by element, and the oracle's norms."""
import numpy as np
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

# edges of the vector (4, 8 elements), of the fine cut (1024) and of the squared-norm cut (16384)
SIZES = [1, 3, 4, 5, 7, 8, 9, 1023, 1024, 1025, 2051, 16383, 16384, 16385, 40003]
OFFSETS = [(1, 0, 0, 0), (2, 0, 0, 0), (3, 1, 1, 1), (1, 2, 3, 0), (0, 1, 0, 0), (5, 3, 3, 3)]
HP = B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)


def _arrays(dtype, seed):
    gen = torch.Generator().manual_seed(seed)
    g = [(torch.randn(n, generator=gen) * 1e-2).to(dtype) for n in SIZES]
    p, m = ([torch.randn(n, generator=gen) * s for n in SIZES] for s in (0.02, 3e-4))
    v = [(torch.rand(n, generator=gen) + 0.5) * 1e-6 for n in SIZES]
    return g, p, m, v


def _placed(ts, offset):
    """On the GPU, each tensor `offset` elements into an allocation that is filled with a pattern on both sides."""
    out = []
    for t in ts:
        buf = torch.full((t.numel() + offset + 16,), 7.0, dtype=t.dtype, device="cuda")
        buf[offset:offset + t.numel()].copy_(t)
        out.append((buf, buf[offset:offset + t.numel()]))
    return out


def _run(op, dtype, gdt, offsets, cap=5000):
    lay = W.layout_flat_split(SIZES, cap)
    placed = [_placed(ts, o) for ts, o in zip(_arrays(dtype, 3), offsets)]
    g, p, m, v = ([view for _, view in ts] for ts in placed)
    plan = B.Plan.from_layout(lay, gdt)
    plan.bind(g, p, m, v)
    thr = torch.full((lay.n_buckets,), 0.3, device="cuda")
    norms, coefs = (torch.zeros(lay.n_buckets, device="cuda") for _ in range(2))
    if op == "adam":
        plan.adam_step(HP, 10)
    elif op == "step":
        plan.bucket_clip_adam(thr, HP, 10, B.BCA_WRITE_BACK_GRADS, norms, coefs)
    elif op == "clip":
        plan.bucket_clip(0, lay.n_buckets, thr, norms, coefs)
    elif op == "two_calls":
        plan.bucket_clip_norms(0, lay.n_buckets, norms)
        plan.bucket_clip_apply(0, lay.n_buckets, thr, norms, coefs)
    else:
        plan.lamb_step(HP, 10)
    torch.cuda.synchronize()
    for ts, o in zip(placed, offsets):      # nothing outside the tensors was touched
        for buf, view in ts:
            assert bool((buf[:o] == 7).all()) and bool((buf[o + view.numel():] == 7).all())
    out = [x.cpu() for ts in (g, p, m, v) for x in ts] + [norms.cpu(), coefs.cpu()]
    plan.close()
    return out


@pytest.mark.parametrize("dtype,gdt", [(torch.float32, B.BCA_GRAD_F32), (torch.float16, B.BCA_GRAD_F16),
                                       (torch.bfloat16, B.BCA_GRAD_BF16)])
@pytest.mark.parametrize("op", ["adam", "step", "clip", "two_calls", "lamb"])
def test_offsets_do_not_change_results(op, dtype, gdt):
    want = _run(op, dtype, gdt, (0, 0, 0, 0))
    for offsets in OFFSETS:
        got = _run(op, dtype, gdt, offsets)
        for a, b in zip(got, want):
            if op == "lamb":      # the trust ratio's fp32 partial sums of at most 1024 squares are grouped differently
                np.testing.assert_allclose(a.float().numpy(), b.float().numpy(), rtol=1e-5, atol=1e-9)
            else:                 # a chunk's elements go to the same lanes wherever it starts
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (op, offsets)


@pytest.mark.parametrize("dtype,gdt", [(torch.float16, B.BCA_GRAD_F16), (torch.bfloat16, B.BCA_GRAD_BF16), (torch.float32, B.BCA_GRAD_F32)])
@pytest.mark.parametrize("op", ["clip", "two_calls", "step"])
def test_whole_squared_norm_chunks_wherever_they_start(op, dtype, gdt):
    """Buckets that leave chunks of 16 384 elements whole: 16-bit ones off 32-bit words go by a path of their own."""
    want = _run(op, dtype, gdt, (0, 0, 0, 0), cap=1 << 20)
    for o in (1, 2, 3, 5, 7, 9, 15):
        got = _run(op, dtype, gdt, (o, 0, 0, 0), cap=1 << 20)
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), o
