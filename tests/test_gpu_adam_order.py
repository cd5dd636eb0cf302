"""The Adam sweep's orders of the chunks: the table's, and runs by XCD (adam_step, by the size of the plan); each against a plan whose sweep
is a persistent grid, which takes the table's order, bit for bit."""
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

HP = B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)
FROM = (144 << 10) * 1024     # elements from which adam_step goes in runs (of 8 * 256 chunks)


@pytest.mark.parametrize("op", ["adam", "whole"])
@pytest.mark.parametrize("sizes", [[1], [5, 0, 3000], [2047 * 1024, 1024], [FROM - 1024], [FROM - 1024, 1], [FROM + 2049 * 1024 + 5, 7]])
def test_every_chunk_once_in_any_order(op, sizes):
    lay = W.layout_flat_split(sizes, 6_553_600)
    gen = torch.Generator(device="cuda").manual_seed(3)
    g = [torch.randn(n, generator=gen, device="cuda") * 1e-3 for n in sizes]
    p = [torch.randn(n, generator=gen, device="cuda") * 0.02 for n in sizes]
    results = []
    for tuning in ({}, {"grid_apply": 512}):
        state = [g, [x.clone() for x in p], [torch.zeros_like(x) for x in p], [torch.zeros_like(x) for x in p]]
        plan = B.Plan.from_layout(lay, B.BCA_GRAD_F32, **tuning)
        plan.bind(*state)
        norms, coefs, status = torch.zeros(lay.n_buckets + 1, device="cuda"), torch.zeros(lay.n_buckets, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        for step in (1, 2):
            if op == "adam":
                plan.adam_step(HP, step)
            else:
                plan.bucket_clip_adam(torch.full((1,), 0.5, device="cuda"), HP, step, B.BCA_CLIP_WHOLE_GRADIENT, norms, coefs, status)
        torch.cuda.synchronize()
        results.append([x for ts in state[1:] for x in ts] + [norms, coefs, status])
        plan.close()
    for a, b in zip(*results):
        assert torch.equal(a, b)
