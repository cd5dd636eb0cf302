"""The stand-alone Adam sweep (adam_step, and behind whole-gradient norms) carries out every chunk exactly once, in the table's order and in runs by
XCD (adam_step, by the size of the plan): one workgroup a chunk, a persistent grid, which takes the table's order, and one that stages the chunk
table in LDS (a loop of its own), the same bits, and first moments that say how often an element was updated."""
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

HP = B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)
FROM = (144 << 10) * 1024     # elements from which adam_step goes in runs (of 8 * 256 chunks)


@pytest.mark.parametrize("op", ["adam", "whole"])
@pytest.mark.parametrize("sizes", [[1], [5, 0, 3000], [2047 * 1024, 1024], [FROM - 1024], [FROM - 1024, 1], [FROM + 1024 * 2047, 1], [FROM + 2049 * 1024 + 5, 7]])
def test_every_chunk_once_in_any_order(op, sizes):
    lay = W.layout_flat_split(sizes, 6_553_600)
    gen = torch.Generator(device="cuda").manual_seed(3)
    g = [torch.randn(n, generator=gen, device="cuda") * 1e-3 for n in sizes]
    p = [torch.randn(n, generator=gen, device="cuda") * 0.02 for n in sizes]
    results = []
    for tuning in ({}, {"grid_apply": 512}, {"grid_apply": 500, "tune_flags": B.BCA_TUNE_STAGE_TABLE_LDS}):
        state = [g, [x.clone() for x in p], [torch.zeros_like(x) for x in p], [torch.zeros_like(x) for x in p]]
        plan = B.Plan.from_layout(lay, B.BCA_GRAD_F32, **tuning)
        plan.bind(*state)
        norms, coefs, status = torch.zeros(lay.n_buckets + 1, device="cuda"), torch.ones(lay.n_buckets, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        for step in (1, 2):
            if op == "adam":
                plan.adam_step(HP, step)
            else:
                plan.bucket_clip_adam(torch.full((1,), 0.5, device="cuda"), HP, step, B.BCA_CLIP_WHOLE_GRADIENT, norms, coefs, status)
            # m = (1 - b1) coef g, then that once more: three roundings of 2^-24 at most in the first, six in the second
            for x, m in zip(g, state[2]):
                want = (1 - 0.9) * (1 if step == 1 else 1.9) * coefs[0].double() * x.double()
                assert bool(((m.double() - want).abs() <= 4e-7 * want.abs() + 1e-40).all()), (tuning, step)
        torch.cuda.synchronize()
        results.append([x for ts in state[1:] for x in ts] + [norms, coefs, status])
        plan.close()
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert torch.equal(a, b)
