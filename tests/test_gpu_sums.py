"""Every lane's share is in a workgroup's sum exactly once: one element of a chunk is not zero, each of the 1 024 in turn."""
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

N = 1024


@pytest.mark.parametrize("dtype,gdt", [(torch.float32, B.BCA_GRAD_F32), (torch.float16, B.BCA_GRAD_F16), (torch.bfloat16, B.BCA_GRAD_BF16)])
def test_norm_of_one_element(dtype, gdt):
    """Bucket i holds a power of two at place i (squares, sums and roots of those are exact)."""
    value = torch.pow(2.0, (torch.arange(N, device="cuda") % 9) - 4.0)
    g = [torch.diag(value).reshape(-1).to(dtype)]
    rest = [[torch.zeros(N * N, device="cuda")] for _ in range(3)]
    plan = B.Plan.from_layout(W.layout_flat_split([N * N], N), gdt)
    plan.bind(g, *rest)
    norms, coefs, status = torch.zeros(N, device="cuda"), torch.zeros(N, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    plan.bucket_clip_norms(0, N, norms)
    want = value.flip(0) if plan.chunk_info(0, B.BCA_TABLE_APPLY)[1] != 0 else value      # buckets run from the stream's end or its start
    torch.cuda.synchronize()
    assert torch.equal(norms, want)
    norms.zero_()
    plan.bucket_clip_adam(torch.full((N,), 1e9, device="cuda"), B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.0), 1, 0, norms, coefs, status)
    torch.cuda.synchronize()
    assert torch.equal(norms, want) and int(status.item()) == 0
    plan.close()


def test_trust_ratio_of_one_element():
    """Tensor i has its parameter at place i and its moments, the same in every tensor, at another: the ratios are in the proportion of
    the parameters, which are powers of two."""
    i = torch.arange(N, device="cuda")
    value = torch.pow(2.0, (i % 9) - 4.0)
    p, m, v = (torch.zeros(N, N, device="cuda") for _ in range(3))
    p[i, i] = value
    at = (i * 5 + 3) % N
    m[i, at], v[i, at] = 3e-4, 1e-6
    state = [[x[t] for t in range(N)] for x in (torch.zeros(N, N, device="cuda"), p, m, v)]
    plan = B.Plan.from_layout(W.layout_flat_split([N] * N, 1 << 20), B.BCA_GRAD_F32)
    plan.bind(*state)
    trust = torch.zeros(N, device="cuda")
    plan.lamb_step(B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.0), 7, trust)
    torch.cuda.synchronize()
    assert float(trust[0]) > 0 and torch.equal(trust, trust[0] * (value / value[0]))
    plan.close()
