"""LAMB in one pass where workgroups take every eighth chunk of a run of 96: tensors and buckets that end just before, at and behind such
runs, waits that expire, and a tensor that is swept chunk by chunk, against the two sweeps, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W
from test_gpu_lamb_one_pass import TYPES, Run, _two_sweeps

pytestmark = pytest.mark.gpu

RUN = 96 * 1024
SIZES = [RUN, RUN - 1, RUN + 1, RUN - 1024, RUN + 1024, 2 * RUN, 2 * RUN + 13 * 1024 + 5, 5, 95 * 1024, 11 * RUN + 60_000, 40 * RUN]


@pytest.mark.parametrize("dtype,gdt", TYPES)
@pytest.mark.parametrize("clip,flags,spin_limit", [(False, 0, 0), (False, 0, 1), (True, 0, 0), (True, B.BCA_WRITE_BACK_GRADS, 0), (True, 0, 1)])
@pytest.mark.parametrize("cap", [1 << 30, 3 * RUN, 3 * RUN - 1024, 262_144 + 7])
def test_runs_that_end_with_the_tensor_and_with_the_bucket(dtype, gdt, clip, flags, spin_limit, cap):
    lay = W.layout_flat_split(SIZES, cap)
    mask = np.arange(len(SIZES)) % 2
    one, two = Run(lay, dtype, gdt, 5, 0, mask, spin_limit=spin_limit), Run(lay, dtype, gdt, 5, 0, mask, **_two_sweeps(clip))
    for r in (one, two):      # one tensor's parameters and moments one element off: swept chunk by chunk
        for ts in r.state[1:]:
            buf = torch.empty(SIZES[5] + 1, device="cuda")
            buf[1:] = ts[5]
            ts[5] = buf[1:]
        r.plan.bind(*r.state)
    assert one.plan.n_lamb_items(clip) > 0 and two.plan.n_lamb_items(clip) == 0
    for step in (3, 4):
        one.go(clip, step, flags)
        two.go(clip, step, flags)
        torch.cuda.synchronize()
        one.same(two)
    one.plan.close()
    two.plan.close()


@pytest.mark.parametrize("clip,flags", [(False, 0), (True, 0), (True, B.BCA_WRITE_BACK_GRADS)])
@pytest.mark.parametrize("large", [22_050_000, 30_000_001])
def test_a_run_in_which_the_held_end_of_a_tensor_begins(clip, flags, large):
    """A tensor of which the last 768 items are held, the first of them amid a run; its other items keep their moments cached, full ones and
    those at the ends of its buckets."""
    lay = W.layout_flat_split([large] + [4 << 20] * 8, 1 << 30 if large & 1 else 3 * RUN + 5)
    one, two = Run(lay, *TYPES[0], 5), Run(lay, *TYPES[0], 5, **_two_sweeps(clip))
    held = [h for kind, _, _, t, h in one.plan.lamb_items(clip) if kind == 1 and t == 0]
    assert sum(held) == 768 and len(held) > 2 * 768 and two.plan.n_lamb_items(clip) == 0
    for step in (3, 4):
        one.go(clip, step, flags)
        two.go(clip, step, flags)
        torch.cuda.synchronize()
        one.same(two)
    one.plan.close()
    two.plan.close()
