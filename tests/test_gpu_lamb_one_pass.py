"""LAMB in one pass over p, m, v (items held on the chip until their tensor's ratio is known) against the two sweeps, bit for
bit: sizes around chunks, items and the limit up to which a tensor is held, and waits that expire."""
import numpy as np
import pytest
import torch

import paper_2402_02447_amd as B
import workloads as W

pytestmark = pytest.mark.gpu

HP = B.AdamHyper(1e-3, 0.9, 0.999, 1e-6, 0.01)
TYPES = [(torch.float32, B.BCA_GRAD_F32), (torch.float16, B.BCA_GRAD_F16), (torch.bfloat16, B.BCA_GRAD_BF16)]
# edges of a chunk (1024), of an item (12 chunks), several items, an empty tensor, single elements
SIZES = [1, 0, 1023, 1024, 1025, 12 * 1024, 12 * 1024 + 1, 13 * 1024, 24 * 1024, 100_003, 7, 300_000, 2]
SIZES += [5 << 20]     # plans below this many elements go in two sweeps
PATTERN = 7.0          # around the tensors


def _state(sizes, dtype, seed, offset=0):
    """g, p, m, v; `offset`: elements by which they (or, as four numbers, each of them) start off an allocation."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    og, op, om, ov = (offset,) * 4 if isinstance(offset, int) else offset

    def place(t, o):
        buf = torch.full((t.numel() + o + 16,), PATTERN, dtype=t.dtype, device="cuda")
        buf[o:o + t.numel()] = t
        return buf[o:o + t.numel()]
    g = [place((torch.randn(n, generator=gen, device="cuda") * 1e-3).to(dtype), og) for n in sizes]
    p = [place(torch.randn(n, generator=gen, device="cuda") * 0.02, op) for n in sizes]
    m = [place(torch.randn(n, generator=gen, device="cuda") * 3e-4, om) for n in sizes]
    v = [place((torch.rand(n, generator=gen, device="cuda") + 0.5) * 1e-6, ov) for n in sizes]
    return g, p, m, v


def _nothing_outside_touched(state):
    for t in (t for ts in state for t in ts):
        o, n = t.storage_offset(), t.numel()
        buf = torch.empty(0, dtype=t.dtype, device="cuda").set_(t.untyped_storage())
        assert bool((buf[:o] == PATTERN).all()) and bool((buf[o + n:] == PATTERN).all())


class Run:
    def __init__(self, lay, dtype, gdt, seed, offset=0, mask=None, **tuning):
        self.lay, self.state = lay, _state([int(n) for n in lay.tensor_numel], dtype, seed, offset)
        self.plan = B.Plan.from_layout(lay, gdt, **tuning)
        if mask is not None:
            self.plan.set_decay_mask(mask)
        self.plan.bind(*self.state)
        nb = lay.n_buckets
        self.norms, self.coefs = (torch.zeros(nb, device="cuda") for _ in range(2))
        self.trust = torch.full((lay.n_tensors,), -1.0, device="cuda")
        self.status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        self.thr = torch.full((nb,), 0.05, device="cuda")

    def go(self, clip, step, flags=0, stream=None):
        if clip:
            self.plan.bucket_clip_lamb(self.thr, HP, step, flags, self.norms, self.coefs, self.trust, self.status, stream=stream)
        else:
            self.plan.lamb_step(HP, step, self.trust, stream=stream)

    def same(self, other):
        for a, b in zip([x for ts in self.state for x in ts] + [self.trust, self.norms, self.coefs],
                        [x for ts in other.state for x in ts] + [other.trust, other.norms, other.coefs]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


def _two_sweeps(clip):
    return dict(tune_flags=B.BCA_TUNE_MULTI_LAUNCH) if clip else dict(lamb_group_elems=1 << 40)


@pytest.mark.parametrize("dtype,gdt", TYPES)
@pytest.mark.parametrize("clip,flags", [(False, 0), (True, 0), (True, B.BCA_WRITE_BACK_GRADS)])
@pytest.mark.parametrize("cap,offset", [(1 << 30, 0), (262_144, 0), (300_001, (3, 0, 0, 0))])
def test_same_bits_as_two_sweeps(dtype, gdt, clip, flags, cap, offset):
    lay = W.layout_flat_split(SIZES, cap)
    mask = np.arange(len(SIZES)) % 2
    one, two = Run(lay, dtype, gdt, 5, offset, mask), Run(lay, dtype, gdt, 5, offset, mask, **_two_sweeps(clip))
    assert one.plan.n_lamb_items(clip) > 0 and two.plan.n_lamb_items(clip) == 0
    for step in (3, 4):
        one.go(clip, step, flags)
        two.go(clip, step, flags)
        torch.cuda.synchronize()
        one.same(two)
        if clip:
            assert int(one.status.item()) == int(two.status.item()) == 0
    one.plan.close()
    two.plan.close()


@pytest.mark.parametrize("clip", [False, True])
@pytest.mark.parametrize("spin_limit", [0, 1])
def test_tensors_too_large_to_be_held_beside_held_ones(clip, spin_limit):
    """A tensor is held up to three quarters of the resident items.  Whole tensors in a bucket: exactly that many and one more;
    buckets that end inside them, which adds an item or two at every end."""
    most = 4 * torch.cuda.get_device_properties(0).multi_processor_count * 3 // 4          # items
    item = 12 * 1024
    for sizes, cap, held in [([most * item, 5000, 3 << 20, most * item + 1, 70_000, 4 << 20, 12], 1 << 40, [1, 1, 1, 0, 1, 1, 1]),
                             ([5000, most * item + 1, 5 << 20, 5 << 20], 1 << 40, [1, 0, 1, 1]),
                             ([(most - 9) * item, 4 << 20, (most + 1) * item, 40, 4 << 20], 6_553_600, [1, 1, 0, 1, 1])]:
        lay = W.layout_flat_split(sizes, cap)
        one = Run(lay, torch.float32, B.BCA_GRAD_F32, 9, spin_limit=spin_limit)
        two = Run(lay, torch.float32, B.BCA_GRAD_F32, 9, **_two_sweeps(clip))
        items = [i for i in one.plan.lamb_items(clip) if i[0] == 1]
        assert [max((h for _, _, _, t, h in items if t == k)) for k in range(len(sizes))] == held and two.plan.n_lamb_items(clip) == 0
        assert [min((h for _, _, _, t, h in items if t == k)) for k in range(len(sizes))] == held
        for step in (3, 4):
            one.go(clip, step)
            two.go(clip, step)
        torch.cuda.synchronize()
        one.same(two)
        one.plan.close()
        two.plan.close()


@pytest.mark.parametrize("clip", [False, True])
@pytest.mark.parametrize("spin_limit", [0, 1])
@pytest.mark.parametrize("where", [0, 4, 9])
def test_held_ends_of_tensors_that_are_too_large(clip, spin_limit, where):
    """First, in the middle and last in registration order (bucket_clip_lamb's buckets run the other way)."""
    per = torch.cuda.get_device_properties(0).multi_processor_count * 3 * 12 * 1024          # elements that can be held
    sizes = [4 << 20, 5000, 3 << 20, 1_000_001] + [4 << 20] * 5
    sizes.insert(where, 2 * per + 5 * 12 * 1024 + 17)
    lay = W.layout_flat_split(sizes, 6_553_600)
    one = Run(lay, torch.float32, B.BCA_GRAD_F32, 9, spin_limit=spin_limit)
    two = Run(lay, torch.float32, B.BCA_GRAD_F32, 9, **_two_sweeps(clip))
    items = [i for i in one.plan.lamb_items(clip) if i[0] == 1]
    assert two.plan.n_lamb_items(clip) == 0
    assert len({h for _, _, _, t, h in items if t == where}) == (2 if where == 0 or not clip else 1)
    for step in (3, 4):
        one.go(clip, step)
        two.go(clip, step)
    torch.cuda.synchronize()
    one.same(two)
    one.plan.close()
    two.plan.close()


@pytest.mark.parametrize("clip", [False, True])
def test_every_wait_expires_at_a_limit_of_one_poll(clip):
    sizes = [400_000, 5, 1_000_000, 20_000, 4_000_000, 1024]
    lay = W.layout_flat_split(sizes, 262_144)
    one, two = Run(lay, torch.float32, B.BCA_GRAD_F32, 2, spin_limit=1), Run(lay, torch.float32, B.BCA_GRAD_F32, 2, **_two_sweeps(clip))
    assert one.plan.n_lamb_items(clip) > 0 and two.plan.n_lamb_items(clip) == 0
    for step in (3, 4, 5):
        one.go(clip, step)
        two.go(clip, step)
        torch.cuda.synchronize()
        one.same(two)
        if clip:
            assert int(one.status.item()) == B.BCA_STATUS_TIMEOUT
    one.plan.close()
    two.plan.close()


def test_two_plans_on_two_streams_at_once():
    """Each may hold slots that the other's tensors wait for: waits are bounded and the results the same."""
    lay = W.layout_flat_split([4_194_304] * 6 + [1_048_576] * 6, 6_553_600)
    runs = [Run(lay, torch.float32, B.BCA_GRAD_F32, 20 + i) for i in range(2)]
    ref = [Run(lay, torch.float32, B.BCA_GRAD_F32, 20 + i) for i in range(2)]
    assert all(r.plan.n_lamb_items(clip) > 0 for r in runs for clip in (False, True))
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for step in range(3, 13):
        for clip in (False, True):
            for r, s in zip(runs, streams):
                r.go(clip, step, stream=s)
    torch.cuda.synchronize()
    for step in range(3, 13):
        for clip in (False, True):
            for r in ref:
                r.go(clip, step)
                torch.cuda.synchronize()
    for a, b in zip(runs, ref):
        a.same(b)
        a.plan.close()
        b.plan.close()


# gradients off the parameters' alignment (packed views), everything off, p, m and v that differ among themselves: the last
# column says whether that can go in one pass
PLACEMENTS = [((0, 0, 0, 0), True), ((1, 0, 0, 0), True), ((2, 0, 0, 0), True), ((3, 1, 1, 1), False), ((1, 2, 3, 0), True), ((0, 1, 0, 0), True), ((1, 1, 1, 1), False)]


@pytest.mark.parametrize("dtype,gdt", TYPES)
@pytest.mark.parametrize("offset,one_pass", PLACEMENTS)
@pytest.mark.parametrize("clip,flags", [(False, 0), (True, 0), (True, B.BCA_WRITE_BACK_GRADS)])
def test_same_bits_by_every_form_wherever_the_arrays_start(dtype, gdt, offset, one_pass, clip, flags):
    lay = W.layout_flat_split(SIZES, 2 << 20)
    mask = np.arange(len(SIZES)) % 3
    forms = [dict(), dict(spin_limit=1), dict(tune_flags=B.BCA_TUNE_MULTI_LAUNCH), dict(lamb_group_elems=1 << 20)]
    runs = [Run(lay, dtype, gdt, 6, offset, mask, **tuning) for tuning in forms]
    assert [r.plan.n_lamb_items(clip) > 0 for r in runs] == [one_pass, one_pass, False, one_pass and clip]
    for r in runs:
        for step in (3, 4):
            r.go(clip, step, flags)
        torch.cuda.synchronize()
        r.same(runs[0])
        _nothing_outside_touched(r.state)
    for r in runs:
        r.plan.close()


def _ms(call):
    """Shortest of ten after two."""
    out = []
    for i in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call(i + 1)
        b.record()
        torch.cuda.synchronize()
        out.append(a.elapsed_time(b))
    return min(out[2:])


def test_giving_up_every_wait_costs_little_more_than_two_sweeps():
    """Another kernel can hold slots that a tensor waits for, and one expired wait ends all others of the launch.  What is left
    must then not be done by a handful of workgroups (it took 3.2 to 3.7 times the two sweeps with 64 of them, 1.15 to 1.25 now)."""
    lay = W.layout_flat_split([4 << 20] * 6 + [1 << 20] * 16 + [65_536] * 100, 6_553_600)
    late = Run(lay, torch.float32, B.BCA_GRAD_F32, 4, spin_limit=1)
    two = Run(lay, torch.float32, B.BCA_GRAD_F32, 4, lamb_group_elems=32 << 20)
    assert late.plan.n_lamb_items(False) > 0 and two.plan.n_lamb_items(False) == 0
    a, b = _ms(lambda k: late.go(False, k)), _ms(lambda k: two.go(False, k))
    late.same(two)
    assert a < 1.8 * b, (a, b)
    late.plan.close()
    two.plan.close()


@pytest.mark.parametrize("clip", [False, True])
def test_in_a_hip_graph_replays_like_eager_calls(clip):
    """The whole sequence of launches captured, replayed several times with eager work and new gradients in between."""
    sizes = [3_000_000, 70_001, 0, 1024, 2_000_000, 513 * 1024]
    lay = W.layout_flat_split(sizes, 1 << 20)
    graph, eager = Run(lay, torch.bfloat16, B.BCA_GRAD_BF16, 12), Run(lay, torch.bfloat16, B.BCA_GRAD_BF16, 12)
    assert graph.plan.n_lamb_items(clip) > 0
    torch.cuda.synchronize()
    cg, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(cg, stream=s):
        graph.go(clip, 7, stream=torch.cuda.current_stream())
    for k in range(5):
        gen = torch.Generator(device="cuda").manual_seed(100 + k)
        for a, b in zip(graph.state[0], eager.state[0]):
            a.copy_((torch.randn(a.numel(), generator=gen, device="cuda") * 10.0 ** (k - 4)).to(a.dtype))
            b.copy_(a)
        cg.replay()
        torch.cuda.synchronize()
        eager.go(clip, 7)
        torch.cuda.synchronize()
        graph.same(eager)
        if clip:
            assert int(graph.status.item()) == int(eager.status.item()) == 0
    graph.plan.close()
    eager.plan.close()
