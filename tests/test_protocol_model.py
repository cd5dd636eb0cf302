"""A host-side model of the fused step's waiting scheme, run on the work list the library really builds (CPU only).

The kernels cannot be run here, and no GPU test may force the hardware to start workgroups in a bad order.  What can
be checked on the CPU is the scheme itself: the rules by which the items of one launch arrive, wait, give up and are
completed by the finish kernel are restated below as a small discrete-event model (written from the description in
bca.h and the kernels' comments; it shares no code with them), and that model is driven with the plan's own work
list under start orders and residency limits chosen to be as bad as possible: reversed, random, one workgroup at
a time, every slot taken by Adam items whose squared norms have not started.

Claims checked for every schedule: the launch ends (no order lets waiting items block the items they wait for, once
waits are bounded); every squared-norm chunk is summed once and every bucket finalized once; every Adam chunk is carried
out exactly once, either by its own item or by the finish kernel; an Adam item never runs before its bucket's
coefficient exists; the skipped list never holds more than one entry per Adam chunk; the state the next call starts
from (arrival counters, abort word, skipped count, epoch) is what a first call finds.  With unbounded waits the same
model deadlocks under the bad schedules, which shows that the model is able to see the problem the bound removes.
The same is done for the launch that finishes itself, and for LAMB in one pass, whose items also wait for items behind them in the list."""
import numpy as np
import pytest

import paper_2402_02447_amd as B
import workloads as W

N, A, E = 0, 1, 2        # item kinds as bca_plan_work_item reports them


def host_plan(lay, **tuning):
    return B.Plan.from_layout(lay, B.BCA_GRAD_F32, device=-1, **tuning)


class Model:
    """State of one plan across calls, and one launch of the step kernel plus its finish kernel."""

    def __init__(self, plan, n_buckets):
        self.items = plan.work_items()
        nN, nA = plan.n_chunks(B.BCA_TABLE_NORM), plan.n_chunks(B.BCA_TABLE_APPLY)
        self.bucket_of_norm = [plan.chunk_info(i, B.BCA_TABLE_NORM)[3] for i in range(nN)]
        self.bucket_of_apply = [plan.chunk_info(i, B.BCA_TABLE_APPLY)[3] for i in range(nA)]
        self.total = [plan.bucket_chunks(b, B.BCA_TABLE_NORM)[1] for b in range(n_buckets)]
        self.nb, self.nN, self.nA = n_buckets, nN, nA
        # what lives in device memory between calls
        self.arrived = [0] * n_buckets
        self.ready_epoch = [0] * n_buckets
        self.epoch, self.abort, self.skipped = 1, 0, []

    def launch(self, order, slots, spin_limit, norm_ticks=3, max_ticks=10_000_000):
        """Workgroups start in `order` (a permutation of the item indices) as slots become free; at most `slots` are
        resident.  A resident squared-norm item needs `norm_ticks` ticks, then arrives; a resident Adam item looks at
        its bucket's ready word once per tick.  spin_limit None = wait for ever.  Returns False on deadlock."""
        epoch = self.epoch
        summed = np.zeros(self.nN, int)
        applied = np.zeros(self.nA, int)
        finalized = np.zeros(self.nb, int)
        timed_out = False
        resident = []                                   # [item index, ticks or polls so far]
        nxt, tick = 0, 0
        while nxt < len(order) or resident:
            tick += 1
            if tick > max_ticks:
                return None
            while nxt < len(order) and len(resident) < slots:
                resident.append([order[nxt], 0])
                nxt += 1
            progressed = False
            still = []
            for w in resident:
                kind, first, count = self.items[w[0]]
                if kind == A:
                    b = self.bucket_of_apply[first]
                    if self.ready_epoch[b] == epoch:
                        applied[first] += 1             # coefficient exists: carry out and leave
                        progressed = True
                        continue
                    w[1] += 1
                    if (spin_limit is not None and w[1] > spin_limit) or self.abort:
                        self.abort, timed_out = 1, True
                        self.skipped.append(first)
                        progressed = True
                        continue
                    still.append(w)
                else:
                    w[1] += 1
                    progressed = True                   # squared-norm items never wait
                    if kind == N and w[1] < norm_ticks:
                        still.append(w)
                        continue
                    b = self.bucket_of_norm[first] if kind == N else first
                    if kind == N:
                        summed[first:first + count] += 1
                        self.arrived[b] += count
                        last = self.arrived[b] == self.total[b]
                    else:
                        last = True                     # a bucket without elements: its stand-in finalizes at once
                    if last:
                        self.arrived[b] = 0
                        finalized[b] += 1
                        self.ready_epoch[b] = epoch
            resident = still
            if not progressed and spin_limit is None and (nxt >= len(order) or len(resident) >= slots):
                return False                            # everybody resident waits for ever and nobody else can start
        # the finish kernel: one workgroup, after the launch has ended
        assert len(self.skipped) <= self.nA
        for first in self.skipped:
            assert self.ready_epoch[self.bucket_of_apply[first]] == epoch, "a skipped item whose coefficient is missing"
            applied[first] += 1
        self.skipped, self.abort = [], 0
        self.epoch = epoch + 1 if epoch + 1 < 2 ** 32 else 1
        return dict(summed=summed, applied=applied, finalized=finalized, timed_out=timed_out, ticks=tick)

    def check(self, r):
        assert r, "the launch did not end"
        assert np.all(r["summed"] == 1), "a squared-norm chunk summed twice or not at all"
        assert np.all(r["finalized"] == 1), "a bucket finalized twice or not at all"
        assert np.all(r["applied"] == 1), "an Adam chunk carried out twice or not at all"
        assert self.arrived == [0] * self.nb and self.abort == 0 and self.skipped == []


def small_plan(**tuning):
    numels = W.scaled_bert_numels(32, 2, 128, vocab=500, max_pos=16) + [0, 7, 1, 9_000]
    lay = W.layout_flat_split(numels, 12_000)
    return host_plan(lay, chunk_norm=1024, **tuning), lay


def orders(m, rng):
    n = len(m.items)
    ident = list(range(n))
    yield "in order", ident
    yield "reversed", ident[::-1]
    yield "random", [int(i) for i in rng.permutation(n)]
    yield "adam first", adam_first(m)


def adam_first(m):
    """Every Adam item before any squared-norm item."""
    return sorted(range(len(m.items)), key=lambda i: (m.items[i][0] != A, i))


@pytest.mark.parametrize("tuning", [{}, {"norm_lead": 2}, {"norm_item_chunks": 4, "group_bytes": 1}])
def test_every_schedule_ends_and_every_chunk_is_done_once(tuning):
    plan, lay = small_plan(**tuning)
    rng = np.random.default_rng(5)
    m = Model(plan, lay.n_buckets)
    n = len(m.items)
    assert m.nA > 50 and m.nN > 20 and lay.n_buckets >= 5
    for name, order in orders(m, rng):
        for slots in (1, 2, 7, 64, n):
            for spin in (1, 5, 200):
                r = m.launch(order, slots, spin)
                m.check(r)
                # in the intended order with room for everything nobody waits long enough to give up
                if name == "in order" and spin == 200:
                    assert not r["timed_out"], (name, slots)
    # the state carries over: the epoch has moved once per call, and an old ready word is never taken for a new one
    assert m.epoch == 1 + 4 * 5 * 3


def test_in_order_start_never_times_out_whatever_the_residency():
    """When workgroups start in list order, everything an Adam item waits for has already been started, so it is
    resident or done: the wait is bounded by the squared-norm items' own duration and no bound is needed."""
    plan, lay = small_plan()
    m = Model(plan, lay.n_buckets)
    for slots in (1, 3, 16, 1000):
        r = m.launch(list(range(len(m.items))), slots, spin_limit=None)
        m.check(r)
        assert not r["timed_out"]


def test_without_the_bound_a_bad_order_deadlocks_in_the_model():
    """The model sees the problem that the bounded wait removes: Adam items that take every slot before their squared
    norms have started wait for ever."""
    plan, lay = small_plan()
    m = Model(plan, lay.n_buckets)
    assert m.launch(adam_first(m), slots=8, spin_limit=None) is False
    m2 = Model(plan, lay.n_buckets)
    m2.check(m2.launch(adam_first(m2), slots=8, spin_limit=3))


def test_an_old_ready_word_is_not_taken_for_this_calls():
    """Second call on the same plan, Adam items first: the ready words still hold the previous epoch and must not let
    an Adam item through before this call's squared norms exist (the model's applied-before-finalized check is the
    epoch comparison itself, so plant the mistake and see the model object to it)."""
    plan, lay = small_plan()
    m = Model(plan, lay.n_buckets)
    n = len(m.items)
    m.check(m.launch(list(range(n)), 64, 50))
    stale = list(m.ready_epoch)
    r = m.launch(adam_first(m), 8, 2)
    m.check(r)
    assert r["timed_out"]                                    # they had to wait: the old words did not count
    assert all(e == 1 for e in stale) and all(e == 2 for e in m.ready_epoch)


class SelfFinishing(Model):
    """The same launch without a finish kernel behind it: a workgroup is counted once its item is decided (squared norms
    published, or the wait ended and what it filed in place), and the one that completes the count finishes the call."""

    def launch(self, order, slots, spin_limit, norm_ticks=3):
        epoch, n = self.epoch, len(self.items)
        summed, applied, finalized = np.zeros(self.nN, int), np.zeros(self.nA, int), np.zeros(self.nb, int)
        words = [0] * 64                                # spread over 64 words as the kernel does, one more for the full ones
        full, finished, timed_out = 0, 0, False
        resident, running, nxt, tick = [], [], 0, 0     # running: items whose wait has ended and that still work

        def decided(i):
            """Counts workgroup i; carries out what was given up if it is the last."""
            nonlocal full, finished
            slot = i % 64
            words[slot] += 1
            if words[slot] != n // 64 + (1 if slot < n % 64 else 0):
                return
            words[slot], full = 0, full + 1
            if full != min(n, 64):
                return
            full, finished = 0, finished + 1
            assert not resident_waiting(), "finished while an item still waits"
            for first in self.skipped:
                assert self.ready_epoch[self.bucket_of_apply[first]] == epoch, "a skipped item whose coefficient is missing"
                applied[first] += 1
            self.skipped, self.abort = [], 0
            self.epoch = epoch + 1

        def resident_waiting():
            return any(w[0] is not None for w in resident)

        while nxt < n or resident or running:
            tick += 1
            running = [(f, k - 1) for f, k in running if k > 1]     # done: nothing left to say
            while nxt < n and len(resident) + len(running) < slots:
                resident.append([order[nxt], 0])
                nxt += 1
            still = []
            for w in resident:
                i = w[0]
                kind, first, count = self.items[i]
                w[1] += 1
                if kind == A:
                    b = self.bucket_of_apply[first]
                    if self.ready_epoch[b] == epoch:
                        w[0] = None
                        applied[first] += 1
                        running.append((first, 2))
                        decided(i)                      # before it loads anything
                    elif w[1] > spin_limit or self.abort:
                        w[0] = None
                        self.abort, timed_out = 1, True
                        self.skipped.append(first)
                        decided(i)
                    else:
                        still.append(w)
                    continue
                if kind == N and w[1] < norm_ticks:
                    still.append(w)
                    continue
                w[0] = None
                b, last = (self.bucket_of_norm[first] if kind == N else first), True
                if kind == N:
                    summed[first:first + count] += 1
                    self.arrived[b] += count
                    last = self.arrived[b] == self.total[b]
                if last:
                    self.arrived[b] = 0
                    finalized[b] += 1
                    self.ready_epoch[b] = epoch
                decided(i)
            resident = still
        assert finished == 1 and full == 0 and words == [0] * 64, "finished twice or not at all"
        return dict(summed=summed, applied=applied, finalized=finalized, timed_out=timed_out, ticks=tick)


def test_a_launch_that_finishes_itself_does_so_once_and_last():
    plan, lay = small_plan()
    rng = np.random.default_rng(6)
    m = SelfFinishing(plan, lay.n_buckets)
    n, calls = len(m.items), 0
    for name, order in orders(m, rng):
        for slots in (1, 2, 7, 64, n):
            for spin in (1, 5, 200):
                r = m.launch(order, slots, spin)
                m.check(r)
                calls += 1
                if name == "in order" and spin == 200:
                    assert not r["timed_out"], slots
    assert m.epoch == 1 + calls


class LambModel:
    """LAMB in one pass: lamb_step's or bucket_clip_lamb's launch, the one that carries out items which gave up on their
    bucket, and the tail; driven with the plan's own work list (bca_plan_lamb_item).  Unlike the fused step's, these items
    also wait for items that come after them in the list: the rest of their own tensor."""

    def __init__(self, plan, n_buckets, clip):
        self.clip, self.items = clip, plan.lamb_items(clip)
        L, self.nN, self.nb = plan.n_chunks(B.BCA_TABLE_LAMB), plan.n_chunks(B.BCA_TABLE_NORM), n_buckets
        self.bucket_of = [plan.chunk_info(i, B.BCA_TABLE_LAMB)[3] for i in range(L)]
        self.bucket_of_norm = [plan.chunk_info(i, B.BCA_TABLE_NORM)[3] for i in range(self.nN)]
        self.total = [plan.bucket_chunks(b, B.BCA_TABLE_NORM)[1] for b in range(n_buckets)]
        self.nL, self.nt = L, plan.n_tensors
        self.items_of = [0] * self.nt
        for kind, _, _, t, _ in self.items:
            self.items_of[t] += kind == A
        self.arrived_b, self.ready_b = [0] * n_buckets, [0] * n_buckets
        self.arrived_t, self.ready_t = [0] * self.nt, [0] * self.nt
        self.epoch, self.abort, self.late_abort, self.skipped, self.late, self.status = 1, 0, 0, [], [], 0

    def moments(self, i):
        """First sweep of item i, and its arrival; the last one of the tensor publishes the ratio."""
        _, first, count, t, _ = self.items[i]
        self.swept[first:first + count] += 1
        self.arrived_t[t] += 1
        if self.arrived_t[t] == self.items_of[t]:
            self.arrived_t[t] = 0
            self.ratios[t] += 1
            self.ready_t[t] = self.epoch

    def update(self, i):
        _, first, count, t, _ = self.items[i]
        assert self.ready_t[t] == self.epoch, "an update before its tensor's ratio exists"
        self.updated[first:first + count] += 1

    def launch(self, order, slots, spin_limit, tensor_limit, norm_ticks=3, sweep_ticks=2, status_word=True, lose=0):
        """One call; limits None = wait for ever.  `lose`: items that the first give-ups fail to file (the list being full)."""
        self.swept, self.updated, self.ratios = np.zeros(self.nL, int), np.zeros(self.nL, int), np.zeros(self.nt, int)
        resident, nxt = [], 0                            # [item, phase, ticks or polls]; phases of LAMB items: bucket, sweep, ratio
        while nxt < len(order) or resident:
            while nxt < len(order) and len(resident) < slots:
                resident.append([order[nxt], 0 if self.clip else 1, 0])
                nxt += 1
            progressed, still = False, []
            for w in resident:
                i, w[2] = w[0], w[2] + 1
                kind, first, count, t, held = self.items[i]
                if kind != A:
                    progressed = True
                    if kind == N and w[2] < norm_ticks:
                        still.append(w)
                        continue
                    b, last = (self.bucket_of_norm[first] if kind == N else first), True
                    if kind == N:
                        self.arrived_b[b] += count
                        last = self.arrived_b[b] == self.total[b]
                    if last:
                        self.arrived_b[b], self.ready_b[b] = 0, self.epoch
                    continue
                if w[1] == 0:
                    if self.ready_b[self.bucket_of[first]] == self.epoch:
                        w[1], w[2], progressed = 1, 0, True
                    elif (spin_limit is not None and w[2] > spin_limit) or self.abort:
                        self.abort, self.status, progressed = 1, self.status | B.BCA_STATUS_TIMEOUT, True
                        self.skipped.append(i)
                        continue
                if w[1] == 1 and w[2] >= sweep_ticks:
                    self.moments(i)
                    progressed = True
                    if not held:
                        continue
                    w[1], w[2] = 2, 0
                elif w[1] == 1:
                    progressed = True
                if w[1] == 2:
                    if self.ready_t[t] == self.epoch:
                        self.update(i)
                        progressed = True
                        continue
                    if self.late_abort or (tensor_limit is not None and w[2] > tensor_limit):
                        if not self.late_abort:
                            self.late_abort, self.status = 1, self.status | B.BCA_STATUS_TIMEOUT
                        if lose:
                            lose, self.status = lose - 1, self.status | B.BCA_STATUS_INCOMPLETE
                        else:
                            self.late.append(i)
                        progressed = True
                        continue
                still.append(w)
            resident = still
            if not progressed:
                if spin_limit is None or tensor_limit is None:
                    return False                         # whoever is resident waits for ever and nobody else can start
        for i in self.skipped:                           # the launch for items that gave up on their bucket: no waits
            assert self.ready_b[self.bucket_of[self.items[i][1]]] == self.epoch
            self.moments(i)
        for i, (kind, _, _, _, held) in enumerate(self.items):   # the tail
            if kind == A and not held:
                self.update(i)
        for i in self.late:
            self.update(i)
        for i in self.skipped:
            if self.items[i][4]:
                self.update(i)
        out = self.status if status_word else None
        self.status = 0 if status_word else self.status & B.BCA_STATUS_INCOMPLETE
        late = len(self.late) + len(self.skipped)
        self.abort, self.late_abort, self.skipped, self.late = 0, 0, [], []
        self.epoch += 1
        return dict(status=out, late=late)

    def check(self, r):
        assert r, "the launch did not end"
        assert np.all(self.swept == 1), "a chunk's moments updated twice or not at all"
        assert np.all(self.updated == 1), "a chunk's parameters updated twice or not at all"
        assert all(x == (1 if n else 0) for x, n in zip(self.ratios, self.items_of)), "a tensor's ratio derived twice or not at all"
        assert self.arrived_t == [0] * self.nt and self.arrived_b == [0] * self.nb


def lamb_plan():
    """Held tensors of one to many items beside one that is too large, cut by buckets; 15 % of the elements in the latter."""
    sizes = [70_000, 5, 0, 1_000_000, 12_288, 300_001, 24 * 1024, 2_000_000] + [1_500_000] * 4 + [1024]
    sizes += [9_600_000] + [4_000_000] * 12
    lay = W.layout_flat_split(sizes, 3 << 20)
    return host_plan(lay), lay


@pytest.mark.parametrize("clip", [False, True])
def test_lamb_in_one_pass_ends_and_does_every_chunk_once_under_any_order(clip):
    plan, lay = lamb_plan()
    m = LambModel(plan, lay.n_buckets, clip)
    kinds = [k for k, *_ in m.items]
    held = [h for k, _, _, _, h in m.items if k == A]
    assert 0 < sum(held) < len(held) and (N in kinds) == clip
    n, rng = len(m.items), np.random.default_rng(8)
    ident = list(range(n))
    for name, order in (("in order", ident), ("reversed", ident[::-1]), ("random", [int(i) for i in rng.permutation(n)]),
                        ("lamb first", sorted(ident, key=lambda i: (kinds[i] != A, i)))):
        for slots in (1, 7, 100, 1024):
            for limits in ((1, 1), (30, 5), (10_000, 10_000)):
                r = m.launch(order, slots, *limits)
                m.check(r)
                assert (r["late"] > 0) == (r["status"] != 0)
                # in the list's order, with the slots of the GPU that the plan was made for, nobody gives up
                if name == "in order" and slots == 1024 and limits[0] == 10_000:
                    assert r["status"] == 0
    assert m.epoch == 1 + 4 * 4 * 3


@pytest.mark.parametrize("clip", [False, True])
def test_in_list_order_the_slots_of_the_gpu_are_enough_without_any_bound(clip):
    """A held tensor's items, with whatever lies between them, are at most three quarters of what is resident at once: started in
    order they all get a slot.  With fewer slots than a tensor has items the bound is what ends the launch."""
    plan, lay = lamb_plan()
    m = LambModel(plan, lay.n_buckets, clip)
    for _ in range(2):
        m.check(m.launch(list(range(len(m.items))), 1024, None, None))
    assert LambModel(plan, lay.n_buckets, clip).launch(list(range(len(m.items))), 100, None, None) is False
    m.check(m.launch(list(range(len(m.items))), 100, 50, 50))


@pytest.mark.parametrize("clip", [False, True])
@pytest.mark.parametrize("front", [True, False])
def test_the_held_end_of_a_tensor_that_is_too_large(clip, front):
    """A tensor of more than twice what can be held, first (its buckets are the last) or last in registration order: its
    last 768 items are held, by bucket_clip_lamb only where hardly anything follows them."""
    big, rest = [19_200_000], [2_000_000] * 10 + [5, 70_000]
    sizes = big + rest if front else rest + big
    lay = W.layout_flat_split(sizes, 3 << 20)
    plan, t = host_plan(lay), sizes.index(big[0])
    m = LambModel(plan, lay.n_buckets, clip)
    held = [h for k, _, _, u, h in m.items if k == A and u == t]
    ends = 768 if front or not clip else 0
    assert len(held) > 2 * 768 and sum(held) <= ends and sum(held) > ends - 2 and held == sorted(held)
    assert all(h for k, _, _, u, h in m.items if k == A and u != t)
    ident = list(range(len(m.items)))
    for order in (ident, ident[::-1], [int(i) for i in np.random.default_rng(1).permutation(len(ident))]):
        for slots, limits in ((100, (1, 1)), (1024, (30, 5)), (1024, (10_000, 10_000))):
            r = m.launch(order, slots, *limits)
            m.check(r)
            assert order is not ident or limits[0] != 10_000 or r["status"] == 0


def test_a_lost_item_is_reported_by_the_next_call_that_has_a_status_word():
    plan, lay = lamb_plan()
    m = LambModel(plan, lay.n_buckets, False)
    order = list(range(len(m.items)))
    assert m.launch(order, 64, 5, 5, status_word=False, lose=1)["status"] is None      # lamb_step
    assert np.sum(m.updated == 0) > 0
    assert m.launch(order, 1024, 10_000, 10_000, status_word=False)["status"] is None    # and again: it stays
    m.check(r := m.launch(order, 1024, 10_000, 10_000))
    assert r["status"] == B.BCA_STATUS_INCOMPLETE
    assert m.launch(order, 1024, 10_000, 10_000)["status"] == 0
