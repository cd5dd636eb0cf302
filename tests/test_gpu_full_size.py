"""GPU parity at the full sizes of the benchmark configurations, in the launch
configuration bench.py times (library defaults): BERT-Base (25 MiB buckets),
BERT-Large (50 MiB buckets, warm state), BERT-Large with fp16 gradients (1 MiB
buckets) and 20 consecutive steps of BERT-Large with 4 MiB buckets.  The oracle
finishes one BERT-Large step in a few seconds, so every element is compared."""
import time

import numpy as np
import pytest

import oracle
import paper_2402_02447_amd as B
import workloads as W
from gpu_util import Device, bits_equal, check_norms, check_state, f64, hp_kwargs, hyper, to_host

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(900)]


def full_fused(w, flags=0):
    lay = w.layout
    t0 = time.time()
    g, p, m, v = w.grads(), w.params(), w.exp_avg(), w.exp_avg_sq()
    print(f"[{w.name}] generated {lay.n_elements} elements in {time.time() - t0:.1f}s", flush=True)
    dev = Device(lay, g, p, m, v)
    assert dev.plan.n_groups >= 1
    dthr = dev.thresholds(w.thresholds)
    dev.plan.bucket_clip_adam(dthr, hyper(w.hyper), w.first_step, flags, dev.norms, dev.coefs, dev.status)
    dev.sync()
    t0 = time.time()
    og = [x.copy() for x in g] if flags & B.BCA_WRITE_BACK_GRADS else g
    op, om, ov = f64(p), f64(m), f64(v)
    onorm, ocoef, ost = oracle.bucket_clip_adam(lay, og, op, om, ov, w.thresholds, step=w.first_step,
                                                write_back=bool(flags & B.BCA_WRITE_BACK_GRADS), **hp_kwargs(w.hyper))
    print(f"[{w.name}] oracle step {time.time() - t0:.1f}s", flush=True)
    rel = check_norms(dev.norms.cpu().numpy(), onorm)
    gcoef = dev.coefs.cpu().numpy()
    assert np.allclose(gcoef, ocoef, rtol=1e-6, atol=0)
    assert int(dev.status.item()) == ost == 0
    rp = check_state("p", to_host(dev.p), op)
    rm = check_state("m", to_host(dev.m), om)
    rv = check_state("v", to_host(dev.v), ov, strict_rel=True)
    print(f"[{w.name}] norm rel {rel:.2e}; p {rp}; m {rm}; v {rv}; clipped {int((ocoef < 1).sum())}/{lay.n_buckets}",
          flush=True)
    if not flags & B.BCA_WRITE_BACK_GRADS:
        assert bits_equal(to_host(dev.g), g)
    dev.close()
    return ocoef


def test_bert_base_25mib_full_size():
    coefs = full_fused(W.config_bert_base())
    assert (coefs < 1).all()            # norm ~ 2.56 > 1: every bucket clips


def test_bert_large_50mib_full_size():
    w = W.config_bert_large()
    coefs = full_fused(w)
    assert (coefs < 1).all() and coefs[w.hot_buckets].max() < 0.01 < coefs.max()


def test_bert_large_fp16_1mib_full_size():
    w = W.config_bert_large_fp16()
    coefs = full_fused(w)
    assert (coefs < 1).mean() > 0.9     # threshold 1/sqrt(B): nearly every bucket clips


def test_bert_large_4mib_20_steps_full_size():
    w = W.config_bert_large_multistep()
    lay = w.layout
    p, m, v = w.params(), w.exp_avg(), w.exp_avg_sq()
    dev = Device(lay, w.grads(0), p, m, v)
    dthr = dev.thresholds(w.thresholds)
    op, om, ov = f64(p), f64(m), f64(v)
    del p, m, v
    worst = {"p": 0.0, "m": 0.0, "v": 0.0}
    clipped = 0
    for k in range(w.n_steps):
        t0 = time.time()
        g = w.grads(k)
        dev.set_grads(g)
        step = w.first_step + k
        dev.plan.bucket_clip_adam(dthr, hyper(w.hyper), step, 0, dev.norms, dev.coefs, dev.status)
        dev.sync()
        onorm, ocoef, ost = oracle.bucket_clip_adam(lay, g, op, om, ov, w.thresholds, step=step, **hp_kwargs(w.hyper))
        assert int(dev.status.item()) == ost == 0
        check_norms(dev.norms.cpu().numpy(), onorm)
        clipped += int((ocoef < 1).sum())
        rp = check_state(f"p@{step}", to_host(dev.p), op)
        rm = check_state(f"m@{step}", to_host(dev.m), om)
        rv = check_state(f"v@{step}", to_host(dev.v), ov, strict_rel=True)
        worst["p"] = max(worst["p"], rp["max_rel_big"])
        worst["m"] = max(worst["m"], rm["max_abs_small"])
        worst["v"] = max(worst["v"], rv["max_rel_all"])
        print(f"[20 steps] step {step}: p rel {rp['max_rel_big']:.2e} abs {rp['max_abs_small']:.2e}; "
              f"m abs {rm['max_abs_small']:.2e}; v rel {rv['max_rel_all']:.2e}; {time.time() - t0:.1f}s", flush=True)
    frac = clipped / (w.n_steps * lay.n_buckets)
    assert 0.4 < frac < 0.6, frac        # about half of the buckets clip
    print("[20 steps] worst", worst, flush=True)
    dev.close()


def test_bert_large_whole_gradient_clipping_full_size():
    # the paper's baseline (clip the whole gradient once, Sec. 3.2) on the 50 MiB layout
    w = W.config_bert_large()
    lay = w.layout
    g, p, m, v = w.grads(), w.params(), w.exp_avg(), w.exp_avg_sq()
    dev = Device(lay, g, p, m, v)
    import torch
    norms = torch.zeros(lay.n_buckets + 1, dtype=torch.float32, device="cuda")
    dc = torch.tensor([1.0], dtype=torch.float32, device="cuda")
    dev.plan.bucket_clip_adam(dc, hyper(w.hyper), w.first_step, B.BCA_CLIP_WHOLE_GRADIENT, norms, dev.coefs, dev.status)
    dev.sync()
    op, om, ov = f64(p), f64(m), f64(v)
    onorms, owhole, ocoef, ost = oracle.whole_clip_adam(lay, g, op, om, ov, 1.0, step=w.first_step, **hp_kwargs(w.hyper))
    gn = norms.cpu().numpy()
    check_norms(gn[:-1], onorms)
    check_norms(gn[-1:], np.asarray([owhole]))
    assert ocoef < 1 and int(dev.status.item()) == ost == 0
    assert np.all(dev.coefs.cpu().numpy() == dev.coefs.cpu().numpy()[0])
    check_state("p", to_host(dev.p), op)
    check_state("m", to_host(dev.m), om)
    check_state("v", to_host(dev.v), ov, strict_rel=True)
    print(f"[whole] norm {owhole:.4f} coef {ocoef:.6f}", flush=True)
    dev.close()


def test_bert_large_lamb_bf16_masked_full_size():
    # LAMB behind bucket-wise clipping on the 50 MiB layout, bf16 gradients, biases and LayerNorm exempt from decay
    w = W.config_bert_large()
    lay = w.layout
    numels = [int(n) for n in lay.tensor_numel]
    g = oracle.Bf16(W.normal_bf16_tensors(numels, 0, 1e-3))
    p, m, v = w.params(), w.exp_avg(), w.exp_avg_sq()
    mask = W.bert_decay_mask(30522, 1024, 24, 4096, 512)
    dev = Device(lay, g, p, m, v)
    dev.plan.set_decay_mask(mask)
    dthr = dev.thresholds(w.thresholds)
    dev.plan.bucket_clip_lamb(dthr, hyper(w.hyper), w.first_step, 0, dev.norms, dev.coefs, dev.trust, dev.status)
    dev.sync()
    t0 = time.time()
    op, om, ov = f64(p), f64(m), f64(v)
    onorm, ocoef, otrust, ost = oracle.bucket_clip_lamb(lay, g, op, om, ov, w.thresholds, step=w.first_step, decay=mask,
                                                        **hp_kwargs(w.hyper))
    print(f"[lamb] oracle step {time.time() - t0:.1f}s", flush=True)
    assert int(dev.status.item()) == ost == 0 and (ocoef < 1).all()
    rel = check_norms(dev.norms.cpu().numpy(), onorm)
    tr = dev.trust.cpu().numpy().astype(np.float64)
    trel = np.abs(tr - otrust) / otrust
    assert trel.max() <= 1e-5, trel.max()
    rp = check_state("p", to_host(dev.p), op)
    rm = check_state("m", to_host(dev.m), om)
    rv = check_state("v", to_host(dev.v), ov, strict_rel=True)
    print(f"[lamb] norm rel {rel:.2e}; trust rel {trel.max():.2e}; p {rp}; m {rm}; v {rv}", flush=True)
    assert bits_equal(to_host(dev.g), g)
    dev.close()


def test_bert_large_lamb_step_in_one_pass_in_runs_and_in_one_run_full_size():
    # lamb_step as bench.py times it (one pass), in runs of tensors of at most 32 Mi elements (11 of them, the moments stored
    # cacheable) and as a single run, bit for bit, and against the oracle
    w = W.config_bert_large()
    lay = w.layout
    g, p, m, v = w.grads(), w.params(), w.exp_avg(), w.exp_avg_sq()
    one = Device(lay, g, p, m, v)
    items = [i for i in one.plan.lamb_items(False) if i[0] == 1]
    assert sum(held for _, _, _, _, held in items) > 0.8 * len(items)
    one.plan.lamb_step(hyper(w.hyper), w.first_step, one.trust)
    one.sync()
    got = (one.trust.cpu().numpy().copy(), to_host(one.p), to_host(one.m), to_host(one.v))
    assert bits_equal(to_host(one.g), g)
    one.close()
    del one
    for limit, n_runs in ((32 << 20, 11), (2 ** 62, 1)):
        runs = Device(lay, g, p, m, v, lamb_group_elems=limit)
        assert len(runs.plan.lamb_runs()) == n_runs and runs.plan.n_lamb_items(False) == 0
        runs.plan.lamb_step(hyper(w.hyper), w.first_step, runs.trust)
        runs.sync()
        assert np.array_equal(got[0], runs.trust.cpu().numpy())
        for name, a, b in (("p", got[1], runs.p), ("m", got[2], runs.m), ("v", got[3], runs.v)):
            assert bits_equal(a, to_host(b)), (name, limit)
        runs.close()
        del runs
    t0 = time.time()
    op, om, ov = f64(p), f64(m), f64(v)
    otrust = oracle.lamb_step(lay, g, op, om, ov, step=w.first_step, **hp_kwargs(w.hyper))
    print(f"[lamb one pass] oracle step {time.time() - t0:.1f}s", flush=True)
    trel = np.abs(got[0][:lay.n_tensors].astype(np.float64) - otrust) / otrust
    assert trel.max() <= 1e-5, trel.max()
    check_state("p", got[1], op), check_state("m", got[2], om), check_state("v", got[3], ov, strict_rel=True)


def test_bert_large_whole_tensor_buckets_full_size():
    # DDP-style packing: whole tensors per bucket (the 31 M-element word embedding is one bucket of its own)
    lay = W.layout_whole_tensors(W.bert_large_numels(), 50 * W.MIB // 4)
    assert lay.tensors_split() == 0 and lay.n_buckets < 26
    w = W.config_bert_large()
    w = W.Workload("bert_large_whole_tensor_buckets", lay, "f32", np.full(lay.n_buckets, 1.0, np.float32), w.hyper,
                   first_step=1000, seed=0, warm=True)
    coefs = full_fused(w, B.BCA_WRITE_BACK_GRADS)
    assert (coefs < 1).all()


def test_one_tensor_of_more_than_2_pow_32_elements():
    # Maximum sizes: element offsets beyond 32 bits, byte offsets beyond 2^34, 4.2 M work items.  The oracle cannot hold
    # 4.3 G elements in fp64, so the norms are checked against their closed form (the gradient repeats a 4 099-value
    # pattern, so a bucket's sum of squares is counts x squares, exact in fp64) and p, m, v on sampled elements, which the
    # oracle updates one by one given the bucket's coefficient.
    import torch
    N = (1 << 32) + (1 << 20) + 7
    cap = 1 << 30
    period = 4099
    lay = W.layout_flat_split([N], cap)
    nb = lay.n_buckets
    assert nb == 5 and int(lay.bucket_numel()[-1]) == (1 << 20) + 7
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    vals = (torch.randn(period, generator=gen, device=dev) * 1e-2).to(torch.float16)
    g = torch.empty(N, dtype=torch.float16, device=dev)
    step_fill = 1 << 28
    for a in range(0, N, step_fill):
        b = min(N, a + step_fill)
        g[a:b] = vals[torch.arange(a, b, device=dev) % period]
    p = torch.randn(N, generator=gen, device=dev) * 0.02
    m = torch.randn(N, generator=gen, device=dev) * 3e-4
    v = (torch.rand(N, generator=gen, device=dev) + 0.5) * 1e-6
    # sampled elements: both ends, both sides of every bucket boundary and of the 2^32 mark
    marks = [0, N] + [cap * k for k in range(1, 5)] + [1 << 32, (1 << 32) + 4096]
    idx = np.unique(np.concatenate([np.arange(max(0, x - 1500), min(N, x + 1500)) for x in marks]))
    didx = torch.from_numpy(idx).to(dev)
    before = [x[didx].cpu().numpy() for x in (p, m, v)]
    gs = g[didx].cpu().numpy()

    # closed-form norms
    sq = vals.cpu().numpy().astype(np.float64) ** 2
    want_norm = np.zeros(nb)
    for bkt in range(nb):
        a, b = bkt * cap, min(N, (bkt + 1) * cap)
        r = np.arange(period)
        counts = (b - r + period - 1) // period - (a - r + period - 1) // period        # indices i in [a, b) with i % period == r
        assert counts.sum() == b - a
        want_norm[bkt] = np.sqrt(np.sum(counts * sq))
    thr = (want_norm * np.asarray([0.5, 2.0, 0.25, 0.9, 0.1])).astype(np.float32)       # bucket 1 is not clipped

    plan = B.Plan.from_layout(lay, B.BCA_GRAD_F16, device=torch.cuda.current_device())
    plan.bind([g], [p], [m], [v])
    norms = torch.zeros(nb, device=dev)
    coefs = torch.zeros(nb, device=dev)
    status = torch.full((1,), -1, dtype=torch.int32, device=dev)
    hp = W.Hyper()
    plan.bucket_clip_adam(torch.from_numpy(thr).to(dev), hyper(hp), 77, 0, norms, coefs, status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    check_norms(norms.cpu().numpy(), want_norm)
    gcoef = coefs.cpu().numpy()
    want_coef = np.where(want_norm >= thr, thr / want_norm, 1.0)
    assert np.allclose(gcoef, want_coef, rtol=1e-6) and gcoef[1] == 1.0
    after = [x[didx].cpu().numpy() for x in (p, m, v)]
    assert np.array_equal(g[didx].cpu().numpy().view(np.uint16), gs.view(np.uint16))

    # the oracle on the samples: one small bucket per original bucket, its threshold set so that it clips by the same factor
    which = np.minimum(idx // cap, nb - 1)
    numels = [int(np.sum(which == bkt)) for bkt in range(nb)]
    small = W.layout_one_tensor_per_bucket(numels)
    sg = [gs[which == bkt] for bkt in range(nb)]
    small_norm = oracle.bucket_norms(small, sg)
    small_thr = np.where(gcoef < 1, gcoef.astype(np.float64) * small_norm, np.inf).astype(np.float32)
    op, om, ov = ([x[which == bkt].astype(np.float64) for bkt in range(nb)] for x in before)
    _, ocoef, _ = oracle.bucket_clip_adam(small, sg, op, om, ov, small_thr, step=77, **hp_kwargs(hp))
    assert np.allclose(ocoef, gcoef, rtol=3e-7)
    check_state("p", [after[0][which == bkt] for bkt in range(nb)], op)
    check_state("m", [after[1][which == bkt] for bkt in range(nb)], om)
    check_state("v", [after[2][which == bkt] for bkt in range(nb)], ov, strict_rel=True)
    # and nothing between the samples was left out: every element of m moved (a skipped chunk would keep its old bits)
    gen2 = torch.Generator(device=dev)
    gen2.manual_seed(5)
    torch.randn(period, generator=gen2, device=dev)
    torch.randn(N, generator=gen2, device=dev)                                           # replays p's draw
    m_old = torch.randn(N, generator=gen2, device=dev) * 3e-4
    unchanged = int((m == m_old).sum().item())
    assert unchanged < N // 1000, unchanged
    plan.close()


def test_bert_large_per_bucket_clip_then_adam_full_size():
    # the paper's own order of work: every bucket clipped on its own as it becomes ready (one launch per bucket),
    # then Adam on the stored, scaled gradients
    w = W.config_bert_large()
    lay = w.layout
    g, p, m, v = w.grads(), w.params(), w.exp_avg(), w.exp_avg_sq()
    dev = Device(lay, g, p, m, v)
    dthr = dev.thresholds(w.thresholds)
    status = 0
    for b in range(lay.n_buckets):
        dev.plan.bucket_clip(b, b + 1, dthr, dev.norms, dev.coefs, dev.status)
        status |= int(dev.status.item())
    dev.plan.adam_step(hyper(w.hyper), w.first_step)
    dev.sync()
    onorm = oracle.bucket_norms(lay, g)
    ocoef, ost = oracle.clip_coefs(onorm, w.thresholds)
    og = [x.copy() for x in g]
    oracle.bucket_scale(lay, og, ocoef)
    op, om, ov = f64(p), f64(m), f64(v)
    oracle.adam_step(lay, og, op, om, ov, step=w.first_step, **hp_kwargs(w.hyper))
    assert status == ost == 0
    check_norms(dev.norms.cpu().numpy(), onorm)
    assert np.allclose(dev.coefs.cpu().numpy(), ocoef, rtol=1e-6, atol=0)
    for a, b in zip(to_host(dev.g), og):
        assert np.allclose(a, b, rtol=5e-7, atol=1e-45)
    rp = check_state("p", to_host(dev.p), op)
    check_state("m", to_host(dev.m), om)
    rv = check_state("v", to_host(dev.v), ov, strict_rel=True)
    print(f"[per-bucket] p {rp}; v {rv}", flush=True)
    dev.close()
