"""GPU tests of the C ABI beyond plain parity: the multi-layer entry point, call-order errors,
bitwise repeatability, reset and re-commit, the measurement hooks."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_08727_amd import binding as A
from paper_2603_08727_amd import synth
from helpers import SideBySide, make_cfg

pytestmark = pytest.mark.gpu


def _prepare(wl, rho=0.5):
    cfg = make_cfg(wl)
    cache = A.arkv_cache_create(cfg)
    stats = torch.zeros((wl.n_layers, wl.batch, 3), dtype=torch.float32, device="cuda")
    ins = []
    for l in range(wl.n_layers):
        k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, l))
        A.arkv_prefill_stats(cache, l, qw, k, wl.prefill, synth.softmax_scale(wl, l), stats[l])
        ins.append((k, v))
    for l in range(wl.n_layers):
        A.arkv_prefill_commit(cache, l, ins[l][0], ins[l][1], wl.prefill, np.full(wl.batch, rho, np.float32))
    return cfg, cache


def _export_all(cache, cfg, L):
    return [A.arkv_cache_export(cache, l, cfg) for l in range(L)]


def test_layers_entry_point_equals_per_layer_calls():
    """arkv_decode_step_layers over 3 layers == three arkv_decode_step calls, bit for bit, through a tailor."""
    wl = synth.C1.scaled(name="multi", n_layers=3, batch=2, decode_steps=30)
    L, B = wl.n_layers, wl.batch
    cfg, c1 = _prepare(wl)
    _, c2 = _prepare(wl)
    try:
        dins = [tuple(t.cuda() for t in synth.decode_inputs(wl, l)) for l in range(L)]
        q = torch.stack([d[0] for d in dins], 1).contiguous()
        kn = torch.stack([d[1] for d in dins], 1).contiguous()
        vn = torch.stack([d[2] for d in dins], 1).contiguous()
        sc = np.array([synth.softmax_scale(wl, l) for l in range(L)], np.float32)
        o1 = torch.empty((L, B, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device="cuda")
        o2 = torch.empty_like(o1)
        for t in range(wl.decode_steps):
            for l in range(L):
                A.arkv_decode_step(c1, l, q[t, l], kn[t, l], vn[t, l], float(sc[l]), o1[l])
            A.arkv_decode_step_layers(c2, 0, L, q[t], kn[t], vn[t], sc, o2)
            assert torch.equal(o1.view(torch.int16), o2.view(torch.int16)), t
        assert A.arkv_cache_progress(c1, 0)[0] >= 2
        for e1, e2 in zip(_export_all(c1, cfg, L), _export_all(c2, cfg, L)):
            for k in e1:
                assert np.array_equal(e1[k], e2[k]), k
    finally:
        A.arkv_cache_destroy(c1); A.arkv_cache_destroy(c2)


@pytest.mark.parametrize("g,bits,byte_budget", [
    (4, 4, False),        # the logits fit the tailor's plan
    (8, 2, False),        # a plan made larger for them
    (2, 8, True),
    (8, 2, True),         # a buffer for one layer's logits; launches of several keep none
])
def test_tailor_at_every_step_through_all_entry_points(g, bits, byte_budget):
    """With a tailor at every step, three layers in one call and the call with static scratch give the same bits as one call per
    layer: outputs of every step and the caches behind the last, through the 17th tailor, whose moves (of more than 1024 rows) are
    made elsewhere."""
    wl = synth.C1.scaled(name="each", n_layers=3, n_q_heads=2 * g, n_kv_heads=2, head_dim=64, bits=bits, prefill=1500,
                         budget_frac=1100.5 / 1500, window=16, decode_steps=21)
    assert wl.capacity == 1100
    L = wl.n_layers
    cfg = make_cfg(wl, every_step=True, byte_budget=byte_budget)
    caches = [A.arkv_cache_create(cfg) for _ in range(3)]
    try:
        sc = np.array([synth.softmax_scale(wl, l) for l in range(L)], np.float32)
        for c in caches:
            for l in range(L):
                k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, l))
                A.arkv_prefill_stats(c, l, qw, k, wl.prefill, float(sc[l]), torch.zeros((1, 3), device="cuda"))
                A.arkv_prefill_commit(c, l, k, v, wl.prefill, np.full(1, 0.4, np.float32))
        dins = [tuple(t.cuda() for t in synth.decode_inputs(wl, l)) for l in range(L)]
        q, kn, vn = (torch.stack([d[i] for d in dins], 1).contiguous() for i in range(3))
        outs = [torch.empty((L, 1, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device="cuda") for _ in caches]
        for t in range(wl.decode_steps):
            for l in range(L):
                A.arkv_decode_step(caches[0], l, q[t, l], kn[t, l], vn[t, l], float(sc[l]), outs[0][l])
                A.arkv_decode_step_static(caches[1], l, q[t, l], kn[t, l], vn[t, l], float(sc[l]), outs[1][l])
            A.arkv_decode_step_layers(caches[2], 0, L, q[t], kn[t], vn[t], sc, outs[2])
            for o in outs[1:]:
                assert torch.equal(outs[0].view(torch.int16), o.view(torch.int16)), t
        assert A.arkv_cache_progress(caches[0], 0)[0] == wl.decode_steps + 1
        ref = _export_all(caches[0], cfg, L)
        for c in caches[1:]:
            for e1, e2 in zip(ref, _export_all(c, cfg, L)):
                for k in e1:
                    assert np.array_equal(e1[k], e2[k]), k
    finally:
        for c in caches:
            A.arkv_cache_destroy(c)


@pytest.mark.parametrize("g,bits,byte_budget", [(1, 4, False), (4, 4, False), (8, 4, False), (2, 8, True), (8, 2, True)])
def test_memory_of_the_policy_without_slack(g, bits, byte_budget):
    """What tailor_policy 1 allocates for logits beyond a cache of the other policy that keeps as many rows: nothing where the
    tailor's plan can hold them (4 bytes per head and row), else what a plan lacks for N rows, with a byte budget one layer's
    logits."""
    L, hkv, N, W = 8, 8, 4096, 32
    used = []
    for policy in (0, 1):
        cfg = A.arkv_config_default(n_layers=L, batch=1, n_q_heads=g * hkv, n_kv_heads=hkv, head_dim=64, capacity_tokens=N,
                                    window=W, alpha=1.0, quant_bits=bits, tailor_policy=policy, budget_mode=int(byte_budget))
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        c = A.arkv_cache_create(cfg)
        used.append(before - torch.cuda.mem_get_info()[0])
        A.arkv_cache_destroy(c)
    cap_q = A.arkv_budget_counts(cfg, 0.0)[2]
    rows, plan = max(N, W + cap_q + 1), 16 + 3 * (N + 17) + 2 * cap_q
    granule = 2 << 20                               # device memory is handed out in blocks of 2 MiB
    extra = 0 if g * rows <= plan else hkv * rows * g * 4 if byte_budget else L * hkv * (g * N - plan + 4) * 4
    assert used[0] > 0 and used[1] - used[0] <= extra + granule, (used, extra)


def test_bitwise_repeatability():
    """Two runs of the same trajectory give identical bytes (no float atomics anywhere)."""
    wl = synth.C1.scaled(name="repeat", decode_steps=40)
    outs = []
    for _ in range(2):
        cfg, c = _prepare(wl, rho=0.4)
        try:
            q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0))
            o = torch.empty((wl.batch, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device="cuda")
            acc = []
            for t in range(wl.decode_steps):
                A.arkv_decode_step(c, 0, q[t], kn[t], vn[t], synth.softmax_scale(wl, 0), o)
                acc.append(o.clone())
            outs.append((torch.stack(acc).cpu().view(torch.int16).numpy(), A.arkv_cache_export(c, 0, cfg)))
        finally:
            A.arkv_cache_destroy(c)
    assert np.array_equal(outs[0][0], outs[1][0])
    for k in outs[0][1]:
        assert np.array_equal(outs[0][1][k], outs[1][1][k]), k


def test_call_order_errors_and_reset():
    wl = synth.C1.scaled(name="order", prefill=200, decode_steps=4)
    cfg = make_cfg(wl)
    c = A.arkv_cache_create(cfg)
    try:
        k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
        q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0))
        o = torch.empty((wl.batch, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device="cuda")
        stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
        rho = np.full(wl.batch, 0.5, np.float32)
        with pytest.raises(A.ArkvError) as e:                      # decode before commit
            A.arkv_decode_step(c, 0, q[0], kn[0], vn[0], 0.1, o)
        assert e.value.code == A.ESTATE
        with pytest.raises(A.ArkvError) as e:                      # commit before scoring
            A.arkv_prefill_commit(c, 0, k, v, wl.prefill, rho)
        assert e.value.code == A.ESTATE
        with pytest.raises(A.ArkvError) as e:                      # prompt not longer than the window
            A.arkv_prefill_stats(c, 0, qw, k, wl.window, 0.1, stats)
        assert e.value.code == A.EINVAL
        with pytest.raises(A.ArkvError) as e:                      # layer out of range
            A.arkv_prefill_stats(c, 5, qw, k, wl.prefill, 0.1, stats)
        assert e.value.code == A.EINVAL
        A.arkv_prefill_stats(c, 0, qw, k, wl.prefill, 0.1, stats)
        with pytest.raises(A.ArkvError) as e:                      # commit with another length
            A.arkv_prefill_commit(c, 0, k, v, wl.prefill - 1, rho)
        assert e.value.code == A.ESTATE
        A.arkv_prefill_commit(c, 0, k, v, wl.prefill, rho)
        with pytest.raises(A.ArkvError) as e:                      # commit twice
            A.arkv_prefill_commit(c, 0, k, v, wl.prefill, rho)
        assert e.value.code == A.ESTATE
        A.arkv_decode_step(c, 0, q[0], kn[0], vn[0], 0.1, o)
        first = A.arkv_cache_export(c, 0, cfg)
        # a new request on the same memory gives the same result
        A.arkv_cache_reset(c, 0)
        A.arkv_prefill_stats(c, 0, qw, k, wl.prefill, 0.1, stats)
        A.arkv_prefill_commit(c, 0, k, v, wl.prefill, rho)
        A.arkv_decode_step(c, 0, q[0], kn[0], vn[0], 0.1, o)
        second = A.arkv_cache_export(c, 0, cfg)
        for key in first:
            assert np.array_equal(first[key], second[key]), key
    finally:
        A.arkv_cache_destroy(c)


def test_prefill_attention_argument_errors():
    wl = synth.C1.scaled(name="attn_err", prefill=200, decode_steps=2)
    cfg = make_cfg(wl)
    c = A.arkv_cache_create(cfg)
    try:
        k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
        T, W = wl.prefill, wl.window
        q = torch.zeros((wl.batch, wl.n_q_heads, T, wl.head_dim), dtype=torch.bfloat16, device="cuda")
        out = torch.empty_like(q)
        stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
        for args in [(0, T + 1, T, 0.1, None),        # more queries than keys
                     (0, 0, T, 0.1, None),            # no query
                     (0, T, T, 0.0, None),            # scale must be positive
                     (3, T, T, 0.1, None),            # layer out of range
                     (0, W - 1, T, 0.1, stats),       # the scorer needs the whole window among the queries
                     (0, W, W, 0.1, stats)]:          # ... and a prompt longer than the window
            layer, Tq, Tk, scale, st = args
            with pytest.raises(A.ArkvError) as e:
                A.arkv_prefill_attention(c, layer, q[:, :, :max(Tq, 1)].contiguous(), k, v, Tq, Tk, scale, out, st)
            assert e.value.code == A.EINVAL, args
        lse = torch.zeros((wl.batch, wl.n_q_heads, W), dtype=torch.float32, device="cuda")
        for layer, Tk, scale in [(3, T, 0.1), (0, W, 0.1), (0, T, -1.0)]:   # the log-sum-exp variant checks the same
            with pytest.raises(A.ArkvError) as e:
                A.arkv_prefill_stats_lse(c, layer, qw, k, Tk, scale, lse, stats)
            assert e.value.code == A.EINVAL
        A.arkv_prefill_attention(c, 0, q, k, v, T, T, 0.1, out, stats)      # scores the layer
        A.arkv_prefill_commit(c, 0, k, v, T, np.full(wl.batch, 0.5, np.float32))
        with pytest.raises(A.ArkvError) as e:
            A.arkv_prefill_stats_lse(c, 0, qw, k, T, 0.1, lse, stats)
        assert e.value.code == A.ESTATE
        with pytest.raises(A.ArkvError) as e:                               # scoring a committed layer again
            A.arkv_prefill_attention(c, 0, q, k, v, T, T, 0.1, out, stats)
        assert e.value.code == A.ESTATE
        A.arkv_prefill_attention(c, 0, q, k, v, T, T, 0.1, out, None)       # attention alone is still allowed
        torch.cuda.synchronize()
    finally:
        A.arkv_cache_destroy(c)


def test_measurement_hooks():
    wl = synth.C1.scaled(name="hooks", decode_steps=6)
    cfg, c = _prepare(wl)
    try:
        q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0))
        o = torch.empty((wl.batch, wl.n_q_heads, wl.head_dim), dtype=torch.bfloat16, device="cuda")
        A.arkv_debug_time_attend(c, True)
        for t in range(wl.decode_steps):
            A.arkv_decode_step(c, 0, q[t], kn[t], vn[t], 0.1, o)
        ms, n = A.arkv_debug_attend_time(c)
        assert n == wl.decode_steps and 0 < ms < 100
        A.arkv_debug_time_attend(c, False)
        buf = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
        for pattern in (0, 1, 2):
            us = A.arkv_measure_stream_read(buf, 16 << 20, 20, pattern)
            assert 0 < us < 1e4
    finally:
        A.arkv_cache_destroy(c)


@pytest.mark.parametrize("layers_per_call", [1, 2])
def test_counts_behind_tailors_reach_the_host_across_resets(layers_per_call):
    """After a decode-time tailor the host learns the units' counts from words that the kernels store in pinned memory.  A cache
    that went through tailors, was reset and took another prompt gives the same bits as a fresh one, whether or not the words of
    the earlier tailors had arrived; so do its counters.  (A step of several layers does not hand its counts to the kernel.)"""
    L, hq, hkv, d, T, N, steps = 2, 8, 2, 64, 200, 90, 70
    wl = synth.C1.scaled(name="words", n_layers=L, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=2, budget_frac=(N + 0.5) / T)
    assert wl.capacity == N
    other = wl.scaled(name="words2", seed=wl.seed + 77)
    cfg = make_cfg(wl)

    def session(cache, w, wait):
        stats = torch.zeros((w.batch, 3), dtype=torch.float32, device="cuda")
        for l in range(L):
            k, v, qw = (t.cuda() for t in synth.prefill_inputs(w, l))
            A.arkv_prefill_stats(cache, l, qw, k, T, 0.1, stats)
            A.arkv_prefill_commit(cache, l, k, v, T, [0.4] * w.batch)
        q, kn, vn = (torch.stack(x).cuda() for x in zip(*[synth.decode_inputs(w, l, steps) for l in range(L)]))
        outs = torch.zeros((steps, L, w.batch, hq, d), dtype=torch.bfloat16, device="cuda")
        for i in range(steps):
            if layers_per_call == L:
                A.arkv_decode_step_layers(cache, 0, L, q[:, i].contiguous(), kn[:, i].contiguous(), vn[:, i].contiguous(), [0.1] * L, outs[i])
            else:
                for l in range(L):
                    A.arkv_decode_step(cache, l, q[l, i], kn[l, i], vn[l, i], 0.1, outs[i, l])
            if wait:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        return outs, [A.arkv_cache_counters(cache, l, w.batch * hkv) for l in range(L)]

    used, fresh = A.arkv_cache_create(cfg), A.arkv_cache_create(cfg)
    try:
        session(used, other, wait=False)
        assert A.arkv_cache_progress(used, 0)[0] >= 3
        A.arkv_cache_reset(used, -1)
        a, ca = session(used, wl, wait=False)
        b, cb = session(fresh, wl, wait=True)
        assert torch.equal(a, b)
        for x, y in zip(ca, cb):
            assert all(np.array_equal(i, j) for i, j in zip(x, y))
    finally:
        A.arkv_cache_destroy(used)
        A.arkv_cache_destroy(fresh)


def test_counts_behind_a_tailor_of_several_layers_reach_each_layers_next_steps():
    """A tailor of two layers in one launch names each layer's counts apart.  The single-layer steps behind it, with the words
    there, hand those counts to the kernel: the same bits as a cache that was driven layer by layer, with layers whose budgets and
    counts differ."""
    L, hq, hkv, d, T, N, steps = 2, 8, 2, 64, 200, 90, 70
    wl = synth.C1.scaled(name="words3", n_layers=L, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=2, budget_frac=(N + 0.5) / T)
    cfg = make_cfg(wl)
    q, kn, vn = (torch.stack(x).cuda() for x in zip(*[synth.decode_inputs(wl, l, steps) for l in range(L)]))
    got = []
    for together in (True, False):
        cache = A.arkv_cache_create(cfg)
        try:
            stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
            for l in range(L):
                k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, l))
                A.arkv_prefill_stats(cache, l, qw, k, T, 0.1, stats)
                A.arkv_prefill_commit(cache, l, k, v, T, [(0.2, 0.7)[l]] * wl.batch)
            outs, layers_tailors = torch.zeros((steps, L, wl.batch, hq, d), dtype=torch.bfloat16, device="cuda"), 0
            for i in range(steps):
                if together and A.arkv_cache_progress(cache, 0)[1] + 1 >= N:       # this step ends with a tailor
                    A.arkv_decode_step_layers(cache, 0, L, q[:, i].contiguous(), kn[:, i].contiguous(), vn[:, i].contiguous(), [0.1] * L, outs[i])
                    torch.cuda.synchronize()
                    layers_tailors += 1
                    assert not np.array_equal(A.arkv_cache_counters(cache, 0, wl.batch * hkv)[0],
                                              A.arkv_cache_counters(cache, 1, wl.batch * hkv)[0])
                else:
                    for l in range(L):
                        A.arkv_decode_step(cache, l, q[l, i], kn[l, i], vn[l, i], 0.1, outs[i, l])
            torch.cuda.synchronize()
            assert layers_tailors == (A.arkv_cache_progress(cache, 0)[0] - 1 if together else 0)
            got.append((outs, [A.arkv_cache_export(cache, l, cfg) for l in range(L)]))
        finally:
            A.arkv_cache_destroy(cache)
    assert torch.equal(got[0][0], got[1][0])
    for a, b in zip(got[0][1], got[1][1]):
        for name in a:
            assert np.array_equal(a[name], b[name]), name


def test_static_steps_with_scores_of_several_workgroups():
    """A static step's own tickets are not those of the tailor behind it, whose rows are scored by several workgroups: the same
    bits as the other entry point, through the first tailors (moves in launches of their own) and the later ones."""
    N, T, steps = 4300, 4800, 20
    wl = synth.C1.scaled(name="static_parts", n_q_heads=8, n_kv_heads=2, head_dim=64, prefill=T, batch=2, n_layers=1, budget_frac=(N + 0.5) / T)
    cfg = make_cfg(wl, every_step=True)
    k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
    q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0, steps))
    caches = [A.arkv_cache_create(cfg) for _ in range(2)]
    try:
        outs = []
        for cache, step in zip(caches, (A.arkv_decode_step, A.arkv_decode_step_static)):
            stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
            A.arkv_prefill_stats(cache, 0, qw, k, T, 0.1, stats)
            A.arkv_prefill_commit(cache, 0, k, v, T, [0.5] * wl.batch)
            out = torch.zeros((steps,) + tuple(q[0].shape), dtype=torch.bfloat16, device="cuda")
            for i in range(steps):
                step(cache, 0, q[i], kn[i], vn[i], 0.1, out[i])
            torch.cuda.synchronize()
            outs.append((out, A.arkv_cache_export(cache, 0, cfg)))
        assert torch.equal(outs[0][0], outs[1][0])
        for name in outs[0][1]:
            assert np.array_equal(outs[0][1][name], outs[1][1][name]), name
        assert A.arkv_cache_progress(caches[0], 0)[0] == 1 + steps
    finally:
        for cache in caches:
            A.arkv_cache_destroy(cache)


def test_eager_steps_behind_a_replayed_tailor():
    """A graph that holds a prompt's commit and steps through a tailor serves two prompts in turn.  The eager steps behind the
    second replay are launched before its tailor has run, when all that the host could know are the first prompt's counts: the
    same bits as without a graph."""
    T, N, steps = 400, 150, 60
    wl = synth.C1.scaled(name="replayed", n_q_heads=8, n_kv_heads=4, head_dim=64, prefill=T, batch=2, n_layers=1, budget_frac=(N + 0.5) / T)
    assert wl.capacity == N
    prompts = [synth.prefill_inputs(w, 0) for w in (wl, wl.scaled(name="replayed2", seed=wl.seed + 91))]
    q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0, steps))
    k, v, qw = (t.cuda() for t in prompts[0])
    stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
    outs = torch.zeros((steps, wl.batch, 8, 64), dtype=torch.bfloat16, device="cuda")
    cfg = make_cfg(wl)

    def ingest(cache):
        A.arkv_prefill_stats(cache, 0, qw, k, T, 0.1, stats)
        A.arkv_prefill_commit(cache, 0, k, v, T, [0.4] * wl.batch)

    def step(cache, i):
        A.arkv_decode_step(cache, 0, q[i], kn[i], vn[i], 0.1, outs[i])

    def load(i):
        for dst, src in zip((k, v, qw), prompts[i]):
            dst.copy_(src)

    graphed, plain = A.arkv_cache_create(cfg), A.arkv_cache_create(cfg)
    try:
        ingest(graphed)                                     # (the scratch of scorer and commit)
        A.arkv_cache_reset(graphed, 0)
        torch.cuda.synchronize()
        first = 0                                           # steps of the graph: up to its tailor
        s, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            ingest(graphed)
            while A.arkv_cache_progress(graphed, 0)[0] < 2:
                step(graphed, first)
                first += 1
        assert 2 < first < steps - 10
        counts = []
        busy = torch.randn(4096, 4096, device="cuda")
        for i in range(2):
            torch.cuda.synchronize()
            load(i)
            torch.cuda.synchronize()
            with torch.cuda.stream(s):
                if i == 1:
                    for _ in range(20):                     # the replay waits behind some 10 ms of work
                        busy @ busy
                graph.replay()
                if i == 1:
                    for j in range(first, steps):
                        step(graphed, j)
            torch.cuda.synchronize()
            if i == 0:
                counts.append(A.arkv_cache_counters(graphed, 0, wl.batch * 4))
        got, end = outs.clone(), A.arkv_cache_counters(graphed, 0, wl.batch * 4)
        ingest(plain)
        for j in range(steps):
            step(plain, j)
            if j == first - 1:
                counts.append(A.arkv_cache_counters(plain, 0, wl.batch * 4))
        torch.cuda.synchronize()
        assert not np.array_equal(counts[0][0], counts[1][0])            # (the prompts' counts do differ there)
        assert torch.equal(got, outs)
        assert all(np.array_equal(a, b) for a, b in zip(end, A.arkv_cache_counters(plain, 0, wl.batch * 4)))
    finally:
        A.arkv_cache_destroy(graphed)
        A.arkv_cache_destroy(plain)


def _launches(cache, step):
    """Kernels that a step launches: the nodes of the graph that captures it (which is not run, so the cache is done with)."""
    lib, s = A.load(), torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        assert lib.hipStreamBeginCapture(ctypes.c_void_p(s.cuda_stream), 2) == 0
        try:
            step()
        finally:
            assert lib.hipStreamEndCapture(ctypes.c_void_p(s.cuda_stream), ctypes.byref(graph)) == 0
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert lib.hipGraphDestroy(graph) == 0
    return n.value


def _launches_of_a_tailor(cfg, T, rho):
    """A prompt of T tokens of one layer, steps up to the first tailor behind it, and what the step that ends with it launches."""
    wl = synth.C1.scaled(name="tailor_launches", n_layers=1, batch=cfg.batch, n_q_heads=cfg.n_q_heads, n_kv_heads=cfg.n_kv_heads,
                         head_dim=cfg.head_dim, prefill=T)
    k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
    q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0, 1))
    cache = A.arkv_cache_create(cfg)
    try:
        stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
        out = torch.zeros_like(q[0])
        A.arkv_prefill_stats(cache, 0, qw, k, T, 0.1, stats)
        A.arkv_prefill_commit(cache, 0, k, v, T, [rho] * wl.batch)
        while A.arkv_cache_progress(cache, 0)[1] + 1 < cfg.capacity_tokens:
            A.arkv_decode_step(cache, 0, q[0], kn[0], vn[0], 0.1, out)
        tailors = A.arkv_cache_progress(cache, 0)[0]
        n = _launches(cache, lambda: A.arkv_decode_step(cache, 0, q[0], kn[0], vn[0], 0.1, out))
        assert A.arkv_cache_progress(cache, 0)[0] == tailors + 1
        return n
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("policy", [0, 1])
def test_tailor_of_a_small_byte_budget_goes_by_the_rows_it_can_hold(policy):
    """A unit of 250 rows' bytes holds 350 to 580 rows at most with this ratio, however many more its pools have room for: its tailor
    takes the launches of a token budget's (attention, waiting scores, and the choice that also moves; or two with kept logits)."""
    common = dict(n_layers=1, batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, capacity_tokens=250, window=32, quant_bits=2,
                  tailor_policy=policy)
    n = [_launches_of_a_tailor(A.arkv_config_default(budget_mode=m, **common), 900, 0.65) for m in (0, 1)]
    assert n[0] == n[1] == 3 - policy


@pytest.mark.parametrize("d,N,T,rho,policy,here", [
    (128, 1000, 997, 0.0, 0, False), (128, 1000, 997, 0.95, 0, True),      # some 950 rows demoted at once, and 30
    (128, 1000, 997, 0.0, 1, False), (128, 98, 95, 0.0, 0, True), (128, 99, 96, 0.0, 0, False),      # 64 and 65 of them
    (64, 160, 157, 0.0, 0, True), (64, 165, 162, 0.0, 0, False),           # 125 and 130
    (128, 384, 900, 0.5, 0, True), (128, 385, 900, 0.5, 0, False),         # the first one behind a commit that chose
    (128, 1024, 1200, 0.5, 1, True), (128, 1025, 1200, 0.5, 1, False),
])
def test_where_a_tailors_moves_are_made(d, N, T, rho, policy, here):
    """Attention, waiting scores (unless the logits are kept) and choice; two launches more unless the choosing workgroups move
    the rows, which only pays for few of them."""
    cfg = A.arkv_config_default(n_layers=1, batch=1, n_q_heads=8, n_kv_heads=2, head_dim=d, capacity_tokens=N, window=32, alpha=0.98,
                                quant_bits=4, tailor_policy=policy)
    kept = policy == 1 and T >= N
    assert _launches_of_a_tailor(cfg, T, rho) == (2 if kept else 3) + (0 if here else 2)


def _one_prompt(hq, hkv, d, W, T, seed=5):
    g = torch.Generator().manual_seed(seed)
    return tuple(torch.randn((1, h, t, d), generator=g).to(torch.bfloat16).cuda() for h, t in ((hq, W), (hkv, T)))


def _scorer_cache(hq, hkv, d, W, batch):
    return A.arkv_cache_create(A.arkv_config_default(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                                                     capacity_tokens=W + 200, window=W))


@pytest.mark.parametrize("hq,d,W,T", [(2, 64, 32, 2200), (4, 128, 20, 4000), (8, 128, 32, 4100), (8, 64, 32, 8190), (2, 128, 5, 6000)])
def test_row_constants_do_not_depend_on_the_pass_that_forms_them(hq, d, W, T):
    """From 17 to 64 chunks of 128 keys and up to 128 rows: a sequence alone, where the column pass forms the row constants, and
    among so many that a launch of its own does.  Same bits of its statistics and of every key's window sums (what a commit keeps)."""
    hkv = 2
    q, k = _one_prompt(hq, hkv, d, W, T)
    many = 640 // ((T + 127) // 128 * hkv) + 1
    got = []
    for batch in (1, many):
        cfg = A.arkv_config_default(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, capacity_tokens=T + 50, window=W)
        cache = A.arkv_cache_create(cfg)
        try:
            A.arkv_debug_set_launch_shape(cache, prefill_chunk=128)
            stats = torch.zeros((batch, 3), dtype=torch.float32, device="cuda")
            qb, kb = (x.expand(batch, -1, -1, -1).contiguous() for x in (q, k))
            A.arkv_prefill_stats(cache, 0, qb, kb, T, 0.1, stats)
            A.arkv_prefill_commit(cache, 0, kb, kb, T, [0.5] * batch)
            e = A.arkv_cache_export(cache, 0, cfg, rows=False, codes=False)
            got.append((stats.cpu().numpy(), e["s1"].reshape(batch, hkv, -1), e["s2"].reshape(batch, hkv, -1)))
        finally:
            A.arkv_cache_destroy(cache)
    for one, all_ in zip(*got):
        assert np.isfinite(one).all() and (all_.view(np.uint32) == one.view(np.uint32)).all()


@pytest.mark.parametrize("hq,hkv,W,T,launches", [
    (4, 1, 32, 16, 3), (4, 1, 32, 640, 3), (4, 1, 32, 641, 4),         # 128 rows of one unit: chunks of 128 keys
    (8, 1, 32, 320, 3), (8, 1, 32, 321, 4), (8, 1, 64, 160, 3), (8, 1, 64, 161, 4), (8, 2, 64, 32, 3), (20, 20, 32, 32, 3), (20, 20, 32, 33, 4),
])
def test_where_row_constants_are_formed(hq, hkv, W, T, launches):
    """Three launches of the scorer where the column pass forms the row constants, four where that takes longer than a launch of
    its own: many workgroups (beyond 32 chunks), fewer of them the more rows they have.  T: chunks of 128 keys."""
    T *= 128
    q, k = _one_prompt(hq, hkv, 64, W, T)
    cache = _scorer_cache(hq, hkv, 64, W, 1)
    try:
        A.arkv_debug_set_launch_shape(cache, prefill_chunk=128)
        stats = torch.zeros((1, 3), dtype=torch.float32, device="cuda")
        score = lambda: A.arkv_prefill_stats(cache, 0, q, k, T, 0.1, stats)
        score()                                             # (the scratch)
        assert _launches(cache, score) == launches
    finally:
        A.arkv_cache_destroy(cache)
