"""Causal prefill attention with the scorer fused (arkv_prefill_attention) against the oracle: every output
row on small prompts (whole prompt at once, in chunks, all group sizes, ragged lengths), sampled rows at the
32K-context size, and the fused scorer against the stand-alone one and the oracle."""
import numpy as np
import pytest
import torch

from oracle import arkv_oracle as O
from paper_2603_08727_amd import binding as A
from paper_2603_08727_amd import synth
from helpers import TOL, SideBySide, make_cfg, rel_err

pytestmark = pytest.mark.gpu


def _full_queries(wl, layer, qw):
    """Queries of the whole prompt [B][Hq][T][d]: seeded draws for positions < T - W, the workload's window
    queries for the last W positions."""
    g = torch.Generator().manual_seed(wl.seed + 1000 * layer + 77)
    q = torch.randn((wl.batch, wl.n_q_heads, wl.prefill, wl.head_dim), generator=g).to(torch.bfloat16)
    q[:, :, wl.prefill - wl.window:, :] = qw
    return q


def _attention(cache, layer, q, k, v, Tq, T, scale, out, stats=None):
    """arkv_prefill_attention with the fp32 parity hook switched on for this call: fills `out` (bf16), checks that it
    is the round-to-nearest-even of the fp32 result, and returns the fp32 result (also kept as out.f32)."""
    f32 = torch.zeros(out.shape, dtype=torch.float32, device="cuda")
    A.arkv_debug_prefill_attention_f32(cache, f32)
    try:
        A.arkv_prefill_attention(cache, layer, q, k, v, Tq, T, scale, out, stats)
        torch.cuda.synchronize()
    finally:
        A.arkv_debug_prefill_attention_f32(cache, None)
    assert torch.equal(out.view(torch.int16), f32.to(torch.bfloat16).view(torch.int16))   # torch rounds to nearest even
    out.f32 = f32
    return f32


def _check_rows(out, q, k, v, scale, group, positions, q0):
    """Rows at absolute `positions` of the GPU's fp32 output (out.f32, [B][Hq][Tq][d], before the rounding to bf16)
    against the oracle: max |x - ref| / max |ref| per head row."""
    worst = 0.0
    for b in range(q.shape[0]):
        ref = O.causal_attention_rows(synth.to_numpy_f32(q[b][:, positions - q0]), positions, synth.to_numpy_f32(k[b]),
                                      synth.to_numpy_f32(v[b]), scale, group)
        got = out.f32[b][:, positions - q0].cpu().numpy()
        for h in range(ref.shape[0]):
            for r in range(ref.shape[1]):
                worst = max(worst, rel_err(got[h, r], ref[h, r]))
    return worst


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 95, 129])
def test_attention_ends_of_tiles(d, group, T):
    """Prompts of one to five key tiles, most with a partial last one, for every shape of a thread's staging share:
    tiles are requested up to four ahead of the one in work, past the prompt's end as well, and what lies behind it
    (here NaN) takes no part."""
    hkv = 2
    cfg = make_cfg(synth.C1.scaled(name="ends", n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, batch=1))
    g = torch.Generator().manual_seed(1000 * T + 10 * group + d)
    q, k, v = (torch.randn((1, h, T, d), generator=g).to(torch.bfloat16) for h in (hkv * group, hkv, hkv))
    behind = torch.full((2, hkv * T * d + 256 * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    kd, vd = (behind[i, : hkv * T * d].view(1, hkv, T, d).copy_(x) for i, x in enumerate((k, v)))
    scale = d ** -0.5
    cache = A.arkv_cache_create(cfg)
    try:
        out = torch.zeros_like(q, device="cuda")
        _attention(cache, 0, q.cuda(), kd, vd, T, T, scale, out)
        assert torch.isfinite(out.f32).all()
        assert _check_rows(out, q, k, v, scale, group, np.arange(T), 0) <= TOL
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("hq,hkv,d,T", [(8, 2, 64, 200), (4, 4, 128, 97), (2, 1, 128, 160), (8, 1, 64, 131), (8, 2, 128, 33)])
def test_attention_small_all_rows(hq, hkv, d, T):
    wl = synth.C1.scaled(name="attn", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=2, budget_frac=2.0)
    cfg = make_cfg(wl)
    cache = A.arkv_cache_create(cfg)
    try:
        k, v, qw = synth.prefill_inputs(wl, 0)
        q = _full_queries(wl, 0, qw)
        scale = synth.softmax_scale(wl, 0)
        out = torch.zeros_like(q, device="cuda")
        _attention(cache, 0, q.cuda(), k.cuda(), v.cuda(), T, T, scale, out)
        assert _check_rows(out, q, k, v, scale, hq // hkv, np.arange(T), 0) <= TOL
        # the same prompt in three ragged chunks: keys so far, queries of the chunk
        out2 = torch.zeros_like(out)
        edges = sorted({0, min(40, T), min(41 + T // 3, T), T})
        for a, e in zip(edges[:-1], edges[1:]):
            if e <= a:
                continue
            oc = torch.zeros((wl.batch, hq, e - a, d), dtype=torch.bfloat16, device="cuda")
            A.arkv_prefill_attention(cache, 0, q[:, :, a:e].contiguous().cuda(), k[:, :, :e].contiguous().cuda(),
                                     v[:, :, :e].contiguous().cuda(), e - a, e, scale, oc)
            out2[:, :, a:e] = oc
        torch.cuda.synchronize()
        assert torch.equal(out, out2)          # a row's result does not depend on how the prompt was cut
    finally:
        A.arkv_cache_destroy(cache)


def test_fused_scorer_equals_standalone_and_oracle():
    """arkv_prefill_attention(stats=...) then commit and decode: same statistics as arkv_prefill_stats (2e-3; the
    row constants come from a different pass) and the usual state parity with the oracle afterwards."""
    wl = synth.C1.scaled(name="fused", prefill=700, decode_steps=20, batch=2, n_layers=2)

    class Fused(SideBySide):
        def prefill(self):
            super().prefill()                     # stand-alone scorer + oracle reference
            stats_alone = self.stats_gpu.copy()
            A.arkv_cache_reset(self.cache, -1)
            wl_ = self.wl
            stats = torch.zeros((wl_.n_layers, wl_.batch, 3), dtype=torch.float32, device=self.dev)
            for l in range(wl_.n_layers):
                k, v, qw = self.inputs[l]
                q = _full_queries(wl_, l, qw)
                out = torch.zeros_like(q, device=self.dev)
                _attention(self.cache, l, q.to(self.dev), k.to(self.dev), v.to(self.dev), wl_.prefill,
                           wl_.prefill, self.scales[l], out, stats[l])
                pos = np.array([0, 1, 31, 32, 333, wl_.prefill - wl_.window - 1, wl_.prefill - 2, wl_.prefill - 1])
                assert _check_rows(out, q, k, v, self.scales[l], wl_.group, pos, 0) <= TOL
            torch.cuda.synchronize()
            self.stats_gpu = stats.cpu().numpy()
            assert np.all(np.abs(self.stats_gpu - stats_alone) <= TOL * np.abs(stats_alone))
            err = np.abs(self.stats_gpu - self.stats_ref) / np.maximum(np.abs(self.stats_ref), 1e-300)
            self.max_err["stats"] = float(err.max())
            self.rho_gpu = A.arkv_oq_ratio(self.stats_gpu, wl_.tau)

    sb = Fused(wl)
    try:
        sb.prefill()
        sb.commit()
        sb.decode(check_every=5)
        sb.assert_within_tol()
    finally:
        sb.close()


def test_attention_32k_sampled_rows():
    """Config 3's prompt (32K tokens, batch 4, 32/8 heads, d = 128), one layer, whole prompt in one call; rows
    the oracle can compute one by one: first, tile borders, middle, the window, last."""
    wl = synth.C3.scaled(n_layers=1)
    cfg = make_cfg(wl)
    cache = A.arkv_cache_create(cfg)
    try:
        T = wl.prefill
        k, v, qw = synth.prefill_inputs(wl, 0)
        q = _full_queries(wl, 0, qw)
        scale = synth.softmax_scale(wl, 0)
        out = torch.zeros_like(q, device="cuda")
        stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
        _attention(cache, 0, q.cuda(), k.cuda(), v.cuda(), T, T, scale, out, stats)
        pos = np.array([0, 31, 32, 4097, 20000, T - wl.window, T - 1])
        assert _check_rows(out, q, k, v, scale, wl.group, pos, 0) <= TOL
        ref = []
        for b in range(wl.batch):
            a = O.window_attention(synth.to_numpy_f32(qw[b]), synth.to_numpy_f32(k[b]), scale, wl.group)
            ref.append(O.layer_statistics(a, wl.window)[:3])
        assert np.all(np.abs(stats.cpu().numpy() - np.array(ref)) <= TOL * np.abs(np.array(ref)))
    finally:
        A.arkv_cache_destroy(cache)


def _run_attention(wl, q, k, v, scale, Tq, T):
    """Queries q [B][Hq][Tq][d] at positions T - Tq .. T - 1 against the first T keys; returns the output."""
    cfg = make_cfg(wl)
    cache = A.arkv_cache_create(cfg)
    try:
        out = torch.zeros((wl.batch, wl.n_q_heads, Tq, wl.head_dim), dtype=torch.bfloat16, device="cuda")
        _attention(cache, 0, q.contiguous().cuda(), k[:, :, :T].contiguous().cuda(),
                   v[:, :, :T].contiguous().cuda(), Tq, T, scale, out)
        return out
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("direction", [+1.0, -1.0])
def test_attention_drifting_logits(direction):
    """Logits that rise (or fall) by about 60 binary orders over the prompt: a row's lazy reference maximum has
    to move many times, long after the first tile (or never again, with all later probabilities tiny).  Checked
    against the oracle on every row, and bit for bit against the same prompt cut into ragged chunks."""
    T, d = 300, 64
    wl = synth.C1.scaled(name="drift", n_q_heads=8, n_kv_heads=2, head_dim=d, prefill=T, batch=1, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0)
    u = torch.zeros(d); u[3] = 1.0
    ramp = torch.arange(T, dtype=torch.float32) / T                       # 0 .. 1 along the keys
    k = (k.float() + direction * 6.0 * ramp[None, None, :, None] * u).to(torch.bfloat16)
    q = (q.float() + (60.0 / (6.0 * scale * 1.4427)) * u).to(torch.bfloat16)   # q.u * scale * log2(e) * 6 = 60
    out = _run_attention(wl, q, k, v, scale, T, T)
    assert _check_rows(out, q, k, v, scale, 4, np.arange(T), 0) <= TOL
    out2 = torch.zeros_like(out)
    for a, e in [(0, 7), (7, 100), (100, 101), (101, 263), (263, T)]:
        out2[:, :, a:e] = _run_attention(wl, q[:, :, a:e], k, v, scale, e - a, e)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("Tq,T", [(20, 20), (1, 300), (5, 77), (1, 1), (33, 64), (31, 95)])
def test_attention_short_and_single_rows(Tq, T):
    """Prompts shorter than one key tile, single query rows against a long context, chunks that start off a
    tile border."""
    wl = synth.C1.scaled(name="short", n_q_heads=8, n_kv_heads=2, head_dim=128, prefill=max(T, 40), batch=2, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0)
    out = _run_attention(wl, q[:, :, T - Tq:T], k, v, scale, Tq, T)
    kk, vv = k[:, :, :T], v[:, :, :T]
    assert _check_rows(out, q[:, :, T - Tq:T], kk, vv, scale, 4, np.arange(T - Tq, T), T - Tq) <= TOL


def test_attention_whole_prompt_and_chunks_agree_bitwise_600():
    """A 601-token prompt at d = 128 (19 key tiles, the last one ragged) in one call and in four chunks of
    very different lengths: same bits, and within tolerance of the oracle on sampled rows."""
    T, d = 601, 128
    wl = synth.C1.scaled(name="paths", n_q_heads=8, n_kv_heads=2, head_dim=d, prefill=T, batch=2, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0)
    out = _run_attention(wl, q, k, v, scale, T, T)
    pos = np.array([0, 31, 32, 255, 256, 300, 599, 600])
    assert _check_rows(out, q, k, v, scale, 4, pos, 0) <= TOL
    out2 = torch.zeros_like(out)
    for a, e in [(0, 50), (50, 290), (290, 330), (330, T)]:
        out2[:, :, a:e] = _run_attention(wl, q[:, :, a:e], k, v, scale, e - a, e)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("hq,hkv,d,T", [(4, 4, 64, 992), (8, 1, 128, 961), (8, 2, 128, 930)])
def test_attention_cuts_of_the_longest_unsplit_prompts(hq, hkv, d, T):
    """Prompts of up to 992 tokens in one call and in chunks, the last ones of few queries against nearly all keys: same bits."""
    wl = synth.C1.scaled(name="cuts", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=1, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0)
    out = _run_attention(wl, q, k, v, scale, T, T)
    assert _check_rows(out, q, k, v, scale, hq // hkv, np.array([0, 500, T - 1]), 0) <= TOL
    for a in (T - 131, T - 33, T - 32, T - 1):
        assert torch.equal(out[:, :, a:], _run_attention(wl, q[:, :, a:], k, v, scale, T - a, T)), a


@pytest.mark.parametrize("seed", range(12))
def test_attention_drawn_shapes_and_chunks(seed):
    """Drawn group size, head dimension, prompt length, batch and chunking: sampled rows against the oracle and
    the chunked run bit for bit against the single call."""
    r = np.random.default_rng(500 + seed)
    hkv = int(r.choice([1, 2, 3]))
    g = int(r.choice([1, 2, 4, 8]))
    d = int(r.choice([64, 128]))
    T = int(r.integers(40, 420))
    wl = synth.C1.scaled(name=f"attn_combo{seed}", n_q_heads=hkv * g, n_kv_heads=hkv, head_dim=d, prefill=T,
                         batch=int(r.choice([1, 2])), budget_frac=2.0, seed=300 + seed)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0) * float(r.choice([0.5, 1.0, 3.0]))
    out = _run_attention(wl, q, k, v, scale, T, T)
    pos = np.unique(np.concatenate([[0, T - 1, T // 2], r.integers(0, T, 6)]))
    assert _check_rows(out, q, k, v, scale, g, pos, 0) <= TOL
    cuts = np.unique(np.concatenate([[0, T], r.integers(1, T, 3)]))
    out2 = torch.zeros_like(out)
    for a, e in zip(cuts[:-1], cuts[1:]):
        out2[:, :, a:e] = _run_attention(wl, q[:, :, a:e], k, v, scale, int(e - a), int(e))
    assert torch.equal(out, out2)


def test_fused_scorer_on_the_last_chunk_of_a_chunked_prompt():
    """The prompt in three chunks, the statistics asked for with the last one (which holds the window): same
    statistics as the stand-alone scorer, and the commit that follows accepts them."""
    wl = synth.C1.scaled(name="chunk_stats", prefill=500, batch=2, n_layers=1, decode_steps=4)
    cfg = make_cfg(wl)
    T, W = wl.prefill, wl.window
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0)
    kd, vd, qd = k.cuda(), v.cuda(), q.cuda()
    cache = A.arkv_cache_create(cfg)
    try:
        alone = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
        A.arkv_prefill_stats(cache, 0, qw.cuda(), kd, T, scale, alone)
        A.arkv_cache_reset(cache, 0)
        fused = torch.zeros_like(alone)
        out = torch.zeros_like(qd)
        out.f32 = torch.zeros(qd.shape, dtype=torch.float32, device="cuda")
        for a, e in [(0, 190), (190, 431), (431, T)]:
            oc = torch.zeros((wl.batch, wl.n_q_heads, e - a, wl.head_dim), dtype=torch.bfloat16, device="cuda")
            out.f32[:, :, a:e] = _attention(cache, 0, qd[:, :, a:e].contiguous(), kd[:, :, :e].contiguous(),
                                            vd[:, :, :e].contiguous(), e - a, e, scale, oc, fused if e == T else None)
            out[:, :, a:e] = oc
        torch.cuda.synchronize()
        sa, sf = alone.cpu().numpy(), fused.cpu().numpy()
        assert np.all(np.abs(sf - sa) <= TOL * np.abs(sa))
        pos = np.array([0, 189, 190, 430, 431, T - 1])
        assert _check_rows(out, q, k, v, scale, wl.group, pos, 0) <= TOL
        A.arkv_prefill_commit(cache, 0, kd, vd, T, A.arkv_oq_ratio(sf[None], wl.tau)[0])
        assert A.arkv_cache_progress(cache, 0)[0] == 1
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("hq,hkv,d,T", [(8, 2, 64, 700), (8, 1, 128, 333), (4, 4, 128, 1500)])
def test_scorer_with_the_callers_log_sum_exp(hq, hkv, d, T):
    """arkv_prefill_stats_lse: the window rows' normalisers come from the caller (here: the oracle's, rounded to
    fp32), the scorer reads the keys once.  Statistics against the oracle; the per-token sums it leaves behind
    against the stand-alone scorer's through the commit and a few decode steps."""
    wl = synth.C1.scaled(name="lse", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=2, n_layers=2,
                         decode_steps=12)

    class WithLse(SideBySide):
        def prefill(self):
            super().prefill()                     # stand-alone scorer + oracle reference
            A.arkv_cache_reset(self.cache, -1)
            wl_ = self.wl
            stats = torch.zeros((wl_.n_layers, wl_.batch, 3), dtype=torch.float32, device=self.dev)
            for l in range(wl_.n_layers):
                k, v, qw = self.inputs[l]
                lse = np.stack([O.window_lse(synth.to_numpy_f32(qw[b]), synth.to_numpy_f32(k[b]), self.scales[l], wl_.group)
                                for b in range(wl_.batch)])
                lse_d = torch.tensor(lse, dtype=torch.float32, device=self.dev)
                A.arkv_prefill_stats_lse(self.cache, l, qw.to(self.dev), k.to(self.dev), wl_.prefill, self.scales[l],
                                         lse_d, stats[l])
            torch.cuda.synchronize()
            self.stats_gpu = stats.cpu().numpy()
            err = np.abs(self.stats_gpu - self.stats_ref) / np.maximum(np.abs(self.stats_ref), 1e-300)
            self.max_err["stats"] = float(err.max())
            self.rho_gpu = A.arkv_oq_ratio(self.stats_gpu, wl_.tau)

    sb = WithLse(wl)
    try:
        sb.prefill()
        sb.commit()
        sb.decode(check_every=4)
        sb.assert_within_tol()
    finally:
        sb.close()


@pytest.mark.parametrize("hq,hkv,d,Tq,T,pieces", [
    (4, 1, 128, 512, 4101, (15, 16)),  # few workgroups: every workgroup in several pieces (first and last block's number)
    (8, 1, 64, 33, 2048, (8, 8)),      # group size 8, the second workgroup holds one row
    (2, 2, 64, 129, 3001, (12, 12)),   # 128-position workgroups, the second holds one row
    (4, 2, 128, 65, 1025, (4, 4)),     # 64-position workgroups at the smallest split
    (4, 1, 64, 1100, 1100, (1, 1)),    # a whole prompt too short to be split
    (4, 1, 128, 1100, 1100, (1, 4)),   # whole prompts: only the late workgroups are split
    (4, 1, 64, 2000, 2000, (1, 7)),
    (2, 1, 128, 1500, 1500, (1, 6)),   # the same with 64-position workgroups
])
def test_attention_split_over_keys(hq, hkv, d, Tq, T, pieces):
    """Launches too small for the chip cut a workgroup's keys into pieces and merge them: outputs against the oracle,
    first and last rows of every block of positions among them, and the window rows' constants through the scorer
    (same tolerances as the unsplit pass: the sums stay in fp32)."""
    assert A.arkv_debug_attention_split(d, hq // hkv, hkv, T, Tq)[2:] == pieces
    wl = synth.C1.scaled(name="split", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=1, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)[:, :, T - Tq:].contiguous()
    scale = synth.softmax_scale(wl, 0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        kd, vd, qd = k.cuda(), v.cuda(), q.cuda()
        alone, fused = (torch.zeros((1, 3), dtype=torch.float32, device="cuda") for _ in range(2))
        A.arkv_prefill_stats(cache, 0, qw.cuda(), kd, T, scale, alone)
        out = torch.zeros_like(qd)
        _attention(cache, 0, qd, kd, vd, Tq, T, scale, out, fused)
        pos = np.unique(np.clip(np.concatenate([np.arange(T - Tq, T, 32), np.arange(T - Tq + 31, T, 32), [T - 1]]), 0, T - 1))
        assert _check_rows(out, q, k, v, scale, hq // hkv, pos, T - Tq) <= TOL
        # a split pass sums the window rows' normalisers from fp32 probabilities, like the stand-alone scorer's first
        # pass: sums of up to 4101 terms in another order (1e-7 seen; 4101 * 2^-24 = 2.4e-4 is the worst case)
        sa, sf = alone.cpu().numpy(), fused.cpu().numpy()
        assert np.all(np.abs(sf - sa) <= 2.4e-4 * np.abs(sa))
        again = torch.zeros_like(out)
        A.arkv_prefill_attention(cache, 0, qd, kd, vd, Tq, T, scale, again)
        assert torch.equal(out, again)             # the cut depends on the shape alone
    finally:
        A.arkv_cache_destroy(cache)


def test_attention_split_under_graph_capture():
    """Nothing is allocated while a stream is being captured: before the scratch exists the call runs unsplit, after an
    eager call has made it the captured call is split; every replay equals the eager result of its kind."""
    T, Tq, d = 3000, 96, 128
    wl = synth.C1.scaled(name="capture", n_q_heads=4, n_kv_heads=1, head_dim=d, prefill=T, batch=1, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)[:, :, T - Tq:].contiguous()
    scale = synth.softmax_scale(wl, 0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        kd, vd, qd = k.cuda(), v.cuda(), q.cuda()
        outs = [torch.zeros_like(qd) for _ in range(3)]
        graphs = []
        for i in (0, 1):
            s = torch.cuda.Stream()
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                A.arkv_prefill_attention(cache, 0, qd, kd, vd, Tq, T, scale, outs[i])
            graphs.append(g)
            if i == 0:
                A.arkv_prefill_attention(cache, 0, qd, kd, vd, Tq, T, scale, outs[2])
                torch.cuda.synchronize()
        for _ in range(3):
            for i, g in enumerate(graphs):
                outs[i].zero_()
                g.replay()
                torch.cuda.synchronize()
                ref = outs[i].float().cpu()
                assert torch.equal(outs[1], outs[2]) or i == 0
                assert (ref - outs[2].float().cpu()).abs().max() <= 8e-3 * ref.abs().max()   # two bf16 roundings
    finally:
        A.arkv_cache_destroy(cache)


def _chunk(wl, Tq):
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)[:, :, wl.prefill - Tq:].contiguous()
    return q.cuda(), k.cuda(), v.cuda()


def test_captured_split_attention_outlives_larger_calls():
    """A graph of a split call holds the address of its scratch: larger calls afterwards take other memory, and what they
    leave for the allocator is not what the replay writes to.  Every replay equals the eager result."""
    T, d = 3000, 128
    wl = synth.C1.scaled(name="outlive", n_q_heads=4, n_kv_heads=1, head_dim=d, prefill=T, batch=1, budget_frac=2.0)
    scale = synth.softmax_scale(wl, 0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        (q, k, v), (qb, _, _), (qc, _, _) = _chunk(wl, 96), _chunk(wl, 512), _chunk(wl, 1200)
        assert all(A.arkv_debug_attention_split(d, 4, 1, T, n)[1] > 1 for n in (96, 512, 1200))
        eager, out = torch.zeros_like(q), torch.zeros_like(q)
        A.arkv_prefill_attention(cache, 0, q, k, v, 96, T, scale, eager)          # the scratch of this size
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            A.arkv_prefill_attention(cache, 0, q, k, v, 96, T, scale, out)
        for big in (qb, qc):
            ref = torch.zeros_like(big)
            A.arkv_prefill_attention(cache, 0, big, k, v, big.shape[2], T, scale, ref)
            torch.cuda.synchronize()
            # the rows both calls have differ by their cut only
            assert (ref[:, :, -96:].float() - eager.float()).abs().max() <= 8e-3 * eager.float().abs().max()
            spare = torch.full((8 << 20,), 7.0, device="cuda")                     # would reuse a freed block
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager)
            assert bool((spare == 7.0).all())
            del spare
    finally:
        A.arkv_cache_destroy(cache)


def test_split_attention_beside_a_capture_on_another_stream():
    """The first split call of a cache allocates its scratch.  It may do so while another stream is being captured (in
    torch's default mode, which forbids the allocations of every thread): the capture stays whole, the call is split."""
    T, Tq, d = 3000, 96, 128
    wl = synth.C1.scaled(name="beside", n_q_heads=4, n_kv_heads=1, head_dim=d, prefill=T, batch=1, budget_frac=2.0)
    scale = synth.softmax_scale(wl, 0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        q, k, v = _chunk(wl, Tq)
        first, later = torch.zeros_like(q), torch.zeros_like(q)
        x = torch.zeros(1000, device="cuda")
        captured, other = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=captured):
            x += 1
            with torch.cuda.stream(other):
                A.arkv_prefill_attention(cache, 0, q, k, v, Tq, T, scale, first)
            x += 1
        torch.cuda.synchronize()
        A.arkv_prefill_attention(cache, 0, q, k, v, Tq, T, scale, later)
        for i in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert bool((x == 2 * (i + 1)).all())
        assert torch.equal(first, later)
    finally:
        A.arkv_cache_destroy(cache)


def test_attention_units_in_groups():
    """Units whose keys and values together exceed the last-level cache go in groups, here of eight and of four of the
    twelve: every row is written, sampled rows of every unit (first and last of a block of positions) against the oracle."""
    T, d, batch, hkv = 16500, 128, 3, 4
    units, rows = batch * hkv, 128                       # group size 1: workgroups of 128 positions
    n_blocks = (T + rows - 1) // rows
    assert A.arkv_debug_attention_split(d, 1, units, T, T)[0] == 0
    assert A.arkv_debug_attention_block(d, units, T, n_blocks, 0, 8)[0] == 0       # the ninth workgroup: the first unit again
    wl = synth.C1.scaled(name="groups", n_q_heads=hkv, n_kv_heads=hkv, head_dim=d, prefill=T, batch=batch, budget_frac=0.1)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)
    scale = synth.softmax_scale(wl, 0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        out = torch.full_like(q, float("nan"), device="cuda")
        _attention(cache, 0, q.cuda(), k.cuda(), v.cuda(), T, T, scale, out)
        assert bool(torch.isfinite(out).all())
        assert _check_rows(out, q, k, v, scale, 1, np.array([0, 127, 128, 4095, 8000, 16383, 16384, T - 1]), 0) <= TOL
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("d,hkv,batch,Tq,T", [
    (64, 3, 3, 70, 70),        # nine units: the shares of eight lie apart, those of the ninth side by side
    (128, 5, 2, 33, 300),      # ten units, a chunk whose second workgroup holds one row
    (128, 3, 3, 40, 2100),     # nine units, split over the keys
    (128, 2, 1, 8200, 8200),   # two units of a prompt long enough for eight heads per workgroup
    (128, 8, 4, 480, 11000),   # 32 units in two groups, four heads, not split
    (64, 8, 2, 770, 2000),     # 400 blocks of nearly the same length: eight heads, two workgroups per CU
])
def test_attention_heads_of_a_workgroup(d, hkv, batch, Tq, T):
    """Group size 8: workgroups of four heads (eight for long prompts that fill the chip, and where that saves a round).  Every row of every head is
    written, sampled rows of all heads against the oracle."""
    g = 8
    wl = synth.C1.scaled(name="heads", n_q_heads=g * hkv, n_kv_heads=hkv, head_dim=d, prefill=T, batch=batch, budget_frac=2.0)
    k, v, qw = synth.prefill_inputs(wl, 0)
    q = _full_queries(wl, 0, qw)[:, :, T - Tq:].contiguous()
    scale = synth.softmax_scale(wl, 0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        out = torch.full_like(q, float("nan"), device="cuda")
        _attention(cache, 0, q.cuda(), k.cuda(), v.cuda(), Tq, T, scale, out)
        assert bool(torch.isfinite(out).all())
        pos = np.unique(np.clip([T - Tq, T - Tq + 31, T - Tq + 32, T - Tq // 2, T - 1], T - Tq, T - 1))
        assert _check_rows(out, q, k, v, scale, g, pos, T - Tq) <= TOL
    finally:
        A.arkv_cache_destroy(cache)
