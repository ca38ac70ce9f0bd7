"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle, element by element on
the same seeded inputs.  Integer results (positions, states, codes, fp16 scale/zero bits, counts,
bf16 rows) must be identical; floating-point results within 2e-3 (helpers.TOL)."""
import numpy as np
import pytest
import torch

from paper_2603_08727_amd import binding as A
from paper_2603_08727_amd import synth
from helpers import SideBySide, make_cfg
from oracle import arkv_oracle as O

pytestmark = pytest.mark.gpu


def _run(wl, rho=None, steps=None, check_every=4, stats=True, **kw):
    sb = SideBySide(wl, rho_override=rho, **kw)
    try:
        sb.prefill()
        sb.commit()
        sb.decode(steps, check_every=check_every)
        print(wl.name, {k: f"{v:.2e}" for k, v in sb.max_err.items()}, flush=True)
        sb.assert_within_tol(stats=stats)
        # the OQ ratios computed from GPU statistics agree with the oracle's
        assert np.abs(sb.rho_gpu - sb.rho_ref).max() <= 2e-3
        return sb
    finally:
        sb.close()


def test_c1_small_lockstep():
    """Config 1 exactly: 1 layer, 8/2 heads, d=64, T=512, N=128, 64 steps, 4-bit."""
    sb = _run(synth.C1, check_every=1)
    assert sb.oracles[(0, 0)].n_tailors == 1 + 64 // 24


def test_below_budget_no_tailor():
    wl = synth.C1.scaled(name="below", prefill=100, budget_frac=3.0, decode_steps=40)
    sb = _run(wl)
    assert sb.oracles[(0, 0)].n_tailors == 0


def test_fills_up_during_decode():
    wl = synth.C1.scaled(name="fills", prefill=100, budget_frac=1.2, decode_steps=50)   # N = 120
    sb = _run(wl, check_every=1)
    assert sb.oracles[(0, 0)].n_tailors >= 1


@pytest.mark.parametrize("rho", [0.0, 1.0, 0.3])
def test_c1_forced_ratio(rho):
    _run(synth.C1.scaled(name=f"c1_rho{rho}", decode_steps=30), rho=rho)


def test_llama_shape_scaled_4bit():
    """Config 2's shape (d=128, 32/8 heads) at reduced length, 2 layers so the OQ ratios differ."""
    wl = synth.C2.scaled(name="c2_scaled", n_layers=2, prefill=1000, budget_frac=0.25, decode_steps=70)
    _run(wl)


def test_qwen_shape_scaled_batched_temperature():
    wl = synth.C3.scaled(name="c3_scaled", n_layers=2, batch=2, prefill=777, budget_frac=0.26, decode_steps=60)
    _run(wl)


def test_long_context_shape_scaled_2bit():
    wl = synth.C4.scaled(name="c4_scaled", n_layers=1, prefill=2048, budget_frac=0.125, decode_steps=40,
                         heavy_frac=0.01)
    _run(wl)


@pytest.mark.parametrize("hq,hkv,d,bits", [(8, 1, 64, 4), (2, 2, 128, 2), (4, 2, 64, 2), (8, 8, 128, 4),
                                           (8, 2, 128, 8), (4, 2, 64, 8), (8, 1, 64, 8)])
def test_group_sizes(hq, hkv, d, bits):
    wl = synth.C1.scaled(name=f"g{hq // hkv}_d{d}_b{bits}", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, bits=bits,
                         prefill=300, budget_frac=0.3, decode_steps=30)
    _run(wl)


def test_every_step_policy():
    """tailor_policy 1: no slack, the cache stays full and a tailor runs at every decode step."""
    wl = synth.C1.scaled(name="every_step", decode_steps=24)
    sb = _run(wl, rho=0.4, check_every=1, every_step=True)
    oc = sb.oracles[(0, 0)]
    assert oc.n_tailors == 1 + wl.decode_steps and oc.b == wl.capacity - wl.window - 1
    assert all(len(u.pos) == wl.capacity - 1 for u in oc.units)


@pytest.mark.parametrize("seed,bits,every_step", [(0, 4, False), (5, 2, False), (11, 8, False), (3, 4, True)])
def test_free_running_protocol(seed, bits, every_step):
    """No score hand-over: the oracle ranks on its own fp64 scores, the GPU on its fp32 scores.  After every
    tailor the two choices are compared under the score-band rule: a token may end in a different state only if
    its score is within 2e-3 of the score at the n_o cut or at the b cut."""
    wl = synth.C1.scaled(name=f"free_running_s{seed}", decode_steps=60, bits=bits, seed=seed,
                         head_dim=128 if bits == 8 else 64)
    sb = _run(wl, check_every=6, lockstep=False, every_step=every_step)
    assert sb.band_tailors == (61 if every_step else 3) * wl.batch
    print("tailors", sb.band_tailors, "with near-tie differences", sb.band_divergences, flush=True)


@pytest.mark.parametrize("seed", range(40))
def test_drawn_combinations_free_running(seed):
    """The drawn combinations again without the score hand-over (score-band rule at every tailor)."""
    wl, rho, kw = _combo(seed)
    if wl.capacity <= wl.window + 2:
        wl = wl.scaled(budget_frac=0.6)
    sb = _run(wl, rho=rho, check_every=3, lockstep=False, **kw)
    print(wl.name, "tailors", sb.band_tailors, "with near-tie differences", sb.band_divergences, flush=True)


def test_wide_window():
    """Observation window of 128: G*W = 512 query rows per unit, 16 row tiles in the prefill scorer."""
    wl = synth.C1.scaled(name="wide_window", window=128, prefill=1500, decode_steps=12)
    _run(wl, check_every=4)


@pytest.mark.parametrize("rho", [0.0, 0.5])
def test_fp8_rows(rho):
    """The paper's own Quantized format: fp8 codes with one scale per token row."""
    wl = synth.C1.scaled(name="fp8", bits=8, head_dim=128, decode_steps=60)
    _run(wl, rho=rho, check_every=6)


@pytest.mark.parametrize("bits,rho", [(4, 0.3), (8, 0.0), (2, 0.6)])
def test_byte_budget_mode(bits, rho):
    """eq. 1 in bytes: Quantized tokens are charged C_quant, more of them are kept; live bytes stay within
    N * C_orig (checked in compare_state) and everything else matches the oracle as in token mode."""
    wl = synth.C1.scaled(name=f"bytes_b{bits}", bits=bits, head_dim=128, decode_steps=70)
    sb = _run(wl, rho=rho, check_every=5, byte_budget=True)
    oc = sb.oracles[(0, 0)]
    assert oc.b > oc.b_rows and oc.n_tailors >= 3
    assert max(sum(oc.counts(g)) for g in range(wl.n_kv_heads)) > wl.capacity * 3 // 4   # more tokens than the token rule keeps


@pytest.mark.parametrize("bits", [4, 8])
def test_degenerate_rows_and_queries(bits):
    """All-zero and constant K / V rows (scale 0, constant groups), a decode step with an all-zero query
    (uniform attention), a new token whose key and value are zero; everything is demoted (rho = 0) so the
    degenerate rows go through the quantiser."""
    def mp(layer, k, v, qw):
        k[:, :, 10:14, :] = 0.0                      # zero key rows
        v[:, :, 10:12, :] = 0.0                      # zero value rows
        v[:, :, 20:24, :] = 1.5                      # constant value rows: every group is constant
        k[:, :, 30, 32:64] = -2.0                    # one constant group inside a row
        qw[:, :, 5, :] = 0.0                         # a zero query row inside the window

    def md(layer, q, kn, vn):
        q[3] = 0.0                                   # zero query at step 3
        kn[5] = 0.0; vn[5] = 0.0                     # zero new token at step 5

    wl = synth.C1.scaled(name=f"degenerate_b{bits}", bits=bits, head_dim=64, decode_steps=40)
    _run(wl, rho=0.0, check_every=2, mutate_prefill=mp, mutate_decode=md)


def _combo(seed):
    """One drawn combination of shape, format, policy and hyper-parameters (the draw is seeded: fixed cases)."""
    r = np.random.default_rng(1000 + seed)
    hkv = int(r.choice([1, 2, 4]))
    g = int(r.choice([1, 2, 4, 8]))
    d = int(r.choice([64, 128]))
    bits = int(r.choice([2, 4, 8]))
    window = int(r.choice([8, 16, 32]))
    prefill = int(r.integers(window + 40, 700))
    frac = float(r.choice([0.2, 0.35, 0.6, 1.5]))
    alpha = float(r.choice([0.5, 0.75, 0.9, 1.0]))
    rho = r.choice([None, 0.0, 0.3, 0.7, 1.0])
    wl = synth.C1.scaled(name=f"combo{seed}", n_layers=int(r.choice([1, 2])), batch=int(r.choice([1, 2, 3])),
                         n_q_heads=hkv * g, n_kv_heads=hkv, head_dim=d, bits=bits, window=window, prefill=prefill,
                         budget_frac=frac, alpha=alpha, decode_steps=int(r.integers(20, 60)), seed=77 + seed)
    kw = dict(every_step=bool(r.random() < 0.25), byte_budget=bool(r.random() < 0.3))
    return wl, (None if rho is None else float(rho)), kw


@pytest.mark.parametrize("seed", range(40))
def test_drawn_combinations(seed):
    """Shapes, formats, windows, slack factors, ratios and policies in combinations no other test names."""
    wl, rho, kw = _combo(seed)
    if wl.capacity <= wl.window + 2:
        wl = wl.scaled(budget_frac=0.6)
    print(wl, rho, kw, flush=True)
    _run(wl, rho=rho, check_every=3, **kw)


@pytest.mark.parametrize("bits,every_step", [(4, False), (8, False), (2, True)])
def test_long_run_many_tailors(bits, every_step):
    """600 decode steps on a small cache: about 25 tailors (600 under the every-step policy), the ring of waiting
    steps wraps dozens of times, the host's token counts are refreshed after every tailor."""
    wl = synth.C1.scaled(name=f"long_b{bits}", bits=bits, head_dim=128 if bits == 8 else 64, decode_steps=600)
    sb = _run(wl, rho=0.5, check_every=37, every_step=every_step)
    oc = sb.oracles[(0, 0)]
    assert oc.n_tailors >= (600 if every_step else 20)


@pytest.mark.parametrize("hq,hkv", [(8, 2), (16, 2), (2, 2)])
def test_many_splits_per_unit(hq, hkv):
    """Two units with 17K live tokens each: the launch uses 128 splits per unit, so the merging workgroup
    reduces the splits' maxima and sums over two keys per lane and fetches the partials in several batches."""
    wl = synth.C1.scaled(name=f"splits_g{hq // hkv}", n_q_heads=hq, n_kv_heads=hkv, head_dim=128, prefill=17000,
                         budget_frac=1.1, decode_steps=10)
    sb = _run(wl, check_every=3)
    assert sb.oracles[(0, 0)].n_tailors == 0


@pytest.mark.parametrize("delta", [-1, 0, 1])
def test_prompt_that_exactly_fills_the_cache(delta):
    """T = N - 1 (no tailor at commit, the first decode step fills the cache), T = N and T = N + 1 (tailor at
    commit): the first append always has room."""
    T = 128 + delta
    wl = synth.C1.scaled(name=f"exact{delta:+d}", prefill=T, budget_frac=128.5 / T, decode_steps=30)
    assert wl.capacity == 128
    sb = _run(wl, check_every=1)
    assert sb.oracles[(0, 0)].n_tailors == 2


@pytest.mark.parametrize("which", ["zero_queries", "identical_keys"])
def test_uniform_attention_statistics(which):
    """Closed form (eqs. 3-5): when every window row attends uniformly the aggregated key distribution is uniform,
    the entropy is ln(T - W), the variance exactly 0 and the kurtosis 0 by the degenerate-case reading; with every
    layer like that every OQ ratio is 1."""
    import math
    import torch
    from paper_2603_08727_amd import binding as A
    from helpers import make_cfg
    wl = synth.C1.scaled(name="uniform", prefill=300, n_layers=2, batch=2)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        stats = torch.zeros((wl.n_layers, wl.batch, 3), dtype=torch.float32, device="cuda")
        for l in range(wl.n_layers):
            k, v, qw = synth.prefill_inputs(wl, l)
            if which == "zero_queries":
                qw = torch.zeros_like(qw)
            else:
                k = k[:, :, :1, :].expand_as(k).contiguous()
            A.arkv_prefill_stats(cache, l, qw.cuda(), k.cuda(), wl.prefill, synth.softmax_scale(wl, l), stats[l])
        torch.cuda.synchronize()
        s = stats.cpu().numpy()
        n = wl.prefill - wl.window
        assert np.allclose(s[..., 0], math.log(n), rtol=1e-6)
        assert (s[..., 1] == 0).all() and (s[..., 2] == 0).all()
        assert (A.arkv_oq_ratio(s, wl.tau) == 1.0).all()
    finally:
        A.arkv_cache_destroy(cache)


def test_one_hot_attention_statistics():
    """Closed form (eqs. 3-5): when every window row puts all its weight on one prompt key, the aggregated
    distribution is one-hot: entropy 0, variance (n - 1) / n^2, kurtosis m4 / m2^2 with
    m4 = ((1 - 1/n)^4 + (n - 1) / n^4) / n, n = T - W."""
    import torch
    from paper_2603_08727_amd import binding as A
    from helpers import make_cfg
    wl = synth.C1.scaled(name="one_hot", prefill=400, n_layers=1, batch=2)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        k, v, qw = synth.prefill_inputs(wl, 0)
        k = torch.zeros_like(k); qw = torch.zeros_like(qw)
        qw[..., 0] = 64.0                                    # logit 64 * 64 / sqrt(d) on the chosen key, 0 elsewhere
        k[0, :, 137, 0] = 64.0                               # sequence 0: key 137; sequence 1: key 5
        k[1, :, 5, 0] = 64.0
        stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
        A.arkv_prefill_stats(cache, 0, qw.cuda(), k.cuda(), wl.prefill, synth.softmax_scale(wl, 0), stats)
        torch.cuda.synchronize()
        s = stats.cpu().numpy().astype(np.float64)
        n = wl.prefill - wl.window
        m2 = (n - 1) / n ** 2
        m4 = ((1 - 1 / n) ** 4 + (n - 1) / n ** 4) / n
        assert (s[:, 0] == 0).all()
        assert np.allclose(s[:, 1], m2, rtol=1e-6) and np.allclose(s[:, 2], m4 / m2 ** 2, rtol=1e-6)
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("T,N,every_step,steps", [
    (2600, 900, False, 4),      # commit over three rounds of 1024 positions, the last one ragged
    (2600, 2100, True, 6),      # tailors over three rounds, every step
    (33200, 33000, True, 2),    # more rows than a unit's scores take in LDS: commit and tailor from memory
])
def test_selection_among_equal_scores(T, N, every_step, steps):
    """Every key of the prompt is the same row, so the scores of all tokens outside the window tie and both ranks are
    decided by the position alone (R15: the older token first); the new tokens differ.  States are compared exactly."""
    def same_keys(layer, k, v, qw):
        k[:] = k[:, :, :1]

    wl = synth.C1.scaled(name="ties", n_q_heads=2, n_kv_heads=1, head_dim=64, prefill=T, budget_frac=(N + 0.5) / T, window=16,
                         decode_steps=steps)
    sb = SideBySide(wl, rho_override=0.4, every_step=every_step, mutate_prefill=same_keys)
    try:
        sb.prefill()
        sb.commit()
        sb.decode(check_every=steps)
        # (a uniform distribution's variance is 0 up to rounding, so its relative error says nothing here; the statistics
        # of uniform attention have a test of their own)
        sb.assert_within_tol(stats=False)
    finally:
        sb.close()


@pytest.mark.parametrize("batch,hkv,g,rho", [
    (3, 3, 1, 0.5),     # 9 units: one workgroup per CU allows 28 splits, the rows allow 6; one merging wave per split
    (5, 5, 2, 1.0),     # 25 units
    (5, 8, 4, 1.0),     # 40 units without packed rows: one workgroup per CU
    (5, 8, 4, 0.4),     # 40 units with packed rows: two
    (9, 8, 1, 0.4),     # 72 units: more than the launch carries counts for
])
def test_split_factors_by_units(batch, hkv, g, rho):
    """Unit counts at which the split factor rounds differently, over eight steps (one of them updates the scores)."""
    wl = synth.C1.scaled(name=f"units{batch * hkv}", batch=batch, n_q_heads=hkv * g, n_kv_heads=hkv, head_dim=128, prefill=700,
                         budget_frac=0.7, window=16, decode_steps=9)
    _run(wl, rho=rho, check_every=9)


@pytest.mark.parametrize("bits", [0x7FC00000, 0xFFC00000, 0x7FFFFFFF, 0xFFFFFFFF])
def test_selection_among_nan_scores(bits):
    """A window row without a finite normaliser (here a caller's NaN log-sum-exp) makes every score of its kv-head a NaN.
    The scores are then ranked by their bits, the older token first, whatever sign and payload they carry: a NaN must not
    be mistaken for a row that is not ranked.  Counts and states follow from the scores that were ranked on."""
    T, N, W, rho, steps = 2300, 1100, 16, 0.5, 20
    wl = synth.C1.scaled(name="nan", n_q_heads=4, n_kv_heads=2, head_dim=64, prefill=T, budget_frac=(N + 0.5) / T, window=W,
                         decode_steps=steps)
    cfg = make_cfg(wl, every_step=True)
    n_o, n_q, b = A.arkv_budget_counts(cfg, rho)
    k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
    q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0, steps))
    scale = synth.softmax_scale(wl, 0)
    lse = torch.full((1, 4, W), 8.0, device="cuda")
    lse.view(torch.int32)[0, 1, 3] = bits - (1 << 32) if bits >> 31 else bits           # a head of kv-head 0
    stats = torch.zeros((1, 3), device="cuda")
    cache = A.arkv_cache_create(cfg)
    try:
        A.arkv_prefill_stats_lse(cache, 0, qw, k, T, scale, lse, stats)
        A.arkv_prefill_commit(cache, 0, k, v, T, [rho])
        cnt, pos, score = A.arkv_debug_last_tailor_scores(cache, 0, 2, T)
        ex = A.arkv_cache_export(cache, 0, cfg, rows=False, codes=False)
        for u in range(2):
            assert cnt[u] == T - W and bool(np.isnan(score[u, :cnt[u]]).all()) == (u == 0)
            order = np.lexsort((pos[u, :cnt[u]], -score[u, :cnt[u]].view(np.uint32).astype(np.int64)))
            want = {int(p): 0 for p in range(T - W, T)}
            want.update({int(pos[u, i]): 0 for i in order[:n_o]})
            want.update({int(pos[u, i]): 1 for i in order[n_o:b]})
            assert ex["n_live"][u] == b + W
            assert dict(zip(ex["pos"][u, : b + W].tolist(), ex["state"][u, : b + W].tolist())) == want
        out = torch.zeros((1, 4, 64), dtype=torch.bfloat16, device="cuda")
        for t in range(steps):
            A.arkv_decode_step(cache, 0, q[t], kn[t], vn[t], scale, out)
        orig, quant, evicted, _ = A.arkv_cache_counters(cache, 0, 2)
        assert (orig + quant == b + W).all() and (orig >= W).all() and (evicted == T + steps - b - W).all()
        ex = A.arkv_cache_export(cache, 0, cfg, rows=False, codes=False)
        for u in range(2):
            p, st = ex["pos"][u, : b + W], ex["state"][u, : b + W]
            assert len(set(p.tolist())) == b + W and (p[-W:] == np.arange(T + steps - W, T + steps)).all()
            assert (st[-W:] == 0).all() and (st == 0).sum() == orig[u]
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("kind,every_step", [("two", False), ("mostly", False), ("mostly", True), ("late", True)])
def test_selection_among_few_distinct_scores(kind, every_step):
    """Few distinct keys: whole waves meet on one or two bins of the selection, in all of its rounds or in some, with the
    two ranks in the same bin and in different ones.  States are compared exactly."""
    T, N, steps = 3100, 1300, 4

    def few_keys(layer, k, v, qw):
        i = torch.arange(T)
        if kind == "two":
            k[:] = k[:, :, :2].repeat(1, 1, T // 2 + 1, 1)[:, :, :T]
        else:
            same = i % 10 != 3 if kind == "mostly" else i >= 1100
            k[:, :, same] = k[:, :, :1]

    wl = synth.C1.scaled(name="few", n_q_heads=4, n_kv_heads=2, head_dim=64, prefill=T, budget_frac=(N + 0.5) / T, window=16,
                         decode_steps=steps)
    sb = SideBySide(wl, rho_override=0.3, every_step=every_step, mutate_prefill=few_keys)
    try:
        sb.prefill()
        sb.commit()
        sb.decode(check_every=steps)
        sb.assert_within_tol(stats=False)
    finally:
        sb.close()


@pytest.mark.parametrize("T,N,g,d,bits,batch,rho", [
    (1024, 700, 4, 128, 4, 1, 0.0),      # one whole block, in parts of eight rows, all packed
    (1025, 900, 2, 64, 8, 3, 1.0),       # the last block holds one position (window)
    (2049, 2049, 1, 128, 2, 1, 0.5),     # T = N: nothing but the slack is evicted, parts larger than their block's last
    (65536, 2000, 1, 64, 4, 1, 0.4),     # 64 blocks and the totals: one entry more than a wave looks at together
    (66100, 9000, 2, 64, 4, 2, 0.7),     # 65 blocks
])
def test_commit_in_parts(T, N, g, d, bits, batch, rho):
    """Survivors by parts of blocks of 1024 positions: positions, states, rows and codes are compared exactly."""
    wl = synth.C1.scaled(name="parts", batch=batch, n_q_heads=2 * g, n_kv_heads=2, head_dim=d, bits=bits, prefill=T,
                         budget_frac=(N + 0.5) / T, window=16, decode_steps=2)
    _run(wl, rho=rho, check_every=2, stats=False)


@pytest.mark.parametrize("T,g,d,batch", [(17, 1, 64, 1), (1000, 4, 128, 1), (1025, 2, 64, 3), (4099, 8, 128, 2)])
def test_commit_of_a_prompt_that_fits(T, g, d, batch):
    """Every row is copied as it lies, the last round of a workgroup's rows ragged: compared exactly."""
    wl = synth.C1.scaled(name="fits", batch=batch, n_q_heads=2 * g, n_kv_heads=2, head_dim=d, prefill=T, budget_frac=(T + 60.5) / T,
                         window=16, decode_steps=2)
    _run(wl, check_every=2)


@pytest.mark.parametrize("hkv,g,d,T", [(2, 8, 128, 5000), (1, 1, 64, 20100), (1, 4, 64, 45000)])
def test_split_factors_of_few_units(hkv, g, d, T):
    """Launches of one and two units, whose splits are limited by their number (48, 64) or by the rows per split."""
    wl = synth.C1.scaled(name=f"few{hkv}", n_q_heads=hkv * g, n_kv_heads=hkv, head_dim=d, prefill=T, budget_frac=1.01, window=16,
                         decode_steps=9)
    _run(wl, check_every=9)


@pytest.mark.parametrize("g,d,T,budget,rho,bits", [
    (4, 128, 234, 2.0, 0.5, 4),       # grows over 240 rows: one split, then more; all bf16
    (8, 64, 330, 2.0, 0.5, 4),        # 336 rows at d = 64
    (1, 64, 20, 3.0, 0.5, 4),         # waves without rows
    (2, 128, 500, 0.42, 0.3, 2),      # packed rows in the only split
    (8, 128, 500, 0.42, 0.3, 8),
])
def test_single_split(g, d, T, budget, rho, bits):
    """Units of few rows are one workgroup's work, output included: over 18 steps, two of which update the scores."""
    wl = synth.C1.scaled(name="single", batch=2, n_q_heads=2 * g, n_kv_heads=2, head_dim=d, prefill=T, budget_frac=budget,
                         bits=bits, window=16, decode_steps=18)
    _run(wl, rho=rho, check_every=6)


@pytest.mark.parametrize("g,d,bits,N,rho,one", [
    (4, 128, 2, 240, 0.0, False),     # 184 to 239 rows booked, about 1000 held
    (1, 128, 4, 230, 0.1, False),
    (8, 64, 2, 330, 0.2, False),
    (4, 128, 8, 190, 0.2, True),      # up to 282 rows held
    (2, 64, 4, 250, 0.4, True),       # up to 429
    (4, 128, 4, 230, 1.0, True),      # none packed: 230
])
def test_split_of_a_byte_budget(g, d, bits, N, rho, one):
    """Under a byte budget a unit holds more rows than are booked for it: whether one workgroup takes all of them goes by
    what it can hold.  A step's output is, bit for bit, that of a cache whose split factor is set to the one expected."""
    hkv, W, T = 4, 16, 1500
    wl = synth.C1.scaled(name="bytes", n_q_heads=hkv * g, n_kv_heads=hkv, head_dim=d, prefill=T, budget_frac=(N + 0.5) / T,
                         window=W, bits=bits, batch=1, n_layers=1, decode_steps=N - int(0.75 * (N - W)) - W - 1)
    k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
    q, kn, vn = (t.cuda() for t in synth.decode_inputs(wl, 0, wl.decode_steps))
    out = torch.empty((1, hkv * g, d), dtype=torch.bfloat16, device="cuda")
    caches = [A.arkv_cache_create(make_cfg(wl, byte_budget=True)) for _ in range(2)]
    try:
        for c in caches:
            A.arkv_prefill_stats(c, 0, qw, k, T, d ** -0.5, torch.zeros((1, 3), device="cuda"))
            A.arkv_prefill_commit(c, 0, k, v, T, np.full(1, rho, np.float32))
        for t in range(wl.decode_steps):
            splits = 1 if one else max(1, A.arkv_cache_progress(caches[1], 0)[1] // 64)
            A.arkv_debug_set_launch_shape(caches[1], splits * hkv)
            f32 = []
            for c in caches:
                A.arkv_decode_step(c, 0, q[t], kn[t], vn[t], d ** -0.5, out)
                f32.append(A.arkv_debug_last_out_f32(c, 0, tuple(out.shape)))
            assert np.array_equal(f32[0].view(np.uint32), f32[1].view(np.uint32)), t
        assert splits == (1 if one else (N - 2) // 64)
        assert A.arkv_cache_progress(caches[0], 0)[0] == 1          # the commit's tailor only
    finally:
        for c in caches:
            A.arkv_cache_destroy(c)


@pytest.mark.parametrize("T,N,gain,steps", [
    (3100, 1300, 2.0 ** -17, 4),       # scores a few units in the last place apart: most tie, the range takes few bits
    (3100, 1300, 2.0 ** -10, 4),       # one digit and a little more
    (4097, 1025, 2.0 ** -5, 0),        # a position behind a whole round of the selection
    (33000, 900, 2.0 ** -12, 0),       # scores read back from memory
])
def test_selection_in_a_narrow_range_of_scores(T, N, gain, steps):
    """Nearly uniform attention: all scores of a unit lie within few representable values, so the selection starts with
    short digits and reaches the positions early.  States are compared exactly, of the commit and of a tailor per step.  (No
    steps over long caches: there the mean of many values nearly cancels, and the 2e-3 of its maximum is less than the fp16
    weights of packed rows give, with any selection.)"""
    def flat(layer, k, v, qw):
        qw *= gain

    def flat_steps(layer, q, kn, vn):
        q *= gain

    wl = synth.C1.scaled(name="narrow", n_q_heads=4, n_kv_heads=2, head_dim=64, prefill=T, budget_frac=(N + 0.5) / T, window=16,
                         decode_steps=steps)
    sb = SideBySide(wl, rho_override=0.3, every_step=steps > 0, mutate_prefill=flat, mutate_decode=flat_steps)
    try:
        sb.prefill()
        sb.commit()
        if steps:
            sb.decode(check_every=4)
        sb.assert_within_tol(stats=False)
    finally:
        sb.close()


@pytest.mark.parametrize("g,d,bits,T,N,rho,byte_budget", [
    (1, 128, 8, 600, 300, 0.3, False),
    (2, 64, 2, 1500, 1100, 0.0, False),       # rows of both pools in every round, all candidates packed
    (8, 128, 4, 700, 90, 0.5, False),         # one split per unit
    (8, 64, 8, 900, 400, 0.4, True),          # more rows than the token rule keeps
    (4, 128, 4, 5000, 4200, 0.6, False),      # two rounds of 4096 rows
    (2, 64, 4, 33400, 33000, 0.9, False),     # rows' scores in memory
])
def test_tailor_from_kept_logits(g, d, bits, T, N, rho, byte_budget):
    """With a tailor at every step the scores' update takes the step's logits from the attention launch, and from the 17th
    tailor on (up to 1024 rows: from the first behind the commit) the choosing workgroup moves the rows: 19 steps against the
    oracle, states and rows exactly."""
    wl = synth.C1.scaled(name="kept", n_q_heads=2 * g, n_kv_heads=2, head_dim=d, bits=bits, prefill=T, budget_frac=(N + 0.5) / T,
                         window=16, decode_steps=19)
    _run(wl, rho=rho, check_every=6, stats=False, every_step=True, byte_budget=byte_budget)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [1500, 1090])          # with a tailor at the commit; a prompt that fits its cache
def test_natural_cadence_above_a_small_cache(T, d, bits):
    """Tailors of more than 1024 rows at their natural cadence move rows in two launches over the whole chip: every row format and
    both head dimensions, through two tailors, states and rows exactly."""
    wl = synth.C1.scaled(name="natural", n_q_heads=4, n_kv_heads=2, head_dim=d, bits=bits, prefill=T, budget_frac=1100.5 / T, alpha=0.98,
                         decode_steps=46 if T > 1100 else 34)
    assert wl.capacity == 1100
    sb = _run(wl, rho=0.4, check_every=12)
    assert sb.oracles[(0, 0)].n_tailors == (3 if T > 1100 else 2)


@pytest.mark.parametrize("n", [1024, 1025])
def test_natural_cadence_at_the_line_of_small_caches(n):
    """1024 rows: the choosing workgroup makes the moves from the fifth tailor on (the commit's is the first), before that two
    launches do; 1025 rows: always the launches.  Through six tailors."""
    wl = synth.C1.scaled(name="line", n_q_heads=4, n_kv_heads=2, head_dim=64, prefill=1400, budget_frac=(n + 0.5) / 1400, alpha=0.99,
                         decode_steps=58)
    assert wl.capacity == n
    sb = _run(wl, rho=0.3, check_every=10)
    assert sb.oracles[(0, 0)].n_tailors >= 6


@pytest.mark.parametrize("every_step", [False, True])
def test_byte_budget_whose_rows_fit_lds_though_its_pools_do_not(every_step):
    """2-bit rows under a byte budget: some 19000 rows of a unit, pools for 44000 (more than a workgroup's LDS has scores for).  The
    tailors go by the rows that the layer's ratio lets a unit hold: states and rows exactly."""
    n, t = 7000, 22000
    wl = synth.C1.scaled(name="pools", n_q_heads=2, n_kv_heads=1, head_dim=64, bits=2, prefill=t, batch=1, budget_frac=(n + 0.5) / t,
                         alpha=0.999, decode_steps=3 if every_step else 9)
    cfg = make_cfg(wl, every_step=every_step, byte_budget=True)
    assert n + A.arkv_budget_counts(cfg, 0.0)[2] > 32768 > n + A.arkv_budget_counts(cfg, 0.6)[2]
    sb = _run(wl, rho=0.6, check_every=3, stats=False, every_step=every_step, byte_budget=True)
    assert sb.oracles[(0, 0)].n_tailors >= 2


def _scores(kind, n):
    """fp32 bits of n scores (0xFFFFFFFF: not ranked)."""
    r = np.random.default_rng(n)
    s = r.random(n).astype(np.float32)
    if kind == "infinite and NaN":
        s[r.random(n) < 0.3] = np.inf
        s[r.random(n) < 0.1] = np.nan
    bits = s.view(np.uint32).copy()
    if kind == "equal":
        bits[:] = np.float32(0.25).view(np.uint32)
    if kind == "few values":
        bits = (np.uint32(0x3E000000) + r.integers(0, 3, n).astype(np.uint32))
    if kind == "widest range":
        bits[1 : 3] = (0, 0xFFDFFFFF)[: max(n - 1, 0)]
    if kind == "none":
        bits[:] = 0xFFFFFFFF
    elif kind == "one":
        bits[np.arange(n) != n // 2] = 0xFFFFFFFF
    else:
        bits[r.random(n) < 0.2] = 0xFFFFFFFF
        bits[0] = 0x3DCCCCCD                         # at least one
    return bits


@pytest.mark.parametrize("in_memory", [False, True])
@pytest.mark.parametrize("n", [1, 1023, 4096, 4097, 32768])
@pytest.mark.parametrize("kind", ["spread", "none", "one", "equal", "few values", "widest range", "infinite and NaN"])
def test_selection_alone(kind, n, in_memory):
    """The thresholds of two ranks let exactly the best rows through, whatever the scores; where no row is ranked nothing
    qualifies (rows that are not ranked, and those that fill the last round of 4096, are no candidates)."""
    bits = _scores(kind, n)
    ranked = np.nonzero(bits != 0xFFFFFFFF)[0]
    keys = (bits.astype(np.uint64) << np.uint64(32)) | (np.uint64(0xFFFFFFFF) - np.arange(n, dtype=np.uint64))
    best = np.sort(keys[ranked])[::-1]
    for k0, k1 in ((0, 1), (1, n), (n // 3, n // 2), (n // 2, n // 2), (0, 0), (n, n + 5)):
        thr = A.arkv_debug_select(bits, k0, k1, in_memory)
        for k, t in zip((k0, k1), thr):
            if k == 0 or len(ranked) == 0:
                assert t == 2 ** 64 - 1
            else:
                assert np.count_nonzero(keys[ranked] >= np.uint64(t)) == min(k, len(ranked))
                assert (best[: k] >= np.uint64(t)).all()


@pytest.mark.parametrize("in_memory", [False, True])
@pytest.mark.parametrize("few", [1, 2, 63, 64, 65, 130])
def test_selection_of_few_candidates(few, in_memory):
    """The last candidates of a rank are ranked among themselves up to 64 of them: rows that share their leading digits, with
    and without equal scores, for ranks at both ends and in the middle of them."""
    n = 6000
    r = np.random.default_rng(few)
    for values in (few, 3):                              # distinct scores; three values, so that ties fall on most ranks
        bits = np.where(np.arange(n) % 2 == 0, np.uint32(0x3F800000), np.uint32(0x30000000)).astype(np.uint32)
        rows = r.choice(n, few, replace=False)
        bits[rows] = np.uint32(0x38000000) + r.permutation(np.arange(few) % values).astype(np.uint32)
        above = int(np.count_nonzero(bits > 0x38FFFFFF))
        keys = (bits.astype(np.uint64) << np.uint64(32)) | (np.uint64(0xFFFFFFFF) - np.arange(n, dtype=np.uint64))
        best = np.sort(keys)[::-1]
        for k0, k1 in ((above + 1, above + few), (above + (few + 1) // 2, above + (few + 1) // 2), (above, above + 1), (above + few, above + few + 1)):
            for k, t in zip((k0, k1), A.arkv_debug_select(bits, k0, k1, in_memory)):
                assert np.count_nonzero(keys >= np.uint64(t)) == k
                assert (best[:k] >= np.uint64(t)).all()


@pytest.mark.parametrize("hq,hkv,d,bits,n", [(4, 1, 64, 4, 4097), (8, 1, 128, 8, 5121), (2, 2, 64, 2, 6200), (2, 1, 128, 4, 4160)])
def test_every_step_policy_rows_of_several_workgroups(hq, hkv, d, bits, n):
    """A tailor at every step over more than 4096 rows: several workgroups score a unit's rows (the last one a few rows only),
    the unit's last one chooses.  More than 16 steps, so that the choosing workgroup makes the moves at the end as well."""
    t = n + 700
    wl = synth.C1.scaled(name=f"parts{n}", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, bits=bits, prefill=t, batch=1,
                         budget_frac=(n + 0.5) / t, decode_steps=21)
    assert wl.capacity == n
    sb = _run(wl, rho=0.4, check_every=7, every_step=True)
    assert all(len(u.pos) == n - 1 for u in sb.oracles[(0, 0)].units)


@pytest.mark.parametrize("T,n,window,batch", [(300, 120, 48, 1), (4096, 1000, 32, 2), (4097, 1001, 32, 1), (8191, 700, 48, 1),
                                              (8192, 700, 16, 1), (8193, 700, 32, 1), (200, 90, 16, 65)])
def test_commit_scores_are_the_formula_bit_for_bit(T, n, window, batch):
    """The scores that a commit ranks on, formed by the selecting workgroups (prompts of up to 8192 positions) or by a launch of
    their own (longer ones, more than 64 sequences): of every survivor, eq. 9's fp32 formula on its exported sums, and the n_o
    (b) best scores are those that became Original (survived)."""
    g, hkv, d = 2, 3, 64
    wl = synth.C1.scaled(name="formula", n_q_heads=g * hkv, n_kv_heads=hkv, head_dim=d, prefill=T, batch=batch, n_layers=1,
                         window=window, budget_frac=(n + 0.5) / T)
    assert wl.capacity == n
    cfg = make_cfg(wl)
    cache = A.arkv_cache_create(cfg)
    try:
        k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
        stats = torch.zeros((batch, 3), dtype=torch.float32, device="cuda")
        A.arkv_prefill_stats(cache, 0, qw, k, T, synth.softmax_scale(wl, 0), stats)
        rho = [0.3 + 0.4 * b / batch for b in range(batch)]
        A.arkv_prefill_commit(cache, 0, k, v, T, rho)
        units = batch * hkv
        e = A.arkv_cache_export(cache, 0, cfg, rows=False, codes=False)
        cnt, pos, score = A.arkv_debug_last_tailor_scores(cache, 0, units, T)
        for u in range(units):
            assert cnt[u] == T - window and (pos[u, : cnt[u]] == np.arange(T - window)).all()
            m = int(e["n_live"][u])
            p, st = e["pos"][u, :m], e["state"][u, :m]
            ranked = p < T - window
            nf = np.float32(g * window)
            mu, ex2 = e["s1"][u, :m] / nf, e["s2"][u, :m] / nf
            S = mu + np.float32(cfg.gamma) * np.maximum(ex2 - mu * mu, np.float32(0))
            assert (S[ranked].view(np.uint32) == score[u, p[ranked]].view(np.uint32)).all()
            order = np.lexsort((pos[u, : cnt[u]], -score[u, : cnt[u]].astype(np.float64)))     # ties: the older token first
            n_o, n_q, _ = A.arkv_budget_counts(cfg, rho[u // hkv])
            original = st == st[-1]                           # (the window's tokens are Original)
            assert set(order[:n_o]) == set(p[ranked & original]) and set(order[n_o : n_o + n_q]) == set(p[~original])
    finally:
        A.arkv_cache_destroy(cache)


@pytest.mark.parametrize("hq,hkv,batch,d,T", [(4, 1, 1, 128, 4096), (4, 1, 1, 128, 4097), (8, 2, 1, 64, 9000), (8, 1, 1, 64, 20000),
                                              (40, 20, 1, 64, 4096), (40, 20, 1, 64, 4097)])
def test_row_constants_of_many_chunks(hq, hkv, batch, d, T):
    """The scorer's row constants put together from 32, 33 and more chunks of 128 keys, by the column pass (up to 32 chunks or 640
    workgroups) or by a launch of their own, against the few chunks of 4096 keys.  A row constant is at most 2^6 here, so its last
    bit is 4e-6 and a probability's relative error 2.7e-6; the kurtosis has the fourth power."""
    wl = synth.C1.scaled(name="chunks", n_q_heads=hq, n_kv_heads=hkv, head_dim=d, prefill=T, batch=batch, n_layers=1, budget_frac=0.25)
    k, v, qw = (t.cuda() for t in synth.prefill_inputs(wl, 0))
    got = []
    for chunk in (128, 4096):
        cache = A.arkv_cache_create(make_cfg(wl))
        try:
            A.arkv_debug_set_launch_shape(cache, prefill_chunk=chunk)
            stats = torch.zeros((batch, 3), dtype=torch.float32, device="cuda")
            A.arkv_prefill_stats(cache, 0, qw, k, T, synth.softmax_scale(wl, 0), stats)
            torch.cuda.synchronize()
            got.append(stats.cpu().numpy())
        finally:
            A.arkv_cache_destroy(cache)
    assert np.all(np.isfinite(got[0])) and np.all(np.abs(got[0] - got[1]) <= 4 * 2.7e-6 * np.abs(got[1]))


@pytest.mark.parametrize("T", [40, 544, 545, 1056, 1057, 2080])
def test_statistics_at_the_ends_of_their_workgroups(T):
    """A sequence's statistics come from one workgroup for 512 (1024) keys in front of the window, else from several whose last
    one adds them up: both sides of every line, a few keys, several sequences, twice in a row.  From 32-bit probabilities the three
    numbers are a few 1e-7 off; 1e-5 is what their order of summation could make of it."""
    wl = synth.C1.scaled(name=f"stats{T}", prefill=T, batch=3, n_layers=1, budget_frac=2.0)
    cache = A.arkv_cache_create(make_cfg(wl))
    try:
        k, v, qw = synth.prefill_inputs(wl, 0)
        scale = synth.softmax_scale(wl, 0)
        for _ in range(2):
            stats = torch.zeros((wl.batch, 3), dtype=torch.float32, device="cuda")
            A.arkv_prefill_stats(cache, 0, qw.cuda(), k.cuda(), T, scale, stats)
            got = stats.cpu().numpy()
            for b in range(wl.batch):
                a = O.window_attention(synth.to_numpy_f32(qw[b]), synth.to_numpy_f32(k[b]), scale, wl.group)
                ref = np.array(O.layer_statistics(a, wl.window)[:3])
                assert np.all(np.abs(got[b] - ref) <= 1e-5 * np.abs(ref) + 1e-30)
    finally:
        A.arkv_cache_destroy(cache)
