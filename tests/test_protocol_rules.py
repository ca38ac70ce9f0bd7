"""The comparison rules of the GPU parity tests, checked on the CPU against the oracle alone: the free-running
protocol's score band (a token may end in a different state on the two sides only if its score is within 2e-3 of
the score at one of eq. 10's two cuts)."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from oracle import arkv_oracle as O
from helpers import TOL, rel_err, score_band_check


def _case(seed, n=400, n_o=90, b=250):
    r = np.random.default_rng(seed)
    S = r.random(n) ** 4 + 1e-3
    pos = r.permutation(n)
    state = np.where(r.random(n) < 0.2, O.STATE_Q, O.STATE_O).astype(np.int8)
    return S, pos, state, n_o, b


def test_identical_choices_pass():
    S, pos, state, n_o, b = _case(0)
    new = O.tailor_assign(S, pos, state, n_o, b)
    assert score_band_check(S, pos, new, new.copy(), n_o, b) is True


@pytest.mark.parametrize("seed", range(5))
def test_rounding_sized_noise_stays_inside_the_band(seed):
    """Scores perturbed by 1e-6 relative (what fp32 accumulation does): whatever the perturbed ranking changes
    lies next to a cut."""
    S, pos, state, n_o, b = _case(seed)
    # plant near-ties on both cuts so that the perturbation does flip some tokens
    order = np.argsort(-S)
    for cut in (n_o, b):
        S[order[cut - 2:cut + 2]] = S[order[cut]] * (1 + np.array([2e-7, 1e-7, 0.0, -1e-7]))
    ref = O.tailor_assign(S, pos, state, n_o, b)
    r = np.random.default_rng(100 + seed)
    flipped = 0
    for _ in range(20):
        got = O.tailor_assign(S * (1 + 1e-6 * r.standard_normal(len(S))), pos, state, n_o, b)
        flipped += not score_band_check(S, pos, ref, got, n_o, b)
    assert flipped > 0


def test_a_token_far_from_both_cuts_fails():
    S, pos, state, n_o, b = _case(1)
    ref = O.tailor_assign(S, pos, state, n_o, b)
    order = np.argsort(-S)
    got = ref.copy()
    j = order[5]                                   # a top token, far above both cuts
    assert abs(S[j] - S[order[n_o]]) / S[order[n_o]] > 10 * TOL
    got[j] = O.STATE_E
    with pytest.raises(AssertionError):
        score_band_check(S, pos, ref, got, n_o, b)
    got = ref.copy()
    j = order[-1]                                  # the lowest-ranked token, kept by mistake
    got[j] = O.STATE_Q
    with pytest.raises(AssertionError):
        score_band_check(S, pos, ref, got, n_o, b)


def test_gross_score_errors_fail():
    """Scores off by 5 % re-rank tokens well outside the band."""
    S, pos, state, n_o, b = _case(2, n=4000, n_o=900, b=2500)
    ref = O.tailor_assign(S, pos, state, n_o, b)
    r = np.random.default_rng(7)
    got = O.tailor_assign(S * (1 + 0.05 * r.standard_normal(len(S))), pos, state, n_o, b)
    with pytest.raises(AssertionError):
        score_band_check(S, pos, ref, got, n_o, b)


def test_a_value_that_is_not_finite_is_an_infinite_error():
    """The folds over rows take max(worst, error), which drops a NaN: an error is infinite instead."""
    ref = np.array([1.0, -2.0, 0.5])
    assert rel_err(ref, ref) == 0.0 and rel_err(np.zeros(2), np.zeros(2)) == 0.0
    for bad in (np.nan, np.inf, -np.inf):
        x = ref.copy()
        x[1] = bad
        assert max(0.0, rel_err(x, ref)) == np.inf and max(0.0, rel_err(ref, x)) == np.inf


def test_one_nan_among_the_attention_rows_fails():
    """The check of the prompt attention's rows accepts the oracle's own output and not the same with one NaN."""
    from test_gpu_attention import _check_rows
    g = torch.Generator().manual_seed(3)
    q, k, v = (torch.randn((1, h, 40, 64), generator=g).to(torch.bfloat16) for h in (2, 1, 1))
    at = np.arange(40)
    ref = O.causal_attention_rows(q[0].float().numpy(), at, k[0].float().numpy(), v[0].float().numpy(), 0.125, 2)
    out = SimpleNamespace(f32=torch.from_numpy(np.asarray(ref, dtype=np.float32))[None].clone())
    assert _check_rows(out, q, k, v, 0.125, 2, at, 0) <= 1e-6
    out.f32[0, 1, 17, 3] = float("nan")
    assert not _check_rows(out, q, k, v, 0.125, 2, at, 0) <= TOL
