"""The separate sampling pass and the dual-distribution scores at the edges of
their vocabulary chunks (4096 entries, 16 per thread), through the C ABI.

The library dumps a step's raw logits; its log-probs, its own samples and its
scores are then compared with float64 arithmetic on those same logits, so only
these passes are under test.  The bar of 2e-5 holds float32 sums over at most
12289 entries of values of order 10: a few units of 2^-24 relative per term,
exponentials of one to two units, logs of order 10 (about 5e-6 in all).
"""
import numpy as np
import pytest

import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu

TOL = 2e-5


@pytest.mark.parametrize("vocab", [2, 5, 255, 1023, 4095, 4096, 4097, 4100, 8191, 12289])
def test_sampling_and_scores_from_the_dumped_logits(vocab):
    from oracle.sampler import gumbel_noise
    from oracle.scoring import dual_scores_rows
    from paper_2606_28166_amd.engine import TandemEngine
    P.log(f"case vocabulary edges: {vocab} entries, fp32 tiny shapes, T = 0.7, EOS bias")
    wl = W.workload("tiny").replace(gain_jitter=0.1, n_prompts=2, group=3, prompt_len=5)
    wl.senior.vocab = wl.junior.vocab = vocab
    wl.sample = W.SampleSettings(0.7, vocab - 1, 0.5, -0.5, 4)
    ws, wj, prompts, _ = W.make_all(wl)
    for w in (ws, wj):
        w["lm_head"] *= 8                       # logits of order one
    n = wl.n_seqs
    eng = TandemEngine(wl.senior, ws, wl.junior, wj, wl.switch, wl.sample, wl.philox_seed, max_seqs=n, max_ctx=16)
    eng.prefill(prompts, wl.group)
    forced = (np.arange(n) * 7 + 1) % (vocab - 1)
    sen, jun = np.zeros((n, vocab)), np.zeros((n, vocab))
    for t in range(1, 4):
        own = eng.state()["owner"]
        dbg = eng.step_forced(forced, logits=True)
        sc = eng.score()[:n].cpu().numpy()
        sen = dbg["logits_senior"][:n].cpu().numpy().astype(np.float64)
        jun = dbg["logits_junior"][:n].cpu().numpy().astype(np.float64)
        assert np.isfinite(sen).all() and np.isfinite(jun).all()
        np.testing.assert_allclose(sc, dual_scores_rows(sen, jun, forced), rtol=0, atol=TOL, err_msg=f"step {t}")
        s_sen, s_jun = sen.copy(), jun.copy()
        s_sen[:, -1] += 0.5
        s_jun[:, -1] -= 0.5
        s_sen, s_jun = s_sen / np.float32(0.7), s_jun / np.float32(0.7)
        mx = s_sen.max(1)
        lse = mx + np.log(np.exp(s_sen - mx[:, None]).sum(1))
        lp = s_sen[np.arange(n), forced] - lse
        np.testing.assert_allclose(eng.outputs()["logprob"][:, t - 1], lp, rtol=0, atol=TOL, err_msg=f"step {t}")
        sampled, margin = dbg["sampled"][:n].cpu().numpy(), dbg["margin"][:n].cpu().numpy()
        for s in range(n):
            g = (s_sen if own[s] else s_jun)[s] + gumbel_noise(wl.philox_seed, s, t, vocab)
            top = np.sort(g)[-2:]
            assert abs(margin[s] - (top[1] - top[0])) < TOL
            if top[1] - top[0] > TOL:
                assert sampled[s] == int(np.argmax(g)), (t, s)
        forced = (forced + 3) % (vocab - 1)
    eng.close()


# an entry alone in its thread's 16 (257), in its chunk (4097), and inside one (300: entry 256 of a full quad)
@pytest.mark.parametrize("vocab,bad", [(257, 256), (4097, 4096), (300, 256)])
def test_a_nan_logit_reaches_the_log_probs_and_scores(vocab, bad):
    """A NaN in one row of both LM heads: the log-softmax and the scores of
    every position are NaN, wherever the entry sits."""
    from paper_2606_28166_amd.engine import TandemEngine
    P.log(f"case NaN logit: entry {bad} of {vocab}")
    wl = W.workload("tiny").replace(gain_jitter=0.1, n_prompts=2, group=2, prompt_len=5)
    wl.senior.vocab = wl.junior.vocab = vocab
    wl.sample = W.SampleSettings(0.7, -1, 0.0, 0.0, 2)
    ws, wj, prompts, _ = W.make_all(wl)
    for w in (ws, wj):
        w["lm_head"][bad, 0] = np.nan
    n = wl.n_seqs
    eng = TandemEngine(wl.senior, ws, wl.junior, wj, wl.switch, wl.sample, wl.philox_seed, max_seqs=n, max_ctx=16)
    eng.prefill(prompts, wl.group)
    dbg = eng.step_forced(np.arange(n), logits=True)
    assert np.isnan(dbg["logits_senior"][:n, bad].cpu().numpy()).all()
    assert np.isnan(eng.score()[:n].cpu().numpy()).all()
    assert np.isnan(eng.outputs()["logprob"][:, 0]).all()
    eng.close()


def test_a_temperature_whose_reciprocal_overflows():
    """T = 1e-39 (2^-128 and below: 1 / T is infinite in float32): scores z / T
    of small logits, zero among them, are finite, and the largest one has all
    the probability.  The bar is the rounding of z / T (2^-24 of scores of 1e37,
    twice)."""
    from paper_2606_28166_amd.engine import TandemEngine
    P.log("case temperature 1e-39")
    wl = W.workload("tiny").replace(gain_jitter=0.1, n_prompts=2, group=3, prompt_len=5)
    wl.sample = W.SampleSettings(1e-39, -1, 0.0, 0.0, 2)
    ws, wj, prompts, _ = W.make_all(wl)
    for w in (ws, wj):
        w["lm_head"] = w["lm_head"] * np.float32(0.05)
        w["lm_head"][7] = 0                      # a logit of zero
    n = wl.n_seqs
    eng = TandemEngine(wl.senior, ws, wl.junior, wj, wl.switch, wl.sample, wl.philox_seed, max_seqs=n, max_ctx=16)
    eng.prefill(prompts, wl.group)
    own = eng.state()["owner"]
    forced = np.array([7, 1, 2, 3, 7, 5])
    dbg = eng.step_forced(forced, logits=True)
    z = {k: dbg[f"logits_{k}"][:n].cpu().numpy().astype(np.float64) for k in ("senior", "junior")}
    s = z["senior"] / np.float64(np.float32(1e-39))
    assert np.abs(s).max() < 1e38
    lp = s[np.arange(n), forced] - s.max(1)
    np.testing.assert_allclose(eng.outputs()["logprob"][:, 0], lp, rtol=0, atol=np.abs(s).max() * 2.0 ** -22)
    owner_z = np.where(own[:, None] != 0, z["senior"], z["junior"])
    np.testing.assert_array_equal(dbg["sampled"][:n].cpu().numpy(), owner_z.argmax(1))
    eng.close()


@pytest.mark.parametrize("first", [1, 5, 4100])
def test_no_score_above_minus_infinity(first):
    """T = 1e-39 and one logit for all entries, about -1 for some rows: their
    scores are all -inf, and NaN up to entry `first`.  The library's sample is the
    first entry that is not NaN."""
    from paper_2606_28166_amd.engine import TandemEngine
    P.log(f"case every score -inf from entry {first} on, NaN below")
    wl = W.workload("tiny").replace(gain_jitter=0.1, n_prompts=8, group=2, prompt_len=5)
    wl.senior.vocab = wl.junior.vocab = 4300
    wl.sample = W.SampleSettings(1e-39, -1, 0.0, 0.0, 2)
    ws, wj, prompts, _ = W.make_all(wl)
    for w in (ws, wj):
        w["lm_head"][:] = w["lm_head"][4200] * np.float32(50)
        w["lm_head"][:first, 0] = np.nan
    n = wl.n_seqs
    eng = TandemEngine(wl.senior, ws, wl.junior, wj, wl.switch, wl.sample, wl.philox_seed, max_seqs=n, max_ctx=16)
    eng.prefill(prompts, wl.group)
    own = eng.state()["owner"]
    dbg = eng.step_forced(np.arange(n), logits=True)
    z = {k: dbg[f"logits_{k}"][:n].cpu().numpy() for k in ("senior", "junior")}
    owner_z = np.where(own[:, None] != 0, z["senior"], z["junior"])
    assert np.isnan(owner_z[:, :first]).all()
    low = (owner_z[:, first:] < -0.5).all(axis=1)
    assert low.sum() >= 2, owner_z[:, first]
    np.testing.assert_array_equal(dbg["sampled"][:n].cpu().numpy()[low], first)
    eng.close()
