"""Batches whose next iteration is launched while the one before it runs: tokens and counts are those of one iteration at a time."""
import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,k", [(1, 3), (2, 0), (5, 4), (16, 3), (40, 2)])
def test_ahead_and_one_by_one(B, k, monkeypatch):
    """Prompts that reach their G tokens in different iterations, answers of 1 and 2 tokens (one iteration, nothing ahead) to 33;
    an end token that never comes sends a context with graphs through the loop without anything ahead."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=3, d_model=256, n_heads=4, d_ffn=768, vocab=2048),
                           draft=dict(kind="prefix", n_layers=1))
    target, draft = si.make_pair(w)
    prompts = [si.make_prompt(w, 2 + (b * 11) % 40) for b in range(B)]
    got = {}
    for mode in ("ahead", "no graphs", "end token"):
        if mode == "no graphs":
            monkeypatch.setenv("STAIRS_NO_GRAPH", "1")
        else:
            monkeypatch.delenv("STAIRS_NO_GRAPH", raising=False)
        with pkg.Stairs(target, draft, k_max=4, max_seq=96) as s:
            s.reserve_batch(max(B, 2))
            res = []
            for G in (1, 2, 33, 7):
                if mode == "end token":
                    s.set_eos(never[G])
                toks, st = s.generate_batch(prompts, G, k)
                res.append((toks, st.as_dict()))
        if mode == "ahead":
            never = {G: next(t for t in range(2048) if not (toks == t).any()) for G, (toks, _) in zip((1, 2, 33, 7), res)}
        got[mode] = res
    for mode in ("no graphs", "end token"):
        for (ta, sa), (tb, sb) in zip(got["ahead"], got[mode]):
            assert np.array_equal(ta, tb), mode
            for key in ("iterations", "tokens", "accepted", "accept_hist"):
                assert sa[key] == sb[key], (mode, key)


@pytest.mark.parametrize("P", [487, 491, 494, 497, 498, 499, 500, 501, 502, 503])
def test_lengths_that_outgrow_the_attention_launch_while_two_iterations_run(P, monkeypatch):
    """512 keys are four units of 128, a launch for more has five: an iteration that is launched while the one before it runs must
    cover the keys that one can still add.  Prompts that cross the line at different iterations; without graphs every launch is
    sized for the length it has."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=3, d_model=256, n_heads=4, d_ffn=768, vocab=2048),
                           draft=dict(kind="prefix", n_layers=1))
    target, draft = si.make_pair(w)
    prompts = [si.make_prompt(w, n) for n in (P, P - 7, 30)]
    got = []
    for mode in ("0", "1"):
        monkeypatch.setenv("STAIRS_NO_GRAPH", mode)
        with pkg.Stairs(target, draft, k_max=3, max_seq=640) as s:
            s.reserve_batch(3)
            toks, st = s.generate_batch(prompts, 40, 3)
            one, st1 = s.generate(prompts[0], 40, 3)
            got.append((toks, st.as_dict()["accept_hist"], one, st1.as_dict()["accept_hist"]))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
