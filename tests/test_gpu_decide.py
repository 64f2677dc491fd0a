"""The launch that chooses, validates and embeds in one: ties go to the lowest id wherever the equal logits lie (in one work-group's
16 columns, in different ones), at every number of rows it takes and just beyond."""
import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si

pytestmark = pytest.mark.gpu


def _pair(dtype, vocab):
    if dtype == "fp32":
        w = si.scaled_workload("cfg1_tiny_fp32", target=dict(n_layers=2, d_model=256, n_heads=4, d_ffn=512, vocab=vocab),
                               draft=dict(kind="prefix", n_layers=1))
    else:
        w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=256, n_heads=4, d_ffn=512, vocab=vocab),
                               draft=dict(kind="prefix", n_layers=1))
    target, draft = si.make_pair(w)
    return w, target, draft


@pytest.mark.parametrize("dtype,vocab", [("bf16", 2048), ("bf16", 4112), ("bf16", 32), ("fp32", 1024), ("fp32", 4096), ("fp32", 4100)])
@pytest.mark.parametrize("step", ["neighbours", "halves"])
def test_ties_go_to_the_lowest_id(dtype, vocab, step):
    w, target, draft = _pair(dtype, vocab)
    head = np.array(target.lm_head)
    if step == "neighbours":
        head[1::2] = head[0::2]
    else:
        head[vocab // 2:] = head[:vocab // 2]
    target.lm_head = head
    draft.lm_head = head
    prompt = si.make_prompt(w, 21) % vocab
    for k in (0, 1, 2, 3, 4, 5, 6, 7, 8):
        with pkg.Stairs(target, draft, k_max=8, max_seq=96) as s:
            tokens, st = s.generate(prompt, 30, k)
            s.prefill(prompt)                          # the same step by step: no launch does more than its own part there
            steps = []
            while len(steps) < 30:
                if k:
                    s.propose(k)
                tgt, n = s.verify(k)[:2]
                steps += [int(t) for t in tgt[:n + 1]]
        assert list(tokens) == steps[:30]
        if k == 0:
            want = list(tokens)
        assert list(tokens) == want
        assert all(t % 2 == 0 for t in tokens) if step == "neighbours" else all(t < vocab // 2 for t in tokens)


@pytest.mark.parametrize("k", [0, 2, 8])
def test_results_on_the_host_in_every_kind_of_loop(k):
    """Odd and even numbers of iterations, one call after the other, with an end token in between (results copied again), draft
    lengths that follow the acceptance, and behind a reservation, which moves what the launches write to."""
    w, target, draft = _pair("bf16", 2048)
    prompt = si.make_prompt(w, 21)
    with pkg.Stairs(target, draft, k_max=8, max_seq=160) as s:
        want, st = s.generate(prompt, 40, k)
        s.prefill(prompt)
        parts = []
        for g in (1, 2, 3, 14, 20):
            parts += list(s.decode(g, k)[0])
        assert parts == list(want)
        never = next(t for t in range(2048) if t not in want)
        s.set_eos(never)
        assert list(s.generate(prompt, 40, k)[0]) == list(want)
        s.set_eos(-1)
        s.prefill(prompt)
        if k:
            assert list(s.decode_adaptive(40, k)[0]) == list(want)
        s.reserve_batch(3)
        again, st2 = s.generate(prompt, 40, k)
        assert list(again) == list(want) and st2.iterations == st.iterations


@pytest.mark.parametrize("dtype,vocab", [("bf16", 2048), ("fp32", 1024)])
def test_logits_that_are_not_numbers_are_not_chosen(dtype, vocab):
    """One NaN in each 16 columns: the choice is the largest of the numbers, on the joined launch (up to 8 rows) and behind it."""
    w, target, draft = _pair(dtype, vocab)
    head = np.array(target.lm_head)
    head[5::16] = 0x7FC0 if dtype == "bf16" else np.nan
    target.lm_head = head
    draft.lm_head = head
    prompt = si.make_prompt(w, 21) % vocab
    for k in (0, 2, 4, 6, 8):
        with pkg.Stairs(target, draft, k_max=8, max_seq=96) as s:
            s.prefill(prompt)
            steps = []
            while len(steps) < 60:
                if k:
                    s.propose(k)
                tgt, n, logits = s.verify(k, logits=True)
                assert np.isnan(logits[:, 5::16]).all()
                assert [int(t) for t in tgt] == np.nanargmax(logits, axis=1).tolist(), k
                steps += [int(t) for t in tgt[:n + 1]]
            s.prefill(prompt)
            assert list(s.decode(60, k)[0]) == steps[:60]
