"""A draft that is the target's first layers reads and writes the target's caches (one copy of the weights on the device is
what tells): the same tokens, proposals and acceptance counts as with a draft of equal weights in arrays of its own, whose
prompts are ingested and whose proposals start with two rows."""
import copy

import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si

pytestmark = pytest.mark.gpu


def _pair(dtype, draft_layers=1):
    if dtype == "fp32":
        w = si.scaled_workload("cfg1_tiny_fp32", draft=dict(kind="prefix", n_layers=draft_layers))
    else:
        w = si.scaled_workload("cfg2_125m", target=dict(n_layers=3, d_model=256, n_heads=4, d_ffn=768, vocab=2048),
                               draft=dict(kind="prefix", n_layers=draft_layers))
    target, draft = si.make_pair(w)
    return w, target, draft, copy.deepcopy(draft)


def _both(target, drafts, k_max, max_seq, use):
    out = []
    for d in drafts:
        with pkg.Stairs(target, d, k_max=k_max, max_seq=max_seq) as s:
            out.append(use(s))
    return out


def _same_stats(a, b):
    for key in ("iterations", "tokens", "accepted", "accept_hist"):
        assert a.as_dict()[key] == b.as_dict()[key], key


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("P,k,layers", [(1, 3, 1), (2, 1, 2), (40, 8, 1), (130, 4, 3)])
def test_one_sequence(dtype, P, k, layers):
    w, target, draft, own = _pair(dtype, layers)
    prompt = si.make_prompt(w, P)
    def use(s):
        res = [s.generate(prompt, 33, k)]
        s.prefill(prompt)
        res.append(s.decode(9, 0))                     # the target alone, then with its draft again
        res.append(s.decode(20, k))
        s.prefill(prompt)
        steps = []
        for i in range(4):                             # step by step; a proposal that is dropped for the caller's own tokens
            steps.append(np.array(s.propose(k)))
            v = s.verify(k) if i % 2 == 0 else s.verify_tokens(np.arange(k, dtype=np.int32))
            steps.append(np.array(v[0]))
            steps.append(np.array([v[1]]))
        return res, steps
    (ra, sa), (rb, sb) = _both(target, (draft, own), k, P + 80, use)
    for (ta, xa), (tb, xb) in zip(ra, rb):
        assert list(ta) == list(tb)
        _same_stats(xa, xb)
    for a, b in zip(sa, sb):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kind", ["sampled", "adaptive"])
def test_sampled_and_adaptive(kind):
    w, target, draft, own = _pair("bf16")
    prompt = si.make_prompt(w, 37)
    def use(s):
        if kind == "sampled":
            return s.generate_sampled(prompt, 40, 4, 0.7, 11)
        s.prefill(prompt)
        return s.decode_adaptive(40, 2)
    (ta, xa), (tb, xb) = _both(target, (draft, own), 8, 37 + 64, use)
    assert list(ta) == list(tb)
    _same_stats(xa, xb)


@pytest.mark.parametrize("B,k", [(3, 4), (16, 3), (40, 2)])
def test_batches(B, k):
    """3 x 5 and 16 x 4 rows on the decode kernels: all the same.  40 x 3 rows on the block kernels, whose additions go another
    way: the target's tokens, which no draft changes; what is accepted may differ in ties of the draft alone."""
    w, target, draft, own = _pair("bf16")
    prompts = [si.make_prompt(w, 3 + (b * 7) % 50) for b in range(B)]
    def use(s):
        s.reserve_batch(B)
        return s.generate_batch(prompts, 20, k)
    (ta, xa), (tb, xb) = _both(target, (draft, own), k, 128, use)
    for a, b in zip(ta, tb):
        assert list(a) == list(b)
    if B * (k + 1) <= 64:
        _same_stats(xa, xb)


def _alike(draft, what):
    """a draft that has the target's arrays but for one thing"""
    d = copy.copy(draft)
    d.layers = [dict(l) for l in draft.layers]
    rng = np.random.default_rng(5)
    if what == "heads":
        d.n_heads = draft.n_heads // 2
    elif what in ("rms_eps", "rope_theta"):
        setattr(d, what, getattr(draft, what) * 30)
    elif what == "layers swapped":
        d.layers[0], d.layers[1] = d.layers[1], d.layers[0]
    elif what.endswith("norm"):
        d.layers[-1][what] = (draft.layers[-1][what] * rng.uniform(0.5, 1.5, draft.d_model)).astype(np.float32)
    else:
        d.layers[-1][what] = np.ascontiguousarray(draft.layers[-1][what][::-1])
    return d


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("what", ["wk", "wv", "w_up", "w_down", "attn_norm", "ffn_norm", "rms_eps", "rope_theta", "heads", "layers swapped"])
def test_drafts_that_differ_in_one_thing(dtype, what):
    """Nothing of the target's that is not the draft's too: the proposals and tokens of the same draft in arrays of its own."""
    w, target, draft, _ = _pair(dtype, 2)
    if what == "heads" and target.head_dim != 64:
        pytest.skip("head_dim 128 is the largest there is")
    near = _alike(draft, what)
    prompt = si.make_prompt(w, 70)
    def use(s):
        tokens, stats = s.generate(prompt, 33, 3)
        s.prefill(prompt)
        steps = []
        for i in range(4):
            drawn, logits = s.propose_sampled(3, 0.7, 11 + i)
            steps += [drawn, logits, s.verify_sampled(3, 0.7, 11 + i)[0]]
        return list(tokens), stats, steps
    (ta, xa, sa), (tb, xb, sb), (tc, xc, sc) = _both(target, (near, copy.deepcopy(near), draft), 3, 70 + 80, use)
    assert ta == tb
    _same_stats(xa, xb)
    for a, b in zip(sa, sb):
        assert np.array_equal(a, b)
    assert not np.array_equal(sa[1], sc[1])            # (the difference shows)
