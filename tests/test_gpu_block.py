"""GPU: row blocks on the block kernels at the row counts and widths where their launches change."""
import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si

pytestmark = pytest.mark.gpu


# widths with a ragged last k chunk (1280, 2816), an odd number of unembedding tiles (528 / 16 = 33), features that end
# inside a 256-, 192- and 128-feature work-group
@pytest.mark.parametrize("d,heads,f", [(256, 2, 256), (1280, 10, 2816), (2048, 32, 1024)])
@pytest.mark.parametrize("rows", [17, 33, 64, 65, 127, 129, 256, 1024, 1025, 2048, 2049])
def test_block_rows_against_decode_kernels(d, heads, f, rows, monkeypatch):
    """A prompt of one forward and the smallest block (33 rows), edges of the 64-, 128- and 256-row tiles, the largest block whose k range is summed in pieces and
    the smallest that is not, a full block and one row more: the stair logits behind a prompt ingested in blocks against
    those behind the same prompt ingested by the decode kernels (same inputs, another order of additions: 1e-5 of the
    logits' size measured; keys and values are rounded to half in both, so single roundings can fall differently)."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=d, n_heads=heads, d_ffn=f, vocab=528),
                           draft=dict(kind="prefix", n_layers=1), P=rows + 1, G=1)
    target, draft = si.make_pair(w)
    prompt = si.make_prompt(w)
    got = {}
    for mode in ("block", "rows"):
        if mode == "rows":
            monkeypatch.setenv("STAIRS_NO_BLOCK_PREFILL", "1")
        with pkg.Stairs(target, None, k_max=0, max_seq=rows + 16) as s:
            s.prefill(prompt)
            got[mode] = s.verify(0, logits=True)[2].astype(np.float64)
    rms = np.sqrt(np.mean(got["rows"] ** 2))
    assert np.max(np.abs(got["block"] - got["rows"])) < 2e-3 * rms


@pytest.mark.parametrize("lens", [[18, 33, 34, 49, 300, 18], [17, 200, 5, 1025, 1026, 65, 1300], [700, 700, 700, 129]])
def test_prompts_of_a_batch_share_blocks(lens):
    """Prompts that share a block (17 .. 1024 rows: the smallest, ends on and beside multiples of 16 rows, more than one block's
    worth), too short, and too long to share one: every sequence's tokens are the bits of the sequence generated alone."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=768, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=2, G=1)
    target, draft = si.make_pair(w)
    rng = np.random.default_rng(len(lens))
    prompts = [rng.integers(0, 1040, P).astype(np.int32) for P in lens]
    with pkg.Stairs(target, draft, k_max=2, max_seq=max(lens) + 32) as s:
        alone = [s.generate(p, 12, 2)[0].copy() for p in prompts]
        s.reserve_batch(len(lens))
        toks, _ = s.generate_batch(prompts, 12, 2)
    for b, want in enumerate(alone):
        assert np.array_equal(toks[b], want), lens[b]


@pytest.mark.parametrize("rows", [16, 17, 24, 31, 32])
def test_prompts_of_one_forward_take_the_decode_kernels(rows, monkeypatch):
    """A prompt that one forward of the decode kernels holds goes through those (they are faster there): the stair logits
    behind it are the bits of the context that has no block kernels for prompts."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=768, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=rows + 1, G=1)
    target, _ = si.make_pair(w)
    prompt = si.make_prompt(w)
    got = []
    for off in (None, "1"):
        if off:
            monkeypatch.setenv("STAIRS_NO_BLOCK_PREFILL", off)
        with pkg.Stairs(target, None, k_max=0, max_seq=rows + 16) as s:
            s.prefill(prompt)
            got.append(s.verify(0, logits=True)[2].copy())
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("B,k", [(8, 2), (22, 2)])
def test_short_prompts_of_a_batch(B, k):
    """Prompts of 17 rows and more share blocks, in forwards of 24 rows (decode kernels) and of 66 (block kernels).  A
    sequence's tokens depend neither on its neighbours nor on their order; they are those of the sequence alone on the
    reserved context, where it takes the same kernels."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=768, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=2, G=1)
    target, draft = si.make_pair(w)
    rng = np.random.default_rng(22)
    prompts = [rng.integers(0, 1040, P).astype(np.int32) for P in ([17, 18, 19, 25, 32, 33, 34, 60] * 3)[:B]]
    with pkg.Stairs(target, draft, k_max=k, max_seq=96) as s:
        s.reserve_batch(B)
        alone = np.stack([s.generate(p, 12, k)[0].copy() for p in prompts])
        first, _ = s.generate_batch(prompts, 12, k)
        turned, _ = s.generate_batch(prompts[::-1], 12, k)
    assert np.array_equal(first, turned[::-1])
    assert np.array_equal(first, alone)
