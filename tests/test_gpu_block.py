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
    """The smallest block, edges of the 64-, 128- and 256-row tiles, the largest block whose k range is summed in pieces and
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
