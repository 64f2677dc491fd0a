"""Sampled generation at vocabularies where the log-sum-exp's shares of a row change: shares of a few values, the last one short,
and more than one turn of a block (beyond 32768 values)."""
import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si
from oracle import sampling_oracle as sa
from oracle import stairs_oracle as so
from parity_util import LOGIT_TOL_BF16, compare_sampled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [16, 272, 2064, 33040])
def test_vocabularies(vocab):
    """Draws and keep / replace decisions are the oracle's own but for near ties (margins from the logit differences of the very
    iteration, as in the other sampling tests; at most 2 of about 60)."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=256, n_heads=4, d_ffn=512, vocab=vocab),
                           draft=dict(kind="prefix", n_layers=1), P=20, G=24)
    target, draft = si.make_pair(w)
    prompt = si.make_prompt(w)
    k, temp, seed, cap = 3, 0.1, 7, 20 + 24 + 5
    orc = sa.SampledStairs(so.OracleModel(target, np.float64), so.OracleModel(draft, np.float64), prompt, cap, temp, seed)
    with pkg.Stairs(target, draft, k_max=k, max_seq=cap) as gpu:
        gpu.prefill(prompt)
        res = compare_sampled(orc, gpu, len(prompt), 24, k, temp, seed, LOGIT_TOL_BF16)
    assert res["max_err"] < 5e-3
    assert res["draft_differs"] + res["final_differs"] + res["decision_differs"] <= 2
