"""Turns of the weight ring around the edges of its four blocks: rows that fill part of a block, one block, two to five
blocks, in both sets of decode kernels, against the oracle; and the two sets against each other, bit for bit."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _run_greedy_against_oracle, _setup, gpu  # noqa: F401

pytestmark = pytest.mark.gpu

# storage type, d_model, d_ffn: a block is 512 float32 or 1024 bfloat16 values of a row
ROWS = [("f32", 256, 688), ("f32", 528, 1040), ("f32", 1536, 2064), ("f32", 2560, 512),
        ("bf16", 1024, 2080), ("bf16", 2080, 4128), ("bf16", 3072, 1056), ("bf16", 5120, 4096)]


def _shape(dtype, d, F):
    return synth.CONFIGS["tiny"].with_(name=f"turns-{dtype}-{d}-{F}", dtype=dtype, d_model=d, d_ffn=F, n_layers=2, skip_layers=(1,),
                                       n_kv_heads=2, vocab=4112, gain_std=0.1)


@pytest.mark.parametrize("dtype,d,F", ROWS)
def test_ragged_rows_against_the_oracle_in_both_sets(gpu, dtype, d, F):
    for span in (0, 1):
        _run_greedy_against_oracle(gpu, _shape(dtype, d, F), K=4, damp=0.05, G=9, n_prompt=11, span=span)


@pytest.mark.parametrize("dtype,d,F", ROWS)
def test_both_sets_give_the_same_bits(gpu, dtype, d, F):
    s = _shape(dtype, d, F)
    out = []
    for span in (0, 1):
        ses, _, _, _ = _setup(gpu, s, damp=0.05, max_seq=64, max_k=8, span=span)
        ses.keep_logits(True)
        ses.prefill(synth.gen_prompt(synth.SEED_PROMPT, 13, s.vocab))
        rows = []
        for K in (1, 4, 8, 0):
            ses.step(K)
            toks, _ = ses.read()
            rows += [ses.dump_logits(gpu.SD_LOGITS_VERIFY, K + 1), toks]
        out.append(rows)
        ses.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
