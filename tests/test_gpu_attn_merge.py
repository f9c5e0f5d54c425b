"""The merge of the attention splits in the decode kernels, where its cut changes: one split, the edges of a split, several
chunks of splits (9 rows: 28 at a time; 16-row prompt chunks: 16 at a time), more statistics than threads, head_dim below and
above the 32 columns of a unit, query heads that share a KV head."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, _setup, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(600)
@pytest.mark.parametrize("hd,H,Hkv", [(16, 8, 2), (32, 8, 8), (64, 4, 4), (128, 4, 1)])
@pytest.mark.parametrize("n", [5, 119, 127, 128, 1030, 3595, 7400])
def test_rows_of_a_verify_against_the_oracle_and_plain_decode(gpu, hd, H, Hkv, n):
    s = synth.CONFIGS["tiny"].with_(name=f"merge-{hd}-{H}-{Hkv}", n_layers=2, skip_layers=(1,), head_dim=hd, n_heads=H, n_kv_heads=Hkv,
                                    vocab=512, gain_std=0.1)
    K = 8
    ses, orc, _, mask = _setup(gpu, s, max_seq=n + 2 * K + 3, max_k=K)
    ses.keep_logits(True)
    prompt = synth.gen_prompt(synth.SEED_PROMPT, n, s.vocab)
    ses.prefill(prompt)
    first = ses.read(0)[1]["t_last"]
    ses.draft(K)
    draft = ses.dump_draft(K)
    ses.verify()
    rows = ses.dump_logits(gpu.SD_LOGITS_VERIFY, K + 1)
    ses.accept(); ses.rollback()
    # one row at a time over the same tokens: the same bits
    for i, tok in enumerate([first] + list(draft)):
        ses.set_pending(n + i, int(tok))
        ses.decode()
        assert np.array_equal(ses.dump_logits(gpu.SD_LOGITS_VERIFY, 1)[0], rows[i]), i
    if n <= 1030:   # the oracle's attention is quadratic in the prompt
        toks = np.concatenate([prompt, [first], draft]).astype(np.int32)
        ref = orc.forward(toks, 0, logits_from=n)
        assert np.abs(rows - ref).max() < TOL["f32"]
    ses.close()
