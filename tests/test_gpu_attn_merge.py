"""The merge of the attention splits in the decode kernels, where its cut changes: one split, the edges of a split, several
chunks of splits (9 rows: 28 at a time; 16-row prompt chunks: 16 at a time), more statistics than threads, head_dim below and
above the 32 columns of a unit, query heads that share a KV head."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, _setup, gpu  # noqa: F401
from test_gpu_parity_wide import _gpu_cache_to_host

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
    if n <= 1030:
        toks = np.concatenate([prompt, [first], draft]).astype(np.int32)
        ref = orc.forward(toks, 0, logits_from=n)
    else:           # the oracle's attention is quadratic in the prompt: its rows alone, over the GPU's cached positions
        ref = _oracle_rows(orc, ses, s, n, [first] + list(draft))
    assert np.abs(rows - ref).max() < TOL["f32"]
    ses.close()


def _oracle_rows(orc, ses, s, n, tokens):
    kc, vc = _gpu_cache_to_host(ses, s, n)
    ok, ov = orc.kv_arrays()
    ok[:, :n] = kc
    ov[:, :n] = vc
    return orc.forward(np.asarray(tokens, np.int32), n)


@pytest.mark.timeout(600)
def test_statistics_that_do_not_fit_are_merged_some_rows_at_a_time(gpu):
    """Beyond 127488 positions (996 splits) the statistics of 16 rows do not fit in LDS, beyond 226560 (1770) those of 9: rows go
    in batches, row 0 in the last.  A verify of 9 rows (8 + 1) against the oracle and one-row decoding, prompt chunks of 16 rows
    (15 + 1; 8 + 8) against one-row decoding, through the rows that the second layer caches."""
    n, K, chunk = 226600, 8, 128000
    s = synth.CONFIGS["tiny"].with_(name="merge-batches", n_layers=2, skip_layers=(1,), d_model=64, d_ffn=64, head_dim=32, n_heads=2,
                                    n_kv_heads=1, vocab=64, gain_std=0.1)
    ses, orc, _, _ = _setup(gpu, s, max_seq=n + 2 * K + 3, max_k=K)
    ses.keep_logits(True)
    prompt = synth.gen_prompt(synth.SEED_PROMPT, n, s.vocab)
    ses.prefill(prompt)
    print("prompt of", n, "done", ses.read(0)[1]["t_last"], flush=True)
    first = ses.read(0)[1]["t_last"]
    cached = [np.stack(_gpu_cache_to_host(ses, s, n))[:, :, p].copy() for p in (*range(chunk, chunk + 16), n - 1)]
    ses.draft(K)
    draft = ses.dump_draft(K)
    ses.verify()
    rows = ses.dump_logits(gpu.SD_LOGITS_VERIFY, K + 1)
    ses.accept(); ses.rollback()
    assert np.abs(rows - _oracle_rows(orc, ses, s, n, [first] + list(draft))).max() < TOL["f32"]
    for i, tok in enumerate([first] + list(draft)):
        ses.set_pending(n + i, int(tok))
        ses.decode()
        assert np.array_equal(ses.dump_logits(gpu.SD_LOGITS_VERIFY, 1)[0], rows[i]), i
    for p, was in zip((*range(chunk, chunk + 16), n - 1), cached):   # writes the rows of position p again
        ses.set_pending(p, int(prompt[p]))
        ses.decode()
        ses.sync()
        assert np.array_equal(np.stack(_gpu_cache_to_host(ses, s, n))[:, :, p], was), p
    ses.close()


def test_not_a_number_in_a_prompt_or_draft_comes_out_as_one(gpu):
    """Partials wait to be merged behind a bit pattern that marks them as not written, a NaN of all ones.  A NaN of that very
    pattern in a token's embedding row must not imitate it: the forward ends with NaN logits, not with the time-out."""
    import torch
    from synth.device import DeviceWeights
    s = synth.CONFIGS["tiny"]
    mask = synth.gen_skip_mask(s)
    dw = DeviceWeights(s, skip_mask=mask)
    bad = 7
    dw.tok_emb.view(torch.int32).view(s.vocab, s.d_model)[bad] = -1
    ses = gpu.Session(s, dw, mask, max_seq=64, max_k=4)
    ses.set_spin_limit(1 << 14)
    ses.keep_logits(True)
    prompt = synth.gen_prompt(5, 20, s.vocab)
    prompt[prompt == bad] = bad + 1
    prompt[5] = bad                       # a row of a 16-row chunk
    ses.prefill(prompt)
    z = ses.dump_logits(gpu.SD_LOGITS_VERIFY, 1)[0]
    ses.read()                            # raises SD_ETIMEOUT if a wait expired
    assert np.isnan(z).all()
    prompt[5] = bad + 1
    ses.prefill(prompt)
    ses.draft(4)
    draft = ses.dump_draft(4).copy()
    draft[2] = bad                        # row 3 of a verify
    ses.set_draft(draft)
    ses.verify()
    z = ses.dump_logits(gpu.SD_LOGITS_VERIFY, 5)
    ses.accept(); ses.rollback()
    ses.read()
    assert np.isnan(z[3:]).all()
    ses.close()
