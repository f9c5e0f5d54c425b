"""The selection kernels (draws by inverse CDF, rejection test, resample) at vocabularies around the edges of their work
split: a row is cut into chunks of 512 entries, at most 256 of them, so one entry, one chunk with and without a remainder,
the largest row of 256 full 512-entry chunks and the first row of longer chunks.  The rules of the oracle, evaluated on the
logits rows the GPU itself produced, must give the GPU's tokens exactly (both sides sum in float64: only a uniform within
about 1e-12 of a boundary could differ; the seeds below are checked not to come near one)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [1, 2, 511, 512, 513, 1025, 32003, 131072, 131073, 200001])
def test_draws_and_accepts_follow_the_oracles_rules(vocab):
    import torch
    from oracle import accept_sample, inv_cdf, softmax64
    from synth.device import DeviceWeights
    import paper_2602_05499_amd as P
    K, n_steps, T = 3, 4, 0.8
    s = synth.CONFIGS["tiny"].with_(name="select", n_layers=2, d_model=64, n_heads=2, n_kv_heads=2, head_dim=32, d_ffn=64,
                                    vocab=vocab, K=K, mode="sample", init_std=0.3)
    mask = np.array([0, 3], np.uint8)
    dw = DeviceWeights(s, damp_skipped=0.1, skip_mask=mask)
    ses = P.Session(s, dw, mask, max_seq=64, max_k=K, temperature=T)
    u = synth.gen_uniforms(77, 1 + n_steps * (2 * K + 1))
    u[1] = 0.0                       # the smallest uniform: the first entry with any weight
    ses.prefill(synth.gen_prompt(3, 7, vocab), P.SD_SAMPLE, u[:1])
    z = ses.dump_logits(P.SD_LOGITS_VERIFY, 1)[0]
    assert ses.read()[1]["t_last"] == inv_cdf(softmax64(z, T), u[0])
    for i in range(n_steps):
        us = u[1 + i * (2 * K + 1):1 + (i + 1) * (2 * K + 1)]
        ses.draft(K, P.SD_SAMPLE, us[:K])
        d, zq = ses.dump_draft(K), ses.dump_logits(P.SD_LOGITS_DRAFT, K)
        ses.verify()
        zp = ses.dump_logits(P.SD_LOGITS_VERIFY, K + 1)
        ses.accept(P.SD_SAMPLE, us[K:])
        ses.rollback()
        st = ses.read()[1]
        assert [int(t) for t in d] == [inv_cdf(softmax64(zq[j], T), us[j]) for j in range(K)], i
        assert (st["last_n"], st["t_last"]) == accept_sample(d, zq, zp, us[K:2 * K], float(us[2 * K]), T), i
    ses.close()
    torch.cuda.synchronize()
