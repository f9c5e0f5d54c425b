"""The selection kernels (draws by inverse CDF, rejection test, resample) at vocabularies around the edges of their work
split: a row is cut into chunks of 512 entries, at most 256 of them, so one entry, one chunk with and without a remainder,
the largest row of 256 full 512-entry chunks and the first row of longer chunks.  The rules of the oracle, evaluated on the
logits rows the GPU itself produced, must give the GPU's tokens exactly (both sides sum in float64: only a uniform within
about 1e-12 of a boundary could differ; every draw and test is checked to be 1e-10 away from its boundary)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _off_boundary(w, u):
    """The draw by u from weights w lies further than any float64 round-off from where it would give another entry."""
    c = np.cumsum(np.asarray(w, np.float64))
    return u == 0.0 or np.abs(c - u * c[-1]).min() > 1e-10 * c[-1]


def _accept_off_boundary(d, zq, zp, u_acc, u_res, T):
    """The same of a step's acceptance tests, up to the first rejection, and of its last draw."""
    from oracle import softmax64
    for i in range(len(d)):
        p, q, t = softmax64(zp[i], T), softmax64(zq[i], T), int(d[i])
        if p[t] == q[t] == 0.0 or float(u_acc[i]) * q[t] >= p[t]:
            r = np.maximum(0.0, p - q)
            return (p[t] == 0.0 or abs(float(u_acc[i]) * q[t] - p[t]) > 1e-10 * p[t]) and _off_boundary(r if r.sum() > 0.0 else p, u_res)
        if abs(float(u_acc[i]) * q[t] - p[t]) <= 1e-10 * p[t]:
            return False
    return _off_boundary(softmax64(zp[len(d)], T), u_res)


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
    assert _off_boundary(softmax64(z, T), u[0])
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
        assert all(_off_boundary(softmax64(zq[j], T), us[j]) for j in range(K))
        assert _accept_off_boundary(d, zq, zp, us[K:2 * K], float(us[2 * K]), T)
        assert [int(t) for t in d] == [inv_cdf(softmax64(zq[j], T), us[j]) for j in range(K)], i
        assert (st["last_n"], st["t_last"]) == accept_sample(d, zq, zp, us[K:2 * K], float(us[2 * K]), T), i
    ses.close()
    torch.cuda.synchronize()


@pytest.mark.parametrize("vocab,masked", [
    (513, slice(512, 513)),      # the last chunk holds one entry
    (1025, slice(1024, 1025)),
    (1300, slice(512, 1024)),    # a whole chunk in the middle
    (1300, slice(0, 600)),       # the first chunk and a part of the second
    (1300, slice(1, 1300)),      # everything but the first entry
    (131073, slice(170 * 768, 131073)),   # chunks of 768 entries: the whole of the last, ragged one
])
def test_entries_of_minus_infinity_are_never_drawn(vocab, masked):
    """Logits of -inf (masked or overflowed) have weight 0, also where they fill a chunk of the selection kernels' split;
    depth 8, the most rows an accept reads; and, on the same logits, a rejection whose residual is zero throughout (draft
    and target equal, the proposed token masked), which draws from the target's row.  -inf comes from the model itself:
    column 0 of the residual stream is the embedding's (8), and the masked rows of the head hold -3e38 there."""
    import torch
    from oracle import accept_sample, inv_cdf, softmax64
    from synth.device import DeviceWeights
    import paper_2602_05499_amd as P
    K, T = 8, 0.8
    s = synth.CONFIGS["tiny"].with_(name="select_inf", n_layers=2, d_model=64, n_heads=2, n_kv_heads=2, head_dim=32, d_ffn=64,
                                    vocab=vocab, K=K, mode="sample", init_std=0.3)
    u = synth.gen_uniforms(91, 1 + 4 * (2 * K + 1))
    for draft_mask in (np.array([0, 3], np.uint8), np.zeros(2, np.uint8)):
        dw = DeviceWeights(s, damp_skipped=0.1, skip_mask=draft_mask)
        dw.tok_emb[:, 0] = 8.0
        for l in dw.layers:
            l["wo"][0] = 0.0
            l["w_down"][0] = 0.0
        dw.lm_head[:, 0] = 0.0
        dw.lm_head[masked, 0] = -3e38
        torch.cuda.synchronize()
        ses = P.Session(s, dw, draft_mask, max_seq=96, max_k=K, temperature=T)
        ses.prefill(synth.gen_prompt(3, 7, vocab), P.SD_SAMPLE, u[:1])
        z = ses.dump_logits(P.SD_LOGITS_VERIFY, 1)[0]
        assert np.isneginf(z[masked]).all() and np.isfinite(np.delete(z, np.arange(vocab)[masked])).all()
        assert _off_boundary(softmax64(z, T), u[0])
        assert ses.read()[1]["t_last"] == inv_cdf(softmax64(z, T), u[0])
        for i in range(4):
            us = u[1 + i * (2 * K + 1):1 + (i + 1) * (2 * K + 1)]
            ses.draft(K, P.SD_SAMPLE, us[:K])
            d, zq = ses.dump_draft(K), ses.dump_logits(P.SD_LOGITS_DRAFT, K)
            assert all(_off_boundary(softmax64(zq[j], T), us[j]) for j in range(K))
            assert [int(t) for t in d] == [inv_cdf(softmax64(zq[j], T), us[j]) for j in range(K)], i
            if i % 2:                     # a masked token proposed: p = q = 0 there, so it is rejected
                d = d.copy()
                d[0] = np.arange(vocab)[masked][0]
                ses.set_draft(d)
            ses.verify()
            zp = ses.dump_logits(P.SD_LOGITS_VERIFY, K + 1)
            ses.accept(P.SD_SAMPLE, us[K:])
            ses.rollback()
            st = ses.read()[1]
            if i % 2 and not draft_mask.any():
                assert np.array_equal(zq[0], zp[0])           # the residual of row 0 is zero throughout
                assert st["last_n"] == 0
            assert _accept_off_boundary(d, zq, zp, us[K:2 * K], float(us[2 * K]), T)
            assert (st["last_n"], st["t_last"]) == accept_sample(d, zq, zp, us[K:2 * K], float(us[2 * K]), T), i
        ses.close()
    torch.cuda.synchronize()
