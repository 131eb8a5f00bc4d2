"""The exact KL's dual-head kernel and its compacted rows where they can go wrong: prompts of no token, of the whole
sequence and of all but one, one-token sequences, more rows than a tile and fewer, a vocabulary that ends inside a
256-column tile, bf16 weights and fp16 copies -- against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
BF16 = synth.ModelShape("klrows", 2, 256, 4, 2, 64, 256, 1152, 10000.0, "bf16", 0.08)
FP32 = synth.ModelShape("klrows32f", 2, 128, 2, 1, 64, 192, 333, 10000.0, "fp32", 0.08)


@pytest.mark.parametrize("shape,copies,tol", [(BF16, 0, 2e-2), (BF16, 1, 2e-2), (BF16, 2, 2e-2), (FP32, 0, 1e-4)],
                         ids=["bf16", "one-copy", "two-copies", "fp32"])
def test_exact_kl_rows(shape, copies, tol):
    seq = np.array([90, 1, 140, 33, 64, 7, 2], np.int32)
    prompt = np.array([0, 1, 5, 33, 63, 0, 1], np.int32)
    B, Lmax = len(seq), int(seq.max())
    w = [synth.make_weights(shape, i, DEV) for i in (1, 2)]
    # three chunks, with 89, 135 and 8 rows for the heads (tiles have 128)
    cfg = R.make_cfg(shape, B, Lmax, max_chunk_tokens=200)
    buf = lambda: torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV)   # noqa: E731
    Wp, Wr = (R.Weights(w[i], shadow=buf() if copies > i else None) for i in (0, 1))
    ro = R.Rollout(cfg, Wp, DEV)
    ids = np.random.default_rng(3).integers(0, shape.vocab, size=(B, Lmax)).astype(np.int32)
    out = torch.full((B, Lmax), 9.0, dtype=torch.float32, device=DEV)
    ro.score_kl_exact(Wp, Wr, torch.tensor(ids, device=DEV), seq, prompt, out)
    ro.rollout_check()
    mp, mr = (O.Model(shape, synth.weights_for_oracle(x)) for x in w)
    want = np.zeros((B, Lmax))
    for b in range(B):
        p = max(int(prompt[b]), 1)
        if seq[b] > p:
            want[b, p:seq[b]] = O.kl_full(mp, mr, ids[b, :seq[b]])[p:]
    got = out.cpu().numpy()
    assert np.abs(got - want).max() < tol and want.max() > 10 * tol
    assert np.all(got[want == 0.0] == 0.0)
    # sequences of prompt only: nothing to score, ids still looked at
    ro.score_kl_exact(Wp, Wr, torch.tensor(ids, device=DEV), seq, seq, out)
    ro.rollout_check()
    assert np.all(out.cpu().numpy() == 0.0)
    ids[2, 5] = shape.vocab
    ro.score_kl_exact(Wp, Wr, torch.tensor(ids, device=DEV), seq, seq, out)
    with pytest.raises(R.RolloutError):
        ro.rollout_check()
    ro.close()


def test_exact_kl_sums_keep_their_small_terms():
    """Every 64 columns: one logit of 0, the others -16.75 (policy) or -40 (reference), all exact (unit hidden state, weights on
    a grid).  The 63 small terms of e^-16.75 = 0.89 x 2^-24 vanish one by one in a sum that starts from the large one, 15 of
    them in a lane that adds its 16 columns in turn: 8e-7 of the KL of 7.4e-5.  Added pairwise, the large term is rounded
    at six levels, 2^-24 each; the two logarithms round once each (of about 0.7), and the reduction over two groups adds two
    roundings: 6e-7 in all."""
    s = synth.ModelShape("klsum", 1, 256, 4, 2, 64, 256, 128, 10000.0, "bf16", 0.02, rms_eps=0.0)
    W = []
    for k, small in enumerate((-16.75, -40.0)):
        w = synth.make_weights(s, k + 1, DEV)
        w["tok_embed"].fill_(1.0)
        w["final_norm"].fill_(1.0)
        for l in ("wo", "w_down"):
            w["layers"][0][l].zero_()
        w["lm_head"].fill_(small / 256)
        w["lm_head"][::64] = 0.0
        W.append(R.Weights(w))
    ro = R.Rollout(R.make_cfg(s, 1, 8), W[0], DEV)
    kl = torch.zeros(1, 8, device=DEV)
    ro.score_kl_exact(*W, torch.zeros(1, 8, dtype=torch.int32, device=DEV), np.array([8], np.int32), np.array([1], np.int32), kl)
    ro.rollout_check()
    ro.close()
    a, b = 63 * np.exp(-16.75), 63 * np.exp(-40.0)
    want = (a * (40.0 - 16.75)) / (1 + a) - np.log1p(a) + np.log1p(b)
    assert np.abs(kl[0, 1:].cpu().numpy() - want).max() < 6e-7
