"""The log-prob of a drawn token that is its row's most probable one: what the LM head's fp32 sums over the model width cost it."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import kernels_run

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("V,wide", [(65408, True), (32768, False)])
def test_likely_tokens_keep_their_log_prob(V, wide):
    """Layers that add nothing, embeddings of +-1 and unit gains make the final norm's output +-1 exactly, so the logits of the 64-bit
    reference are those of the same numbers.  Token v is followed by v + 1 with a logit of ln V + 3.5 and most of the probability: the drawn token
    is the largest logit, its log-prob -log(1 + s) with s about 0.05 over the others.  Errors of single logits (a few 1e-6 of 15
    at d = 8192) reach it through s only, 3e-7; the exponentials of s and two roundings near 1 add as much.  As a difference of that
    logit summed twice, in different order, it was off by 2e-6."""
    d, B, G = 8192, 24, 3
    s = synth.ModelShape("likely", 1, d, 2, 1, 128, 128, V, 10000.0, "bf16", 0.02)
    w = synth.make_weights(s, 1, DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    emb, head, c = w["tok_embed"], w["lm_head"], (np.log(V) + 3.5) / d
    for r0 in range(0, V, 8192):
        emb[r0:r0 + 8192] = torch.randint(0, 2, emb[r0:r0 + 8192].shape, generator=g, device=DEV).to(emb.dtype) * 2 - 1
    for r0 in range(0, V, 8192):
        idx = torch.arange(r0 - 1, min(r0 + 8192, V) - 1, device=DEV) % V
        head[r0:r0 + 8192] = (c * (emb[idx].float() + 5.0 * torch.randn(len(idx), d, generator=g, device=DEV))).to(head.dtype)
    w["final_norm"].fill_(1)
    for l in w["layers"]:
        l["wo"].zero_()
        l["w_down"].zero_()
    ro = R.Rollout(R.make_cfg(s, B, 8), R.Weights(w), DEV)
    ids = torch.randint(0, V - 8, (B, 1), generator=g, dtype=torch.int32, device=DEV)
    out, lp = torch.zeros(B, G, dtype=torch.int32, device=DEV), torch.zeros(B, G, device=DEV)

    def generate():
        ro.rollout_generate(R.sample_cfg(4, 0.5), ids, np.ones(B, np.int32), G, out, None, lp)
        ro.rollout_check()
    assert any("gemm_wide_kernel<7," in k for k in kernels_run(generate)) == wide
    tok = torch.cat([ids, out], 1).long()
    likely, worst = 0, 0.0
    for n in range(G):
        h = emb[tok[:, n]].double()
        z = torch.cat([h @ head[r0:r0 + 8192].double().T for r0 in range(0, V, 8192)], 1)
        want = torch.log_softmax(z, 1).gather(1, tok[:, n + 1:n + 2])[:, 0]
        top = z.argmax(1) == tok[:, n + 1]
        likely += int(top.sum())
        worst = max(worst, float((lp[:, n].double() - want)[top].abs().max()))
    print(V, likely, worst)
    assert likely > 0.8 * B * G and worst < 1e-6, (likely, worst)
    ro.close()
