"""Causal attention and values that overflow: what a later token holds does not reach the key blocks before its own."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("precise", [0, 1])
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("at", [32, 45, 63, 64, 97, 190])
def test_an_infinite_value_leaves_earlier_key_blocks_alone(at, hd, precise):
    """One token's embedding has a component that no other token has, and the value projection carries it past the fp16
    range (16 x 8192): its values are infinite.  Rows of the 32-key blocks before its own attend to none of it and give
    the bits they give with an ordinary token in its place, with single values and with pairs (precise layers)."""
    s = synth.ModelShape(f"ovf{hd}", 2, 256, 512 // hd, 256 // hd, hd, 512, 1024, 10000.0, "bf16", 0.06)
    w = synth.make_weights(s, 1, DEV)
    odd = 7
    w["tok_embed"][:, 0] = 0.0
    w["tok_embed"][odd] = 0.0
    w["tok_embed"][odd, 0] = 1.0
    q_k = (s.n_q_heads + s.n_kv_heads) * hd
    for layer in w["layers"]:
        layer["wqkv"][q_k:, 0] = 8192.0
        layer["wo"][0] = 0.0                   # component 0 stays the embedding's
        layer["w_down"][0] = 0.0
    W = R.Weights(w)
    L = 200
    ids = np.random.default_rng(at).integers(8, s.vocab, size=(2, L)).astype(np.int32)
    ids[1] = ids[0]
    ids[1, at] = odd
    ro = R.Rollout(R.make_cfg(s, 2, L), W, DEV)
    ro.rollout_set_precise_layers(precise)
    lp = torch.zeros(2, L, device=DEV)
    lens = np.array([L, L], np.int32)
    ro.score_logprobs_kl(W, None, torch.tensor(ids, device=DEV), lens, np.ones(2, np.int32), 0.0, lp)
    ro.rollout_check()
    ro.close()
    lp = lp.cpu().numpy()
    assert np.isfinite(lp[0]).all()
    before = at // 32 * 32                     # a log-prob is its predecessor row's
    assert np.array_equal(lp[0, :before], lp[1, :before])
    assert not np.isfinite(lp[1, at + 1:]).any()
