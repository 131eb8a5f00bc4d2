"""Causal prefill attention: every size of a query-head group (how heads and query blocks share a workgroup) and
sequence lengths around its 32-query blocks and 64-key steps, against the plain kernels and the oracle."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
LENS = np.array([1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 128, 200], np.int32)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 3, 4, 5, 6, 7, 8])
def test_group_sizes_and_ragged_lengths(group, hd):
    hkv = 2 if group * hd % 128 == 0 else 4
    s = synth.ModelShape(f"att{group}_{hd}", 2, 256, group * hkv, hkv, hd, 512, 1024, 10000.0, "bf16", 0.06)
    w = synth.make_weights(s, 1, DEV)
    Wp = R.Weights(w)
    B, L = len(LENS), int(LENS.max())
    ro = R.Rollout(R.make_cfg(s, B, L), Wp, DEV)
    ids = torch.tensor(np.random.default_rng(group).integers(0, s.vocab, size=(B, L)).astype(np.int32), device=DEV)
    model = O.Model(s, synth.weights_for_oracle(w))
    want = np.zeros((B, L))
    for b, n in enumerate(LENS):
        want[b, :n] = O.score(model, ids[b, :n].cpu().numpy())
    got = []
    for impl in (1, 0):
        ro.rollout_set_impl(impl)
        lp = torch.zeros(B, L, device=DEV)
        ro.score_logprobs_kl(Wp, None, ids, LENS, np.ones(B, np.int32), 0.0, lp)
        ro.rollout_check()
        got.append(lp.cpu().numpy())
    ro.close()
    # both round activations to fp16 (pairs in the first layer of the tuned path): 2^-11 relative at each of the eight
    # rounding points of a layer, as between any two of these kernels
    assert np.isfinite(got[0]).all() and np.abs(got[0] - got[1]).max() < 2e-2
    assert (got[0][np.arange(L)[None, :] >= LENS[:, None]] == 0).all()
    # against the oracle: nine rounding points behind the pair layer, each 2^-11 / sqrt(3) relative at most, independent, put
    # 8.5e-4 of the logits' rms (about 1) on a logit; seven times that covers every position
    assert np.abs(got[0] - want).max() < 6e-3
