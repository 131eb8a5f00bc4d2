"""Decode GEMMs of layers carried as fp16 pairs, in which every k-tile of W meets the hi and then the lo tile of the activations:
at two, four and eight 16-row tiles (one, and whole layers of few rows, are in test_gpu_parity), K split and not, workgroups
that start apart in k and not, bf16 weights and an fp16 copy."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# d = 2048: gate/up not split, 16 k-tiles of rows a power of two long, so its workgroups start apart; K of all GEMMs even
# numbers of k-tiles.  d = 384: three k-tiles, fewer trips than the loop has stages to fill on its own
SHAPES = {"wide": synth.ModelShape("pair_wide", 2, 2048, 8, 2, 128, 1024, 768, 10000.0, "bf16", 0.02),
          "odd": synth.ModelShape("pair_odd", 2, 384, 6, 3, 64, 640, 768, 10000.0, "bf16", 0.04)}


@pytest.mark.parametrize("most", [20, 50, 100])
@pytest.mark.parametrize("copy", [False, True], ids=["bf16", "fp16copy"])
@pytest.mark.parametrize("name", SHAPES)
def test_pairs_carry_their_bits_through_decode(name, copy, most):
    """With both layers as pairs only the final norm's output is rounded to fp16: the generated log-probs' error falls well
    below that of the plain fp16 path (with a lo term missing or doubled it does not).  A row alone has the batch's bits."""
    shape, P, G = SHAPES[name], 9, 6
    w = synth.make_weights(shape, 1, DEV)
    cfg = R.make_cfg(shape, most, P + G)
    shadow = torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copy else None
    ro = R.Rollout(cfg, R.Weights(w, shadow=shadow), DEV)
    m = O.Model(shape, synth.weights_for_oracle(w))
    ids, lens = synth.make_prompts(shape.vocab, most, P, 3, 3)
    rows = sorted({0, 1, 15, 16, most // 2, most - 2, most - 1})

    def generate(n):
        out = torch.full((n, G), -1, dtype=torch.int32, device=DEV)
        lp = torch.full((n, G), 9.0, dtype=torch.float32, device=DEV)
        ro.rollout_generate(R.sample_cfg(4, 0.8), torch.tensor(ids[:n], device=DEV), lens[:n], G, out, None, lp)
        ro.rollout_check()
        return out.cpu().numpy(), lp.cpu().numpy()

    rms = {}
    for n in (0, 2):
        ro.rollout_set_precise_layers(n)
        out, lp = generate(most)
        e = [lp[b] - O.score(m, np.concatenate([ids[b, :lens[b]], out[b]]))[lens[b]:lens[b] + G] for b in rows]
        rms[n] = float(np.sqrt(np.mean(np.concatenate(e) ** 2)))
    one, one_lp = generate(1)
    assert np.array_equal(one[0], out[0]) and np.array_equal(one_lp[0], lp[0])
    print(name, copy, most, rms)
    assert rms[2] < 0.4 * rms[0], rms                      # 0.4 as in the test of few rows
    ro.close()
