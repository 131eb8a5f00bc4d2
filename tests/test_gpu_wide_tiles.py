"""Decode GEMMs that are more than one round of workgroups, on tiles of 256 columns: gate/up and LM heads with a short last
workgroup and a full one, one to eight 16-row tiles of activations with remainders, plain and pair layers, K of a few steps and
one whose workgroups start apart, bf16 weights and an fp16 copy -- against the oracle, and row by row against smaller batches."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import kernels_run, verify_rollout

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# the second layer (or the first) carries its activations as fp16 pairs; 16-column tiles of gate/up and LM head and which of them go wide
SHAPES = {"short": (synth.ModelShape("wide_short", 2, 384, 6, 3, 64, 27456, 65408, 10000.0, "bf16", 0.03), (True, True)),
          "apart": (synth.ModelShape("wide_apart", 2, 2048, 8, 2, 128, 28672, 4096, 10000.0, "bf16", 0.015), (True, False)),
          "two": (synth.ModelShape("wide_two", 2, 256, 4, 2, 64, 2048, 128256, 10000.0, "bf16", 0.06), (False, True))}


def _wide(n_tiles, most, pair, step):
    """The launcher's rule: rounds of 256 workgroups, weighed by what one draws per k-step and does alone."""
    rows = (1 if most <= 64 else 4) << pair
    rounds = lambda c: -(-(-(-n_tiles // c)) // 256)
    ct = min(range(step, 9, step), key=lambda c: rounds(c) * (c + rows))
    return rounds(16) * (18 + rows) <= rounds(ct) * (ct + 2 + rows)


@pytest.mark.parametrize("most", [64, 128])
@pytest.mark.parametrize("copy", [False, True], ids=["bf16", "fp16copy"])
@pytest.mark.parametrize("name", SHAPES)
def test_wide_tiles_rows_and_widths(name, copy, most):
    shape, wide = SHAPES[name]
    for pair in (0, 1):
        assert _wide(shape.d_ffn // 8, most, pair, 1) == wide[0]
    assert _wide(shape.vocab // 16, most, 0, 2) == wide[1]
    P, G = 9, 4
    w = synth.make_weights(shape, 1, DEV)
    cfg = R.make_cfg(shape, most, P + G)
    shadow = torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copy else None
    ro = R.Rollout(cfg, R.Weights(w, shadow=shadow), DEV)
    m = O.Model(shape, synth.weights_for_oracle(w))
    ids, lens = synth.make_prompts(shape.vocab, most, P, 3, 3)
    res = {}
    few = (1, 15, 16, 17, 33) if most == 64 else (1, 17, 33, 64, 65, 113)
    for n in few + (most,):
        out = torch.full((n, G), -1, dtype=torch.int32, device=DEV)
        lp = torch.full((n, G), 9.0, dtype=torch.float32, device=DEV)

        def generate():
            ro.rollout_generate(R.sample_cfg(4, 0.8), torch.tensor(ids[:n], device=DEV), lens[:n], G, out, None, lp)
            ro.rollout_check()
        if n == most:                                  # gate/up is epilogue 3, the LM head 7
            ran = kernels_run(generate)
            assert tuple(any(f"gemm_wide_kernel<{epi}," in k for k in ran) for epi in (3, 7)) == wide, ran
        else:
            generate()
        res[n] = (out.cpu().numpy(), lp.cpu().numpy())
    for n in few:                                      # a row's bits do not depend on its batch-mates
        assert np.array_equal(res[n][0], res[most][0][:n]) and np.array_equal(res[n][1], res[most][1][:n]), n
    # the lowest of several equal maxima, the logits of the last columns and the sum over all of them: the oracle's own sampling
    verify_rollout(m, [ids[b, :lens[b]] for b in range(most)], *res[most], 0.8, 4, 0, 1e-3, 2e-2, rows=[0, 16, most - 1])
