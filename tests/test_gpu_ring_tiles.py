"""Small-M GEMMs on a weight set's fp16 copy (tiles of 64 x 64, 64 x 128 and 128 x 128 fed by global -> LDS loads) against the same
GEMMs on bf16 weights (staged through registers): the same products in the same order, so the same bits."""
import re

import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import kernels_run

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# K of 256 and 320 is fewer k-tiles than the kernel has stages; the second shape's gate/up has 16 column blocks of 128
SHAPES = {"hd64": synth.ModelShape("ring64", 2, 256, 4, 2, 64, 320, 512, 10000.0, "bf16", 0.05),
          "hd128": synth.ModelShape("ring128", 2, 512, 8, 2, 128, 1024, 1024, 10000.0, "bf16", 0.05)}


def _tile(rows, cols):
    """The launcher's rule; 0: past the kernel."""
    for bm, bn in ((64, 64), (64, 128), (128, 128)):
        if -(-rows // bm) * (cols // bn) <= 256:
            return bm, bn
    return 0


@pytest.mark.parametrize("chunk", [32, 96, 480, 1056, 2016])
@pytest.mark.parametrize("name", SHAPES)
def test_fp16_copy_gives_the_bits_of_bf16_weights(name, chunk):
    """Scores of policy and reference (chunks of one model, and of both models' rows with two weight sets) and a prefill into the
    cache followed by decode, with and without the copies: the kernel runs with them and only with them."""
    s = SHAPES[name]
    if chunk == 2016 and name == "hd128":
        assert {_tile(chunk, 2 * s.d_ffn), _tile(chunk, s.d_model), _tile(chunk // 2, 2 * s.d_ffn)} == {(128, 128), (64, 64), (64, 128)}
    wp, wr = synth.make_weights(s, 1, DEV), synth.make_weights(s, 2, DEV)
    r = np.random.default_rng(chunk)
    B, L = max(1, chunk // 32), 32 if chunk < 1000 else 96
    lens = np.maximum(1, r.integers(1, L + 1, size=B)).astype(np.int32)
    lens[0] = L
    ids = torch.tensor(r.integers(0, s.vocab, size=(B, L)).astype(np.int32), device=DEV)
    got = []
    for copies in (True, False):
        cfg = R.make_cfg(s, B, L + 4, max_chunk_tokens=max(chunk, L + 4))
        shadow = [torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copies else None for _ in range(2)]
        Wp, Wr = R.Weights(wp, shadow=shadow[0]), R.Weights(wr, shadow=shadow[1])
        ro = R.Rollout(cfg, Wp, DEV)
        outs = [torch.zeros(B, L, device=DEV) for _ in range(4)]
        one = torch.zeros(B, L, device=DEV)
        out = torch.zeros(B, 4, dtype=torch.int32, device=DEV)
        lp = torch.zeros(B, 4, device=DEV)

        def passes():
            ro.score_logprobs_kl(Wp, Wr, ids, lens, np.ones(B, np.int32), 0.003, *outs)
            ro.score_logprobs_kl(Wp, None, ids, lens, np.ones(B, np.int32), 0.003, one)
            ro.rollout_generate(R.sample_cfg(4, 0.7), ids, lens, 4, out, None, lp)
            ro.rollout_check()
        names = kernels_run(passes)
        ring = {(int(m[1]) * 64, int(m[2]) * 64) for n in names if (m := re.search(r"gemm_ring_kernel<\d, (\d), 4, (\d)>", n))}
        assert ring if copies else not ring, (copies, names)
        if copies and chunk == 2016 and name == "hd128":
            assert ring == {(64, 64), (64, 128), (128, 128)}
        got.append([t.cpu().numpy() for t in outs + [one, out, lp]])
        ro.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert np.isfinite(got[0][0]).all() and (got[0][0] < 0).any() and np.array_equal(got[0][0], got[0][4])
