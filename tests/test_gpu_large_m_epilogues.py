"""Epilogues of the large-M GEMM kernel (16-byte stores through LDS) against those of the 128 x 128 tile kernel."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = {64: synth.ModelShape("epi64", 3, 512, 8, 4, 64, 1024, 3072, 10000.0, "bf16", 0.05),
          128: synth.ModelShape("epi128", 3, 512, 8, 2, 128, 1024, 3072, 500000.0, "bf16", 0.05)}


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("precise", [0, 2])
def test_prefill_gives_the_bits_of_the_small_tile_kernel(hd, precise):
    """Both kernels sum a row over k in the same order and their epilogues round alike, so prefilled caches (rotated keys,
    dim-major values, pairs in the precise layers) and what is generated from them are equal bit for bit.  Ragged prompts
    leave padding rows, partial tiles and partial pages; few enough rows that the rule itself picks the small tiles."""
    s = SHAPES[hd]
    w = synth.make_weights(s, 1, DEV)
    got = []
    for impl in (1, 2):                        # 2: the large-M kernel whenever the shape allows
        ro = R.Rollout(R.make_cfg(s, 6, 160), R.Weights(w), DEV)
        ro.rollout_set_impl(impl)
        ro.rollout_set_precise_layers(precise)
        lens = np.array([1, 2, 16, 33, 97, 150], np.int32)
        ids = torch.tensor(np.random.default_rng(3).integers(0, s.vocab, size=(6, 150)).astype(np.int32), device=DEV)
        out = torch.zeros(6, 8, dtype=torch.int32, device=DEV)
        lp = torch.zeros(6, 8, device=DEV)
        ro.rollout_generate(R.sample_cfg(4, 1.0), ids, lens, 8, out, None, lp)
        ro.rollout_check()
        got.append((out.cpu().numpy(), lp.cpu().numpy()))
        ro.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert np.isfinite(got[0][1]).all() and (got[0][1] < 0).all()
