"""Tile sizes of the small-M GEMM (64 x 64, 64 x 128, 128 x 128, from the number of tiles): the same bits from each."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("hd", [64, 128])
def test_tile_sizes_give_the_same_bits(hd):
    """d = 512: four column blocks of 128 for the two residual GEMMs, so chunks of 256 and 1216 rows put them on
    64 x 64 tiles (16 and 76 of 64 rows), 64 x 128 at 2720 (172) and 128 x 128 at 5056 (160 of 128 rows); the QKV projection
    and the LM head take 64 x 128 tiles up to 1216 rows.  Scores of the same sequences, each chunked differently."""
    s = synth.ModelShape(f"small{hd}", 2, 512, 512 // hd, 512 // hd // 2, hd, 1024, 1024, 10000.0, "bf16", 0.05)
    w = synth.make_weights(s, 1, DEV)
    r = np.random.default_rng(3)
    lens = r.integers(1, 161, size=64).astype(np.int32)
    lens[:3] = 160, 1, 64
    L = int(lens.max())
    ids = torch.tensor(r.integers(0, s.vocab, size=(len(lens), L)).astype(np.int32), device=DEV)
    rows = int(((lens + 31) // 32 * 32).sum())
    assert rows > 5056
    got = []
    for chunk in (256, 1216, 2720, 5056):
        W = R.Weights(w)
        ro = R.Rollout(R.make_cfg(s, len(lens), L, max_chunk_tokens=chunk), W, DEV)
        lp = torch.zeros(len(lens), L, device=DEV)
        ro.score_logprobs_kl(W, None, ids, lens, np.ones(len(lens), np.int32), 0.0, lp)
        ro.rollout_check()
        got.append(lp.cpu().numpy())
        ro.close()
    for g in got[1:]:
        assert np.array_equal(g, got[0])
    assert np.isfinite(got[0]).all() and (got[0] < 0).any()
