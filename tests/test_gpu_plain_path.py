"""The plain (fp32) path's kernels at the sizes where they can go wrong, against the oracle: the GEMM's three tile sizes
with remainders in rows and columns, and the captured decode step against the eager one."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import check_scores, verify_rollout

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# vocabularies that are no multiple of any tile width; 517 rows of 6001 columns reach the 64 x 64 tiles, 70 rows of
# 3001 the 32 x 32 ones, 3 rows the 16 x 16 ones
WIDE = synth.ModelShape("wide32f", 1, 128, 2, 1, 64, 192, 6001, 10000.0, "fp32", 0.08)
MID = synth.ModelShape("mid32f", 2, 192, 3, 3, 64, 320, 3001, 10000.0, "fp32", 0.08)
HD128 = synth.ModelShape("hd128f", 2, 256, 2, 1, 128, 128, 333, 10000.0, "fp32", 0.08)


@pytest.mark.parametrize("shape,lens", [(WIDE, [200, 317]), (MID, [1, 33, 36]), (HD128, [17, 3])], ids=["64", "32", "16"])
def test_plain_gemm_tiles_against_oracle(shape, lens):
    B, Lmax = len(lens), max(lens)
    wp, wr = synth.make_weights(shape, 1, DEV), synth.make_weights(shape, 2, DEV)
    Wp, Wr = R.Weights(wp), R.Weights(wr)
    ro = R.Rollout(R.make_cfg(shape, B, Lmax), Wp, DEV)
    rng = np.random.default_rng(7)
    ids = rng.integers(0, shape.vocab, size=(B, Lmax)).astype(np.int32)
    L = np.array(lens, np.int32)
    P = np.maximum(1, L // 2).astype(np.int32)
    outs = [torch.full((B, Lmax), 7.0, dtype=torch.float32, device=DEV) for _ in range(4)]
    ro.score_logprobs_kl(Wp, Wr, torch.tensor(ids, device=DEV), L, P, 0.003, *outs)
    ro.rollout_check()
    mp, mr = (O.Model(shape, synth.weights_for_oracle(w)) for w in (wp, wr))
    check_scores(*[o.cpu().numpy() for o in outs], O.score_batch(mp, mr, ids, L, P, 0.003), 1e-4, 0.003)
    ro.close()


@pytest.mark.parametrize("shape", [MID, HD128], ids=["hd64", "hd128"])
def test_plain_decode_captured_and_eager(shape):
    """A captured step (side stream) gives the eager step's tokens and log-probs bit for bit, also when the next run's
    contexts are longer than the first one's; both match the oracle."""
    B, P, G = 3, 21, 30
    wp = synth.make_weights(shape, 1, DEV)
    ro = R.Rollout(R.make_cfg(shape, B, 64 + G), R.Weights(wp), DEV)
    side = torch.cuda.Stream()
    m = O.Model(shape, synth.weights_for_oracle(wp))
    out = torch.zeros(B, G, dtype=torch.int32, device=DEV)
    lp = torch.zeros(B, G, dtype=torch.float32, device=DEV)
    for pmax in (P, 64):
        ids, lens = synth.make_prompts(shape.vocab, B, pmax, 5, 3)
        got = []
        for stream in (side, torch.cuda.default_stream(), side):
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                ro.rollout_generate(R.sample_cfg(4, 0.7), torch.tensor(ids, device=DEV), lens, G, out, None, lp)
            torch.cuda.synchronize()
            ro.rollout_check()
            got.append((out.cpu().numpy().copy(), lp.cpu().numpy().copy()))
        for o, l in got[1:]:
            assert np.array_equal(o, got[0][0]) and np.array_equal(l, got[0][1])
        verify_rollout(m, [ids[b, :lens[b]] for b in range(B)], got[0][0], got[0][1], 0.7, 4, 0, 1e-5, 1e-4)
    ro.close()
