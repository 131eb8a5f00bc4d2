"""The decode step's weight-streaming GEMMs (contexts of at most 64 and 128 rows): one to eight 16-row tiles of activations
with remainders, every number of tiles of W a gate/up or LM-head workgroup may take, K split and not, rows of a power of two long (start
rotated) and not, bf16 weights and an fp16 copy -- against the oracle, and row by row against smaller batches."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import verify_rollout

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# 16-row tiles of W that a workgroup of the gate/up GEMM and of the LM head takes (the LM head: even numbers only).  C's
# last gate/up workgroup is short, and its FFN width is no multiple of 128: the pair layer's down projection wraps inside
# a k-tile and runs on the 128 x 128 tile kernel.  (QKV, O and down projections take more than two tiles only at model
# widths, which the tests of the five configurations cover.)
SHAPES = {
    synth.ModelShape("stream_a", 2, 1024, 8, 2, 128, 14336, 32768, 10000.0, "bf16", 0.02): (7, 8),
    synth.ModelShape("stream_b", 2, 384, 6, 3, 64, 6144, 12288, 10000.0, "bf16", 0.04): (3, 4),
    synth.ModelShape("stream_c", 2, 256, 32, 8, 128, 10304, 24576, 10000.0, "bf16", 0.04): (6, 6),
    synth.ModelShape("stream_d", 2, 640, 10, 5, 64, 8320, 8064, 10000.0, "bf16", 0.04): (5, 2),
    synth.ModelShape("stream_e", 2, 256, 4, 2, 64, 2048, 4096, 10000.0, "bf16", 0.06): (1, 2),
    synth.ModelShape("stream_f", 2, 256, 4, 2, 64, 4096, 4096, 10000.0, "bf16", 0.06): (2, 2),
    synth.ModelShape("stream_g", 2, 256, 4, 2, 64, 8192, 4096, 10000.0, "bf16", 0.06): (4, 2),
    synth.ModelShape("stream_h", 2, 256, 4, 2, 64, 16384, 4096, 10000.0, "bf16", 0.06): (8, 2),
}


def _tiles(n_tiles, most, step):
    """The launcher's rule for a GEMM that is not split over K: fewest rounds of 256 workgroups, weighed by their size."""
    rows = 1 if most <= 64 else 4
    return min(range(step, 9, step), key=lambda c: -(-(-(-n_tiles // c)) // 256) * (c + rows))


@pytest.mark.parametrize("most", [64, 128])
@pytest.mark.parametrize("copy", [False, True], ids=["bf16", "fp16copy"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_stream_gemm_rows_and_widths(shape, copy, most):
    assert (_tiles(shape.d_ffn // 8, most, 1), _tiles(shape.vocab // 16, most, 2)) == SHAPES[shape]
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
        ro.rollout_generate(R.sample_cfg(4, 0.8), torch.tensor(ids[:n], device=DEV), lens[:n], G, out, None, lp)
        ro.rollout_check()
        res[n] = (out.cpu().numpy(), lp.cpu().numpy())
    for n in few:                                      # a row's bits do not depend on its batch-mates
        assert np.array_equal(res[n][0], res[most][0][:n]) and np.array_equal(res[n][1], res[most][1][:n]), n
    verify_rollout(m, [ids[b, :lens[b]] for b in range(most)], *res[most], 0.8, 4, 0, 1e-3, 2e-2, rows=[0, 16, most - 1])
    ro.close()


@pytest.mark.parametrize("most,max_seq,plen", [(64, 336, 300), (512, 4320, 4290)], ids=["8-waves", "4-waves-300-pages"])
def test_decode_attention_waves_and_page_blocks(most, max_seq, plen):
    """Eight waves on one (sequence, kv head) without splits, with remainders of pages per wave; and four waves over more
    pages than the 64 per wave whose numbers are fetched at once (a context for many sequences, one of them long)."""
    shape = synth.ModelShape("waves", 1, 256, 4, 2, 64, 256, 512, 10000.0, "bf16", 0.08)
    G, lens = 5, np.array([plen, 1, 17, 130], np.int32)
    w = synth.make_weights(shape, 1, DEV)
    ro = R.Rollout(R.make_cfg(shape, most, max_seq, n_pages=400, max_chunk_tokens=max(max_seq, 512)), R.Weights(w), DEV)
    ids = np.random.default_rng(3).integers(0, shape.vocab, size=(4, plen)).astype(np.int32)
    out = torch.full((4, G), -1, dtype=torch.int32, device=DEV)
    lp = torch.full((4, G), 9.0, dtype=torch.float32, device=DEV)
    ro.rollout_generate(R.sample_cfg(4, 0.8), torch.tensor(ids, device=DEV), lens, G, out, None, lp)
    ro.rollout_check()
    m = O.Model(shape, synth.weights_for_oracle(w))
    verify_rollout(m, [ids[b, :lens[b]] for b in range(4)], out.cpu().numpy(), lp.cpu().numpy(), 0.8, 4, 0, 1e-3, 2e-2)
    ro.close()
