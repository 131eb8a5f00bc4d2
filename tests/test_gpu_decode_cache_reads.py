"""Decode attention reads large caches as non-temporal.  Which form runs follows from the rows and the longest context of a run, not
from what the context could hold; both forms give the same bits, whatever the head dimension, waves and key splits, in plain and pair
layers, whether the attention consumes the QKV partial sums or not."""
import re

import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import kernels_run

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
LIMIT = 100 << 20


def _forms(names):
    """(pair, non-temporal) of the decode attention kernels among them, and their wave counts."""
    found = [re.search(r"attn_decode_kernel<(\d+), 16, (\w+), (\w+), (\d), (\w+)>", n) for n in names]
    found = [m for m in found if m]
    return {(m[2] == "true", m[5] == "true") for m in found}, {int(m[4]) for m in found}


@pytest.mark.parametrize("fused", [True, False], ids=["consumer", "separate"])
@pytest.mark.parametrize("hd,Hkv,B,waves", [(64, 8, 32, 8), (64, 8, 64, 4), (128, 4, 24, 8), (128, 8, 64, 4)])
def test_cache_reads_follow_the_run(hd, Hkv, B, waves, fused):
    """One context with room for long sequences: a run whose longest row makes the cache large, one between the pair layer's line
    and the plain layer's, a short one and the first again, all with the same buffers on one stream, so that a captured step is
    replaced where the form changes.  (128, 4, 24) splits the keys."""
    shape, G = synth.ModelShape("reads", 2, 512, 2 * Hkv, Hkv, hd, 512, 1024, 10000.0, "bf16", 0.05), 4
    key = Hkv * hd * 4
    most = LIMIT // (B * key) + 80
    ro = R.Rollout(R.make_cfg(shape, B, most + 20), R.Weights(synth.make_weights(shape, 1, DEV)), DEV)
    ro.rollout_set_fused_qkv_consumer(fused)
    rng = np.random.default_rng(3)
    ids = torch.tensor(rng.integers(0, shape.vocab, size=(B, most)).astype(np.int32), device=DEV)
    side = torch.cuda.Stream()
    out, lp = torch.zeros(B, G, dtype=torch.int32, device=DEV), torch.zeros(B, G, device=DEV)
    one, one_lp = torch.zeros(1, G, dtype=torch.int32, device=DEV), torch.zeros(1, G, device=DEV)
    torch.cuda.synchronize()

    def generate(ids, lens, out, lp, first=0):
        with torch.cuda.stream(side):
            ro.rollout_generate(R.sample_cfg(4, 0.7, -1, first), ids, lens, G, out, None, lp)
        torch.cuda.synchronize()
        ro.rollout_check()
        return out.cpu().numpy(), lp.cpu().numpy()

    between = LIMIT // (B * key) * 3 // 4
    for longest, forms in [(most, {(True, True), (False, True)}), (between, {(True, True), (False, False)}),
                           (64, {(True, False), (False, False)}), (most, {(True, True), (False, True)})]:
        lens = rng.integers(1, 60, size=B).astype(np.int32)
        lens[-1] = longest + 1 - G
        want = generate(ids, lens, out, lp)
        got, w = _forms(kernels_run(lambda: generate(ids, lens, out, lp)))            # the step captured before
        assert got == forms and w == {waves}, (longest, got, w)
        again = out.cpu().numpy(), lp.cpu().numpy()
        assert np.array_equal(want[0], again[0]) and np.array_equal(want[1], again[1])
        for b in (0, B - 1):                                                          # alone a row's cache is small
            o, l = generate(ids[b:b + 1].contiguous(), lens[b:b + 1], one, one_lp, b)
            assert np.array_equal(o[0], want[0][b]) and np.array_equal(l[0], want[1][b])
    ro.close()
