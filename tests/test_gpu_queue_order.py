"""The queue's order: longest limits first where the page pool holds them together, as they come where it does not."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [synth.ModelShape("qo128", 2, 256, 4, 2, 128, 512, 1024, 10000.0, "bf16", 0.06),
          synth.ModelShape("qo32f", 2, 128, 4, 2, 64, 256, 1000, 10000.0, "fp32", 0.08)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("limits", [[40, 3, 3, 3, 3, 3, 3, 40], [1, 2, 9, 17, 33, 40, 40, 5, 8, 16, 24], [7, 7, 7]],
                         ids=["two-long", "mixed", "equal"])
def test_rows_do_not_depend_on_the_order(shape, limits):
    """A row takes at most four pages (16 cached prompt tokens and 40 generated).  Two slots and eight pages: longest first.
    Six pages: as they come, which here never has both long rows live (longest first would run out of pages)."""
    lim = np.array(limits, np.int32)
    Q, P = len(lim), 17
    w = synth.make_weights(shape, 1, DEV)
    ids = torch.tensor(np.random.default_rng(5).integers(0, shape.vocab, size=(Q, P)).astype(np.int32), device=DEV)
    plen = np.full(Q, P, np.int32)
    got = []
    for slots, pages in ((2, 8), (2, 6), (3, 12), (1, 4)) if limits[0] == 40 else ((2, 8), (3, 12), (1, 4)):
        ro = R.Rollout(R.make_cfg(shape, slots, 64, n_pages=pages), R.Weights(w), DEV)
        out, n = torch.zeros(Q, 40, dtype=torch.int32, device=DEV), torch.zeros(Q, dtype=torch.int32, device=DEV)
        lp = torch.zeros(Q, 40, device=DEV)
        ro.rollout_generate_queue(R.sample_cfg(3, 1.0), ids, plen, lim, 40, out, n, lp)
        ro.rollout_check()
        assert np.array_equal(n.cpu().numpy(), lim)
        got.append((out.cpu().numpy(), lp.cpu().numpy()))
        ro.close()
    for o, l in got[1:]:
        assert np.array_equal(o, got[0][0])
        if shape.dtype == "bf16":
            assert np.array_equal(l, got[0][1])
        else:
            assert np.abs(l - got[0][1]).max() < 1e-5


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("pages,steps", [(8, 64), (6, 96)], ids=["longest-first", "as-they-come"])
def test_decode_steps_of_either_order(shape, pages, steps):
    """Limits 40, six times 3, 40 on two slots, steps in bursts of eight, counted in attention launches.  Longest first: both
    long rows (five bursts), then the short ones two at a time as soon as a slot is free (three bursts).  As they come, refilled
    when both slots are free: 40 steps for rows 0 and 1, 8 for 2 and 3, 8 for 4 and 5, 40 for 6 and 7."""
    lim = np.array([40, 3, 3, 3, 3, 3, 3, 40], np.int32)
    Q, P = len(lim), 17
    ro = R.Rollout(R.make_cfg(shape, 2, 64, n_pages=pages), R.Weights(synth.make_weights(shape, 1, DEV)), DEV)
    ids = torch.tensor(np.random.default_rng(5).integers(0, shape.vocab, size=(Q, P)).astype(np.int32), device=DEV)
    out, n = torch.zeros(Q, 40, dtype=torch.int32, device=DEV), torch.zeros(Q, dtype=torch.int32, device=DEV)
    ro.rollout_profile_enable(R.RL_K_ATTN_DECODE, 1)
    ro.rollout_generate_queue(R.sample_cfg(3, 1.0), ids, np.full(Q, P, np.int32), lim, 40, out, n)
    launches = ro.rollout_profile_read(R.RL_K_ATTN_DECODE)[1]
    ro.rollout_check()
    ro.close()
    assert np.array_equal(n.cpu().numpy(), lim)
    assert launches == steps * shape.n_layers
