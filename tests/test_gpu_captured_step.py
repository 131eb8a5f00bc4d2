"""The captured decode step when calls follow each other without a wait: every call returns with its replays queued."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
PLAIN = synth.ModelShape("cap32f", 2, 128, 2, 1, 64, 192, 333, 10000.0, "fp32", 0.08)
TUNED = synth.ModelShape("cap16", 2, 256, 4, 2, 64, 256, 512, 10000.0, "bf16", 0.08)


@pytest.mark.parametrize("shape", [PLAIN, TUNED], ids=["plain", "tuned"])
def test_steps_replaced_while_their_replays_are_queued(shape):
    """Runs of other seeds, batches and output buffers, and queue runs, issued on one side stream without a wait in
    between: each replaces the captured step of the one before, whose replays are still queued, and gives what it gives
    when everything is waited for.  More runs than the number of replaced steps that are kept."""
    B, P, G, runs = 5, 12, 40, 14
    w = synth.make_weights(shape, 1, DEV)
    ro = R.Rollout(R.make_cfg(shape, B, P + G), R.Weights(w), DEV)
    ids, lens = synth.make_prompts(shape.vocab, B + 3, P, 3, 3)
    dev_ids = torch.tensor(ids, device=DEV)
    limit = (np.arange(B + 3) % 9 + 2).astype(np.int32)
    side = torch.cuda.Stream()

    def run_all(wait):
        res = [(torch.zeros(B + 3, G, dtype=torch.int32, device=DEV), torch.zeros(B + 3, G, device=DEV)) for _ in range(runs)]
        qlen = torch.zeros(B + 3, dtype=torch.int32, device=DEV)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for i, (out, lp) in enumerate(res):
                if i % 6 == 5:
                    ro.rollout_generate_queue(R.sample_cfg(i, 0.9), dev_ids, lens, limit, G, out, qlen, lp)
                else:
                    n = B - i % 2
                    ro.rollout_generate(R.sample_cfg(i, 0.9), dev_ids[:n], lens[:n], G, out[:n], None, lp[:n])
                if wait:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        ro.rollout_check()
        return [(o.cpu().numpy(), l.cpu().numpy()) for o, l in res]

    want, got = run_all(True), run_all(False)
    for i, (a, b) in enumerate(zip(want, got)):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), i
    assert any(not np.array_equal(want[0][0], x[0]) for x in want[1:])
    ro.close()
