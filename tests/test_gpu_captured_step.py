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


@pytest.mark.parametrize("shape", [PLAIN, TUNED], ids=["plain", "tuned"])
def test_calls_refused_while_the_stream_is_captured(shape):
    """Prefill, generation, scoring and reward calls move host state on with the work they queue: on a stream under
    capture they are refused before they record or change anything, and the capture goes on."""
    B, P, G = 3, 9, 4
    w, w2 = synth.make_weights(shape, 1, DEV), synth.make_weights(shape, 2, DEV)
    cfg = R.make_cfg(shape, B, P + G)
    copy = shape.dtype == "bf16"
    shadow = torch.zeros(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copy else None
    W, W2 = R.Weights(w), R.Weights(w2, shadow=shadow)
    ro = R.Rollout(cfg, W, DEV)
    ids, lens = synth.make_prompts(shape.vocab, B, P, 3, 3)
    ids, half = torch.tensor(ids, device=DEV), np.maximum(1, lens // 2)
    f32 = lambda *n: torch.zeros(*n, device=DEV)   # noqa: E731
    out, qlen = torch.zeros(B, G, dtype=torch.int32, device=DEV), torch.zeros(B, dtype=torch.int32, device=DEV)
    head, sc, o = torch.ones(shape.d_model, dtype=shape.torch_dtype, device=DEV), R.sample_cfg(1, 0.0), f32(B, P)
    seq_reward, kl, marker = f32(B), f32(B, P), torch.ones(4, device=DEV)
    calls = [lambda: ro.rollout_prefill(ids, lens), lambda: ro.rollout_generate(sc, ids, lens, G, out),
             lambda: ro.rollout_generate_queue(sc, ids, lens, [G] * B, G, out, qlen),
             lambda: ro.score_logprobs_kl(W, W2, ids, lens, half, 0.1, o, f32(B, P)),
             lambda: ro.score_kl_exact(W, W2, ids, lens, half, o), lambda: ro.score_values(W, head, ids, lens, o),
             lambda: ro.ppo_rewards(kl, seq_reward, lens, half, 0.1, o)]
    scores = []

    def score():
        a, b = f32(B, P), f32(B, P)
        ro.score_logprobs_kl(W, W2, ids, lens, half, 0.1, a, b)
        ro.rollout_check()
        scores.append((a.cpu().numpy(), b.cpu().numpy()))

    ro.rollout_prefill(ids, lens)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    refused = 0
    with torch.cuda.stream(side):
        graph.capture_begin(capture_error_mode="thread_local")
        marker.zero_()
        for call in calls:
            try:
                call()
            except R.RolloutError as e:
                refused += e.code == R.RL_EHIP
        graph.capture_end()
    torch.cuda.synchronize()
    assert refused == len(calls)
    assert marker.sum() == 4
    graph.replay()
    torch.cuda.synchronize()
    assert marker.sum() == 0
    ro.rollout_decode_step(sc, None, qlen)                  # the sequences of the prefill before are still live
    score()                                                 # and the reference's copy is built by the first call that runs
    if copy:
        ro.rollout_forget_fp16_copies()
    score()
    assert all(np.array_equal(a, b) for a, b in zip(*scores)) and np.abs(scores[0][1]).max() > 0
    ro.close()
