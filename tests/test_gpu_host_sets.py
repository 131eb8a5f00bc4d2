"""Host-resident weight sets: what may be changed or used again when a call returns."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPE = synth.ModelShape("hostset", 10, 1024, 8, 2, 128, 4096, 16384, 10000.0, "bf16", 0.02)


def _tensors(w):
    return [w["tok_embed"], w["final_norm"], w["lm_head"]] + [t for lay in w["layers"] for t in lay.values()]


@pytest.mark.parametrize("call", ["logprobs", "values"])
def test_host_tensors_may_change_when_the_call_returns(call):
    """Every host tensor is overwritten right behind the call, without a wait for the stream; the scores are those of the
    same set device-resident.  The uploads take milliseconds and wait for layers of 4096 rows."""
    B, L = 16, 256
    w = synth.make_weights(SHAPE, 1, DEV)
    cfg = R.make_cfg(SHAPE, B, L)
    W = R.Weights(w)
    ro = R.Rollout(cfg, W, DEV)
    staging = torch.empty(R.rollout_weight_staging_bytes(cfg), dtype=torch.uint8, device=DEV)
    ids = torch.tensor(np.random.default_rng(3).integers(0, SHAPE.vocab, size=(B, L)).astype(np.int32), device=DEV)
    lens, head = np.full(B, L, np.int32), torch.ones(SHAPE.d_model, dtype=SHAPE.torch_dtype, device=DEV)
    host = [torch.empty(t.shape, dtype=t.dtype, pin_memory=True) for t in _tensors(w)]
    it = iter(host)
    named = {k: next(it) for k in ("tok_embed", "final_norm", "lm_head")}
    named["layers"] = [{k: next(it) for k in lay} for lay in w["layers"]]

    def score(model):
        out = torch.zeros(B, L, device=DEV)
        if call == "values":
            ro.score_values(model, head, ids, lens, out)
        else:
            ro.score_logprobs_kl(model, None, ids, lens, lens // 2, 0.0, out)
        return out

    want = score(W).cpu().numpy()
    streamed = R.Weights(named, staging=staging)
    for _ in range(2):
        for h, t in zip(host, _tensors(w)):
            h.copy_(t)
        torch.cuda.synchronize()
        got = score(streamed)
        for h in host:
            h.zero_()
        assert np.array_equal(got.cpu().numpy(), want) and np.abs(want).max() > 0
    ro.rollout_check()
    ro.close()


def _pinned(w):
    pin = lambda t: t.cpu().pin_memory()   # noqa: E731
    out = {k: pin(w[k]) for k in ("tok_embed", "final_norm", "lm_head")}
    out["layers"] = [{k: pin(v) for k, v in lay.items()} for lay in w["layers"]]
    return out


@pytest.mark.parametrize("overwrite", [False, True], ids=["buffers-alternate", "host-tensors-change"])
def test_policies_swapped_in_without_waits(overwrite):
    """Policies uploaded in turn into two device buffers, each generating, with no wait anywhere.  The third goes into the
    first one's buffer while that one's long run is still queued.  With `overwrite` every set's host tensors are
    overwritten (the last to be uploaded first) when the first call under it has returned."""
    shape = synth.ModelShape("swaps", 3, 1024, 8, 2, 128, 2048, 32768, 10000.0, "bf16", 0.02)
    B, P, runs = 8, 8, (400, 3, 5)
    cfg = R.make_cfg(shape, B, P + max(runs))
    ids, lens = synth.make_prompts(shape.vocab, B, P, 3, 3)
    ids = torch.tensor(ids, device=DEV)
    sets = [synth.make_weights(shape, i, DEV) for i in (1, 2, 3)]
    ro = R.Rollout(cfg, R.Weights(sets[2]), DEV)
    bufs = [torch.empty(R.rollout_weight_resident_bytes(cfg), dtype=torch.uint8, device=DEV) for _ in range(2)]
    side = torch.cuda.Stream()

    def swap_all(wait):
        host = [_pinned(w) for w in sets]
        outs = [(torch.zeros(B, g, dtype=torch.int32, device=DEV), torch.zeros(B, g, device=DEV)) for g in runs]
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for i, (out, lp) in enumerate(outs):
                ro.rollout_set_policy(R.Weights(host[i], staging=bufs[i % 2]))
                ro.rollout_generate(R.sample_cfg(4, 1.0), ids, lens, runs[i], out, None, lp)
                if overwrite and not wait:
                    for t in reversed(_tensors(host[i])):
                        t.zero_()
                if wait:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        return [(o.cpu().numpy(), l.cpu().numpy()) for o, l in outs]

    for want, got in zip(swap_all(True), swap_all(False)):
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    ro.rollout_check()
    ro.close()
