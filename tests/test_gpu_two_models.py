"""Scoring two models in one pass (sequences listed twice, each half of the rows on its own weight set): bit for bit what
two passes give, whichever of the sets have an fp16 copy."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPE = synth.ModelShape("two512", 2, 512, 8, 2, 128, 1024, 2048, 10000.0, "bf16", 0.05)


def _ids(B, L):
    return np.random.default_rng(7).integers(0, SHAPE.vocab, size=(B, L)).astype(np.int32)


def _run(impl, copies, rows, lens, plens, L, wp, wr, alone):
    """Log-probs of both models, their KL terms and the exact KL; with alone, the log-probs from one call per model."""
    B = len(lens)
    cfg = R.make_cfg(SHAPE, B, L, max_chunk_tokens=rows)
    buf = [torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if on else None for on in copies]
    Wp, Wr = R.Weights(wp, shadow=buf[0]), R.Weights(wr, shadow=buf[1])
    ro = R.Rollout(cfg, Wp, DEV)
    ro.rollout_set_impl(impl)
    ids = torch.tensor(_ids(B, L), device=DEV)
    outs = [torch.full((B, L), 9.0, device=DEV) for _ in range(5)]
    if alone:
        for w, o in zip((Wp, Wr), outs):
            ro.score_logprobs_kl(w, None, ids, lens, plens, 0.0, o)
    else:
        ro.score_logprobs_kl(Wp, Wr, ids, lens, plens, 0.003, *outs[:4])
    ro.score_kl_exact(Wp, Wr, ids, lens, plens, outs[4])
    ro.rollout_check()
    ro.close()
    return [o.cpu().numpy() for o in outs]


@pytest.mark.parametrize("copies", [(False, False), (True, False), (True, True)], ids=["none", "policy", "both"])
@pytest.mark.parametrize("impl", [1, 2], ids=["by-size", "large-m"])
def test_one_pass_gives_the_bits_of_two(impl, copies):
    """One chunk of both models; several of them; and, for comparison, the same sequences at the head of a chunk of more than
    8192 rows, which the workspace does not hold twice and which is run for one model after the other (with a last chunk
    behind it that is again run for both together)."""
    lens = np.array([1, 33, 64, 150, 200, 97, 31], np.int32)               # 704 rows with their padding
    plens = np.array([1, 10, 64, 1, 100, 96, 1], np.int32)                 # one prompt without a response
    more = np.concatenate([lens, np.random.default_rng(11).integers(150, 201, size=53).astype(np.int32)])
    wp, wr = synth.make_weights(SHAPE, 1, DEV), synth.make_weights(SHAPE, 2, DEV)
    B, L = len(lens), int(lens.max())
    apart = _run(impl, copies, 10016, more, np.concatenate([plens, np.maximum(1, more[B:] // 2)]).astype(np.int32), L, wp, wr, True)
    for rows in (1024, 416):
        got = _run(impl, copies, rows, lens, plens, L, wp, wr, False)
        for i in (0, 1, 4):
            assert np.isfinite(got[i]).all() and np.array_equal(got[i], apart[i][:B]), (rows, i)
        assert np.abs(got[0] - got[1]).max() > 0.1 and np.abs(got[4]).max() > 0
    whole = _run(impl, copies, 10016, more, np.ones(len(more), np.int32), L, wp, wr, False)
    assert all(np.array_equal(whole[i], apart[i]) for i in (0, 1))


@pytest.mark.parametrize("copies", [(False, False), (True, False), (False, True), (True, True)], ids=["none", "policy", "reference", "both"])
@pytest.mark.parametrize("impl", [1, 2], ids=["by-size", "large-m"])
def test_weights_converted_for_both_models(impl, copies):
    """Chunks of 2048 to 4095 rows per model: the pair layer's GEMMs count twice as long and have the weight sets that bring no
    copy converted into idle workspace, both or one of them, behind one another.  Against one model at a time."""
    r = np.random.default_rng(17)
    lens = r.integers(150, 201, size=50).astype(np.int32)
    plens = np.maximum(1, lens // 2).astype(np.int32)
    rows = (lens + 31) // 32 * 32
    assert 4096 < rows.sum() < 16384 and rows.max() <= 224          # chunks of 3500: two full ones and more than 2048 rows behind
    L = int(lens.max())
    wp, wr = synth.make_weights(SHAPE, 1, DEV), synth.make_weights(SHAPE, 2, DEV)
    alone = _run(impl, copies, 10016, lens, plens, L, wp, wr, True)
    both = _run(impl, copies, 3500, lens, plens, L, wp, wr, False)
    for i in (0, 1, 4):
        assert np.isfinite(both[i]).all() and np.array_equal(both[i], alone[i]), i


@pytest.mark.parametrize("copies,rows,passes", [((True, False), 2048, 1), ((True, False), 2176, 2), ((False, True), 2176, 2),
                                               ((False, False), 2176, 1), ((True, True), 2176, 1)])
def test_one_copy_joins_only_small_passes(copies, rows, passes):
    """Width 4096: with a copy of one model of two, 2048 rows are the most that run as one pass (its GEMMs read no copy).
    Counted in GEMM launches, four per layer and pass; the results are those of the models alone."""
    s = synth.ModelShape("wide", 1, 4096, 2, 1, 64, 256, 256, 10000.0, "bf16", 0.02)
    L = rows // 4
    cfg = R.make_cfg(s, 4, L)
    W = [R.Weights(synth.make_weights(s, i + 1, DEV),
                   shadow=torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if on else None)
         for i, on in enumerate(copies)]
    ro = R.Rollout(cfg, W[0], DEV)
    ids = torch.tensor(np.random.default_rng(1).integers(0, s.vocab, size=(4, L)).astype(np.int32), device=DEV)
    lens, plens = np.full(4, L, np.int32), np.ones(4, np.int32)
    alone = [torch.zeros(4, L, device=DEV) for _ in W]
    for w, o in zip(W, alone):
        ro.score_logprobs_kl(w, None, ids, lens, plens, 0.0, o)
    both = [torch.zeros(4, L, device=DEV) for _ in W]
    ro.rollout_profile_enable(R.RL_K_GEMM_PREFILL, 1)
    ro.score_logprobs_kl(*W, ids, lens, plens, 0.0, *both)
    launches = ro.rollout_profile_read(R.RL_K_GEMM_PREFILL)[1]
    ro.rollout_check()
    ro.close()
    assert launches == 4 * passes
    assert all(torch.equal(a, b) for a, b in zip(alone, both))


@pytest.mark.parametrize("two_models,max_batch,passes", [(True, 7, 1), (False, 7, 2), (False, 14, 1)])
def test_workspace_of_either_size(two_models, max_batch, passes):
    """The smaller workspace serves every call: two models run one after the other in it, or as one pass where the chunk is
    small enough and half of max_batch lists its sequences (704 rows of 1408, 7 sequences).  One byte less is refused."""
    lens = np.array([1, 33, 64, 150, 200, 97, 31], np.int32)
    plens = np.array([1, 10, 64, 1, 100, 96, 1], np.int32)
    B, L = len(lens), int(lens.max())
    cfg = R.make_cfg(SHAPE, max_batch, L, max_chunk_tokens=704 if max_batch == 7 else 1408)
    need, scoring = R.rollout_workspace_bytes(cfg), R.rollout_scoring_workspace_bytes(cfg)
    assert need < scoring
    wp, wr = synth.make_weights(SHAPE, 1, DEV), synth.make_weights(SHAPE, 2, DEV)
    Wp, Wr = R.Weights(wp), R.Weights(wr)
    h = R.C.c_void_p()
    kv = torch.empty(R.rollout_kv_pool_bytes(cfg), dtype=torch.uint8, device=DEV)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    assert R.lib().rollout_init(R.C.byref(cfg), R.C.byref(Wp.struct), R._ptr(ws), need - 1, R._ptr(kv), kv.numel(),
                                R.C.byref(h)) == R.RL_ENOSPACE
    ro = R.Rollout(cfg, Wp, DEV, two_models=two_models)
    assert ro.workspace.numel() == (scoring if two_models else need)
    ids = torch.tensor(_ids(B, L), device=DEV)
    outs = [torch.full((B, L), 9.0, device=DEV) for _ in range(5)]
    ro.rollout_profile_enable(R.RL_K_GEMM_PREFILL, 1)
    ro.score_logprobs_kl(Wp, Wr, ids, lens, plens, 0.003, *outs[:4])
    assert ro.rollout_profile_read(R.RL_K_GEMM_PREFILL)[1] == 4 * SHAPE.n_layers * passes
    ro.score_kl_exact(Wp, Wr, ids, lens, plens, outs[4])
    ro.rollout_check()
    ro.close()
    want = _run(1, (False, False), 1024, lens, plens, L, wp, wr, True)
    for i in (0, 1, 4):
        assert np.array_equal(outs[i].cpu().numpy(), want[i])
