"""The large-M GEMM's tile heights (96 to 256 rows, chosen from the number of rows): every height gives the same bits."""
import numpy as np
import pytest
import torch

from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPE = synth.ModelShape("tiles1024", 2, 1024, 8, 2, 128, 1024, 2048, 10000.0, "bf16", 0.02)


def _height(rows, cols, residual):
    """The launcher's rule for a GEMM of K = 1024 (its plain layer, and the LM head): tile height / 32."""
    loop = {3: 0.575, 4: 0.62, 5: 0.76, 6: 0.855, 7: 0.95, 8: 1.0}

    def cost(mi):
        tiles = -(-rows // (32 * mi)) * (cols // 256)
        rest = tiles % 256 / 256
        return (tiles // 256 + (0.7 + 0.3 * rest if rest else 0)) * (loop[mi] * 32 + (24 if residual else 8) * mi / 8)
    return min(range(8, 2, -1), key=cost)


@pytest.mark.parametrize("copy", [False, True], ids=["bf16", "fp16copy"])
def test_tile_heights_give_the_same_bits(copy):
    """One chunk of many rows (tall tiles) against chunks of at most 1024 rows (96-row tiles throughout, which the
    oracle tests of the large-M kernel cover): scores equal bit for bit, last partial tile and ragged ends included.
    Without copies, 4096 rows and more also take the fp16 copy made in idle workspace (plain layer and LM head)."""
    w = synth.make_weights(SHAPE, 1, DEV)
    B, L = 32, 512
    res = {}
    totals = (2600, 3300, 3900, 5500, 7000, 8000, 9500, 11000, 13000, 15000)
    seen = {c: set() for c in ("qkv", "residual", "gate/up, LM head")}
    rng = np.random.default_rng(5)
    ids = rng.integers(0, SHAPE.vocab, size=(B, L)).astype(np.int32)
    d = torch.tensor(ids, device=DEV)
    for chunk in (16384, 1024):
        cfg = R.make_cfg(SHAPE, B, L, max_chunk_tokens=chunk)
        shadow = torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copy else None
        W = R.Weights(w, shadow=shadow)
        ro = R.Rollout(cfg, W, DEV)
        ro.rollout_set_impl(2)
        for n in totals:
            r = np.random.default_rng(n)
            lens = np.full(B, n // B, np.int32) + r.integers(-20, 21, size=B).astype(np.int32)
            plens = np.maximum(1, lens // 2).astype(np.int32)
            if chunk == 16384:                              # one chunk: every sequence starts at a multiple of 32 rows
                rows = int(((lens + 31) // 32 * 32).sum())
                for (name, s), cols in zip(seen.items(), (1536, 1024, 2048)):
                    s.add(_height(rows, cols, name == "residual"))
            lp = torch.full((B, L), 9.0, dtype=torch.float32, device=DEV)
            ro.score_logprobs_kl(W, None, d, lens, plens, 0.0, lp)
            ro.rollout_check()
            res[chunk, n] = lp.cpu().numpy()
        ro.close()
    assert all(s == {3, 4, 5, 6, 7, 8} for s in seen.values()), seen
    for n in totals:
        assert np.isfinite(res[1024, n]).all()
        assert np.array_equal(res[16384, n], res[1024, n]), n


@pytest.mark.parametrize("on", [True, False], ids=["on", "off"])
def test_copy_switch_leaves_sets_without_a_copy_alone(on):
    """rollout_set_large_gemm_copy only decides whether existing copies are read: with the switch off, a set that has none
    still has its LM head converted into idle workspace ahead of a GEMM of 4096 rows (the converted rows are still there
    after the call), as does a set that has one, and nobody reads the copy (which is overwritten here)."""
    w = synth.make_weights(SHAPE, 77 + on, DEV)
    B, L = 8, 512
    ids = torch.tensor(np.random.default_rng(5).integers(0, SHAPE.vocab, size=(B, L)).astype(np.int32), device=DEV)
    lens = np.full(B, L, np.int32)
    cfg = R.make_cfg(SHAPE, B, L)
    first = w["lm_head"][0, :128].half().view(torch.int64)                  # 256 bytes
    got = []
    R.rollout_set_large_gemm_copy(on)
    try:
        for copy in (False, True) if not on else (False,):
            shadow = torch.empty(R.rollout_weight_shadow_bytes(cfg), dtype=torch.uint8, device=DEV) if copy else None
            W = R.Weights(w, shadow=shadow)
            ro = R.Rollout(cfg, W, DEV)
            ro.rollout_set_impl(2)
            if copy:
                shadow.fill_(0xff)
            lp = torch.zeros(B, L, device=DEV)
            ro.score_logprobs_kl(W, None, ids, lens, lens // 2, 0.0, lp)
            ro.rollout_check()
            ws = ro.workspace[:ro.workspace.numel() // 256 * 256].view(torch.int64).view(-1, 32)
            assert (ws == first).all(dim=1).any()
            got.append(lp.cpu().numpy())
            ro.close()
    finally:
        R.rollout_set_large_gemm_copy(True)
    assert all(np.isfinite(g).all() and np.array_equal(g, got[0]) for g in got)
