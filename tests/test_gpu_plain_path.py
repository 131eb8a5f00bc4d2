"""The plain path's kernels at the sizes where they can go wrong, against the oracle: the GEMM's three tile sizes with
remainders in rows and columns under every epilogue, the captured decode step against the eager one, and the longest
context."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import check_scores, verify_rollout

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# widths that are no multiple of any tile; the rows of a scoring pass are one chunk, of which the LM head takes 512 at a time
WIDE = synth.ModelShape("wide32f", 1, 128, 2, 1, 64, 192, 6001, 10000.0, "fp32", 0.08)
MID = synth.ModelShape("mid32f", 2, 192, 3, 3, 64, 320, 3001, 10000.0, "fp32", 0.08)
HD128 = synth.ModelShape("hd128f", 2, 256, 2, 1, 128, 128, 333, 10000.0, "fp32", 0.08)
# layer GEMMs on taller tiles: the O and down projections (residual) and gate/up (SwiGLU) with few k and many columns
LAYER32 = synth.ModelShape("layer32", 1, 1536, 2, 1, 64, 1600, 130, 10000.0, "fp32", 0.03)
LAYER64 = synth.ModelShape("layer64", 1, 2048, 2, 1, 64, 2112, 130, 10000.0, "fp32", 0.03)


def _tile(rows, cols):
    """The launcher's rule: the largest tile that gives the 256 compute units two workgroups each."""
    for t in (64, 32):
        if -(-rows // t) * -(-cols // t) >= 512:
            return t
    return 16


# tile of the QKV, O, gate/up and down GEMMs, and of the LM head's blocks of rows; each taller tile meets a remainder of rows
# and, in the LM head, of columns (the layers' widths are multiples of 64)
CASES = {
    "head64": (WIDE, [200, 250], (16, 16, 16, 16), {64}),
    "head32": (MID, [100, 33, 67], (16, 16, 16, 16), {32}),
    "16": (HD128, [17, 3], (16, 16, 16, 16), {16}),
    "layer32": (LAYER32, [200, 133], (16, 32, 32, 32), {16}),
    "layer64": (LAYER64, [600, 425], (16, 64, 64, 64), {16}),
}


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("name", CASES)
def test_plain_gemm_tiles_against_oracle(name, dtype):
    """fp32 has the norm inside the GEMM; bf16 weights (plain kernels asked for) have it in a kernel of its own."""
    shape, lens, layer_tiles, head_tiles = CASES[name]
    shape = synth.scaled_shape(shape, shape.name, dtype=dtype)
    B, Lmax, n = len(lens), max(lens), sum(lens)
    qd = shape.n_q_heads * shape.head_dim
    assert tuple(_tile(n, w) for w in (qd + 2 * shape.n_kv_heads * shape.head_dim, shape.d_model, shape.d_ffn,
                                       shape.d_model)) == layer_tiles
    assert {_tile(min(512, n - r), shape.vocab) for r in range(0, n, 512)} == head_tiles
    wp, wr = synth.make_weights(shape, 1, DEV), synth.make_weights(shape, 2, DEV)
    Wp, Wr = R.Weights(wp), R.Weights(wr)
    ro = R.Rollout(R.make_cfg(shape, B, Lmax), Wp, DEV)
    if dtype == "bf16":
        ro.rollout_set_impl(0)
    rng = np.random.default_rng(7)
    ids = rng.integers(0, shape.vocab, size=(B, Lmax)).astype(np.int32)
    L = np.array(lens, np.int32)
    P = np.maximum(1, L // 2).astype(np.int32)
    outs = [torch.full((B, Lmax), 7.0, dtype=torch.float32, device=DEV) for _ in range(4)]
    ro.score_logprobs_kl(Wp, Wr, torch.tensor(ids, device=DEV), L, P, 0.003, *outs)
    ro.rollout_check()
    mp, mr = (O.Model(shape, synth.weights_for_oracle(w)) for w in (wp, wr))
    check_scores(*[o.cpu().numpy() for o in outs], O.score_batch(mp, mr, ids, L, P, 0.003),
                 1e-4 if dtype == "fp32" else 2e-2, 0.003)
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


def test_plain_attention_longest_context():
    """The longest context whose scores a workgroup's LDS holds (head_dim + 16 + 256 floats of its 160 KB are taken by
    everything else): prefill, decode and scoring take it.  One layer, so the last positions' keys and values come
    straight from the embeddings and the oracle's formulas need one query at a time."""
    shape = synth.ModelShape("long32f", 1, 64, 1, 1, 64, 64, 97, 10000.0, "fp32", 0.3)
    most, G = 163840 // 4 - (64 + 16 + 256), 6
    w = synth.make_weights(shape, 1, DEV)
    W = R.Weights(w)
    ro = R.Rollout(R.make_cfg(shape, 1, most), W, DEV)
    P = most - G + 1                                        # the last decode step attends to `most` keys
    ids = np.random.default_rng(5).integers(0, shape.vocab, size=(1, P)).astype(np.int32)
    out = torch.zeros(1, G, dtype=torch.int32, device=DEV)
    lp = torch.zeros(1, G, device=DEV)
    ro.rollout_generate(R.sample_cfg(4, 0.0), torch.tensor(ids, device=DEV), [P], G, out, None, lp)
    ro.rollout_check()
    full = np.concatenate([ids, out.cpu().numpy()], axis=1)[:, :most]
    scored = torch.zeros(1, most, device=DEV)
    ro.score_logprobs_kl(W, None, torch.tensor(full, device=DEV), [most], [P], 0.003, scored)
    ro.rollout_check()
    o = synth.weights_for_oracle(w)
    l = {k: np.asarray(v, np.float64) for k, v in o["layers"][0].items()}
    x = np.asarray(o["tok_embed"], np.float64)[full[0]]
    qkv = O.rmsnorm(x, l["attn_norm"], shape.rms_eps) @ l["wqkv"].T
    pos = np.arange(most)
    q, k = (O.rope(qkv[:, None, i * 64:i * 64 + 64], pos, shape.rope_base)[:, 0] for i in (0, 1))
    v = qkv[:, 128:]
    for t in range(P - 1, most):                            # the state after token t draws token t + 1
        s = k[:t + 1] @ q[t] / 8.0
        p = np.exp(s - s.max())
        h = x[t] + (p @ v[:t + 1] / p.sum()) @ l["wo"].T
        n = O.rmsnorm(h[None], l["ffn_norm"], shape.rms_eps)[0]
        g, u = l["w_gate_up"][:64] @ n, l["w_gate_up"][64:] @ n
        h = h + l["w_down"] @ (g / (1 + np.exp(-g)) * u)
        z = np.asarray(o["lm_head"], np.float64) @ O.rmsnorm(h[None], np.asarray(o["final_norm"], np.float64), shape.rms_eps)[0]
        lse = z.max() + np.log(np.exp(z - z.max()).sum())
        tok = int(out[0, t - P + 1])
        assert z[tok] > z.max() - 1e-3
        assert abs(float(lp[0, t - P + 1]) - (z[tok] - lse)) < 1e-4
        if t + 1 < most:
            assert abs(float(scored[0, t + 1]) - (z[tok] - lse)) < 1e-4
    ro.close()
