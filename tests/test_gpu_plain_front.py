"""The fp32 decode step's fused front (norm, QKV projection, rotation, append and attention in one kernel) and its products for
few rows, against the oracle: every head group the kernel is built for, up to the widest it takes, widths that are no multiple of its
256-wide steps, as many blocks as it takes, contexts across its passes of 64 (head_dim 128: 32) keys, rows on both sides of the limit
of 8; and shapes just past it, which the separate kernels run."""
import numpy as np
import pytest
import torch

from oracle import rollout_oracle as O
from paper_2405_01481_amd import rollout as R
from paper_2405_01481_amd import synth
from tests.helpers import kernels_run, verify_rollout

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _shape(G, hd, d, F):
    return synth.ModelShape(f"front_{G}_{hd}", 2, d, 2 * G, 2, hd, F, 515, 10000.0, "fp32", 0.08)


def _ran(names):
    """Whether the fused front ran, and whether the product for few rows did."""
    return any("plain_front_kernel" in n for n in names), any("gemm_rows_kernel" in n for n in names)


@pytest.mark.parametrize("G,hd,d,F,B,front", [
    (1, 64, 64, 64, 1, True), (2, 64, 320, 320, 4, True), (4, 64, 256, 576, 5, True), (1, 128, 192, 448, 8, True),
    (2, 128, 128, 320, 9, True), (1, 64, 640, 320, 2, True), (2, 64, 512, 64, 4, True), (1, 128, 320, 64, 6, True),
    (2, 128, 256, 320, 8, True), (1, 64, 64, 64, 128, True), (1, 64, 64, 64, 129, False), (1, 64, 704, 64, 2, False),
    (2, 64, 576, 64, 2, False), (4, 64, 320, 64, 3, False), (1, 128, 384, 64, 2, False), (2, 128, 320, 64, 2, False),
    (4, 128, 128, 64, 3, False)])
def test_front_against_oracle(G, hd, d, F, B, front):
    """Prompts of 1 to 70 tokens, so that the contexts cross 16-token pages and the passes of 32 and 64 keys; a row of the batch
    gives the same bits alone; an early end of sequence parks a row.  `front`: what the shape takes."""
    shape, Gen = _shape(G, hd, d, F), 11
    w = synth.make_weights(shape, 1, DEV)
    ro = R.Rollout(R.make_cfg(shape, B, 70 + Gen), R.Weights(w), DEV)
    rng = np.random.default_rng(3)
    plen = rng.integers(1, 71, size=B).astype(np.int32)
    plen[-1] = 58
    ids = rng.integers(0, shape.vocab, size=(B, 70)).astype(np.int32)
    side = torch.cuda.Stream()

    def generate(rows, eos=-1, base=0):
        out = torch.zeros(len(rows), Gen, dtype=torch.int32, device=DEV)
        lp = torch.zeros(len(rows), Gen, device=DEV)
        n = torch.zeros(len(rows), dtype=torch.int32, device=DEV)
        prompts = torch.tensor(ids[rows], device=DEV)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            ro.rollout_generate(R.sample_cfg(4, 0.7, eos, base), prompts, plen[rows], Gen, out, n, lp)
        torch.cuda.synchronize()
        ro.rollout_check()
        return out.cpu().numpy(), lp.cpu().numpy(), n.cpu().numpy()

    names = kernels_run(lambda: generate(list(range(B))))
    # K > 256 takes the product for few rows, as long as the context holds at most 8
    assert _ran(names) == (front, B <= 8 and (F > 256 or 2 * G * hd > 256)), sorted(names)
    out, lp, _ = generate(list(range(B)))
    m = O.Model(shape, synth.weights_for_oracle(w))
    verify_rollout(m, [ids[b, :plen[b]] for b in range(B)], out, lp, 0.7, 4, 0, 1e-5, 1e-4, rows=None if B < 16 else [0, 1, 63, B - 1])
    one, one_lp, _ = generate([B - 1], base=B - 1)
    assert np.array_equal(one[0], out[-1]) and np.array_equal(one_lp[0], lp[-1])
    eos = int(out[0, 4])
    ended, ended_lp, n = generate(list(range(B)), eos)
    for b in range(B):
        hit = np.flatnonzero(out[b] == eos)
        stop = int(hit[0]) + 1 if len(hit) else Gen
        assert n[b] == stop and np.array_equal(ended[b, :stop], out[b, :stop]) and np.array_equal(ended_lp[b, :stop], lp[b, :stop])
        assert (ended[b, stop:] == eos).all() and (ended_lp[b, stop:] == 0).all()
    ro.close()


@pytest.mark.parametrize("heads,hd", [(1, 64), (4, 128)], ids=["front", "separate"])
def test_steps_per_graph_and_the_ones_left_over(heads, hd):
    """Runs of 1 to 37 tokens on one context, captured (several steps a graph, a remainder of eager ones) and eager: the same
    tokens and log-probs; a run as long as max_seq allows."""
    shape, B, P, most = _shape(heads, hd, 128, 128), 3, 9, 37
    ro = R.Rollout(R.make_cfg(shape, B, P - 1 + most), R.Weights(synth.make_weights(shape, 1, DEV)), DEV)
    ids, lens = synth.make_prompts(shape.vocab, B, P, P, 3)
    prompts, side, want = torch.tensor(ids, device=DEV), torch.cuda.Stream(), None
    for stream, G in [(torch.cuda.default_stream(), most)] + [(side, g) for g in (1, 4, 7, 8, 15, 33, most, most)]:
        out = torch.zeros(B, G, dtype=torch.int32, device=DEV)
        lp = torch.zeros(B, G, device=DEV)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ro.rollout_generate(R.sample_cfg(4, 0.7), prompts, lens, G, out, None, lp)
        torch.cuda.synchronize()
        ro.rollout_check()
        got = out.cpu().numpy(), lp.cpu().numpy()
        want = want or got
        assert np.array_equal(got[0], want[0][:, :G]) and np.array_equal(got[1], want[1][:, :G]), G
    ro.close()
