"""The tau grid over rows cut into several chunks, whose sums meet in the last kernel, and over rows of one chunk, whose
block finishes them; the scratch of both is what it was when the normalizers were a pass of their own."""
import numpy as np
import pytest
import torch

from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

import helpers as H


def chunks_of(rows, tokens, pairs):
    """Chunks of a query row, by the rule of tau_workspace_layout: as many as their sums (three per pair and two) and a ratio
    per pair fit the scratch of about 1024 blocks of whole rounds of 256 tokens, with 2 pairs + 1 sums each."""
    up = lambda a, b: -(-a // b)
    rounds, want = up(tokens, 256), up(1024, rows)
    shares = up(rounds, up(rounds, want))
    fit = (shares * (2 * pairs + 1) - pairs) // (3 * pairs + 2)
    return up(rounds, up(rounds, fit)) if fit > 1 else 1


# batch, query heads, tokens, tail, chunks: one row of many chunks with a ragged last one; many rows of four and of two chunks;
# one chunk, because four shares of scratch would be needed for two, because there are many rows, because there are few tokens
CASES = [(1, 1, 9000, 1, 18), (16, 8, 1700, 39, 4), (40, 8, 1000, 20, 2), (20, 8, 600, 39, 1), (65, 16, 300, 7, 1), (1, 2, 130, 0, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,n_vis,n_text,chunks", CASES)
@pytest.mark.parametrize("grid1,grid2", [((0.0, 1.0, 2.0, 3.0), (0.0, 1.0, 2.0, 3.0)), ((0.0, 0.5, 3.0, 1.0, 2.0), (0.25,)),
                                         ((60.0, 0.0), (1.0, 0.0))])
def test_chunks(batch, heads, n_vis, n_text, chunks, grid1, grid2):
    assert chunks_of(batch * heads, n_vis + n_text, len(grid1) * len(grid2)) == chunks
    n_kv = max(1, heads // 4)
    w = synth.WORKLOADS[1].replace(batch=batch, n_kv_heads=n_kv, n_q_heads=heads, n_vis=n_vis, n_text=n_text, seed=n_vis)
    lay = cq.make_layout(batch, heads, n_kv, 128, n_vis, 2, 0, 0, n_vis, n_vis)
    x_cpu = synth.make_inputs(w, "cpu")
    kq = O.quantize_tensor(x_cpu["k"].numpy(), 2, 0, n_vis)
    want = O.tau_grid_mse(x_cpu["q"].numpy(), x_cpu["k"].numpy(), kq, x_cpu["k_text"].numpy() if n_text else None, n_text,
                          grid1, grid2, 0.0)
    x = H.to_device(x_cpu)
    k_dev, _ = cq.cq_quantize_kv(lay, x["k"], x["v"])
    got = cq.cq_tau_search(lay, x["q"], x["k"], k_dev, x["k_text"] if n_text else None, n_text, grid1, grid2).cpu().numpy()
    # fp32 logits (about 1e-6 of the largest each), everything after them in fp64
    assert np.isfinite(got).all() and (np.abs(got - want) <= 1e-4 * np.abs(want)).all(), (got, want)


def grid_of_logits(lq, lx, n_vis, grid1, grid2):
    """The grid from the logits (quantized visual and text; exact visual) in 80 bits, and a bound of its error in 64 bits.

    A weight is off by the rounding of its exponent, some steps of the largest (A), and of a few exponentials and products (40
    steps cover both): relative to the difference of the two softmaxes that is 1 / delta times as much, twice for its
    square and once more for each normalizer.  The sum of d^2 (see calib_search.hip) is off by a step for each of the
    tokens that a thread adds up and for each level above, and what is subtracted from it is known no better."""
    eps, n_all = 2.0 ** -53, lq.shape[1]
    lq, lx = lq.astype(np.longdouble), np.concatenate([lx, lq[:, n_vis:]], 1).astype(np.longdouble)
    s, lo, hi = lq[:, :n_vis], lq[:, :n_vis].min(1, keepdims=True), lq[:, :n_vis].max(1, keepdims=True)
    u = (s - lo) / (hi - lo)
    ref = np.exp(lx - lx.max(1, keepdims=True))
    q = ref / ref.sum(1, keepdims=True)
    value, bound = np.zeros((len(grid1), len(grid2))), np.zeros((len(grid1), len(grid2)))
    for i, t1 in enumerate(grid1):
        for j, t2 in enumerate(grid2):
            g = np.concatenate([s + t1 * (u - 1) - t2 * u, lq[:, n_vis:]], 1)
            w = np.exp(g - g.max(1, keepdims=True))
            p = w / w.sum(1, keepdims=True)
            square = ((p - q) ** 2).sum(1)
            delta = np.sqrt(square / np.maximum((p ** 2).sum(1), (q ** 2).sum(1)))
            largest = max(float(np.ptp(lq)), float(np.ptp(lx))) + abs(t1) + abs(t2)
            summed = ((w - ref) ** 2).sum(1) / w.sum(1) ** 2
            off = 8 * eps * (largest + 40) / delta * square + 4 * eps * (n_all / 256 + 20) * summed
            value[i, j], bound[i, j] = float(square.mean() / n_all), float(off.mean() / n_all)
    return value, bound


# near weights (8 bits), weights that are nearly flat, weights of which a few tokens hold all; several chunks and one
@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,n_vis,n_text,bits,scale", [(1, 4, 9000, 3, 8, 0.0), (2, 8, 3000, 40, 2, 0.001),
                                                                 (2, 8, 3000, 40, 2, 0.5), (64, 16, 300, 7, 2, 0.5),
                                                                 (64, 16, 300, 7, 8, 0.0)])
@pytest.mark.parametrize("grid1,grid2", [((0.0, 1.0, 2.0, 3.0), (0.0, 1.0, 2.0, 3.0)), ((0.0, 0.5, 3.0, 1.0, 2.0), (0.25,)),
                                         ((60.0, 0.0), (1.0, 0.0))])
def test_everything_behind_the_logits(batch, heads, n_vis, n_text, bits, scale, grid1, grid2):
    """The search against its own fp32 logits, which its scratch begins with: first those of the quantized and text
    keys, then, from the next 64 floats on, those of the exact keys."""
    n_kv = heads // 4
    w = synth.WORKLOADS[1].replace(batch=batch, n_kv_heads=n_kv, n_q_heads=heads, n_vis=n_vis, n_text=n_text, seed=n_vis + bits)
    lay = cq.make_layout(batch, heads, n_kv, 128, n_vis, bits, 0, 0, n_vis, n_vis)
    x = H.to_device(synth.make_inputs(w, "cpu"))
    k_dev, _ = cq.cq_quantize_kv(lay, x["k"], x["v"])
    ws = torch.empty(cq.cq_tau_search_workspace_bytes(lay, n_text, len(grid1), len(grid2)), dtype=torch.uint8, device="cuda")
    got = cq.cq_tau_search(lay, x["q"], x["k"], k_dev, x["k_text"], n_text, grid1, grid2, scale, workspace=ws).cpu().numpy()
    rows, n_all = batch * heads, n_vis + n_text
    at = (rows * n_all + 63) // 64 * 64
    floats = ws.view(torch.float32).cpu().numpy()
    want, bound = grid_of_logits(floats[:rows * n_all].reshape(rows, n_all), floats[at:at + rows * n_vis].reshape(rows, n_vis),
                                 n_vis, grid1, grid2)
    assert (bound <= 1e-9 * want).all(), (bound, want)
    assert (np.abs(got - want) <= bound).all(), (np.abs(got - want) / bound, np.abs(got - want) / want)


@pytest.mark.parametrize("args,n_text,pairs,size", [
    ((1, 1, 1, 128, 9000, 2, 0, 0, 9000, 9000), 1, (4, 4), 83456),
    ((20, 8, 2, 128, 600, 2, 0, 0, 600, 600), 39, (8, 8), 1534208),
    ((65, 16, 4, 128, 300, 2, 0, 0, 300, 300), 7, (1, 1), 4147712)])
def test_scratch(args, n_text, pairs, size):
    assert cq.cq_tau_search_workspace_bytes(cq.make_layout(*args), n_text, *pairs) == size
