"""The tau grid over rows cut into several chunks, whose sums meet in the last kernel, and over rows of one chunk, whose
block finishes them; the scratch of both is what it was when the normalizers were a pass of their own."""
import numpy as np
import pytest
import torch

from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

import helpers as H

# batch, query heads, tokens, tail: one row of many chunks with a ragged last one; rows of two chunks; one chunk, because
# there are many rows, because there are few tokens
CASES = [(1, 1, 9000, 1), (20, 8, 600, 39), (65, 16, 300, 7), (1, 2, 130, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("batch,heads,n_vis,n_text", CASES)
@pytest.mark.parametrize("grid1,grid2", [((0.0, 1.0, 2.0, 3.0), (0.0, 1.0, 2.0, 3.0)), ((0.0, 0.5, 3.0, 1.0, 2.0), (0.25,)),
                                         ((60.0, 0.0), (1.0, 0.0))])
def test_chunks(batch, heads, n_vis, n_text, grid1, grid2):
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


@pytest.mark.parametrize("args,n_text,pairs,size", [
    ((1, 1, 1, 128, 9000, 2, 0, 0, 9000, 9000), 1, (4, 4), 83456),
    ((20, 8, 2, 128, 600, 2, 0, 0, 600, 600), 39, (8, 8), 1534208),
    ((65, 16, 4, 128, 300, 2, 0, 0, 300, 300), 7, (1, 1), 4147712)])
def test_scratch(args, n_text, pairs, size):
    assert cq.cq_tau_search_workspace_bytes(cq.make_layout(*args), n_text, *pairs) == size
