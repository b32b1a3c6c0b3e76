"""The tau grid away from 4 x 4: grids that are no multiple of the kernel's block of pairs, taus on both
sides of the limit up to which a weight is formed as a product of factors, ragged token counts."""
import numpy as np
import pytest
import torch

from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n_vis,n_text", [(128, 1003, 300), (64, 255, 0), (256, 192, 5)])
@pytest.mark.parametrize("grid1,grid2", [((0.0, 1.0, 2.0, 3.0, 4.5), (0.0, 0.5, 1.0)),
                                         ((50.0, 0.0), (-50.0, 1.0)), ((50.5, 0.0), (700.0, 1.0))])
def test_grids(d, n_vis, n_text, grid1, grid2):
    w = synth.WORKLOADS[1].replace(batch=2, n_kv_heads=2, n_q_heads=10, head_dim=d, n_vis=n_vis,
                                   n_text=n_text, seed=d)
    lay = cq.make_layout(2, 10, 2, d, n_vis, 2, 0, 0, n_vis, n_vis)
    x_cpu = synth.make_inputs(w, "cpu")
    kq = O.quantize_tensor(x_cpu["k"].numpy(), 2, 0, n_vis)
    want = O.tau_grid_mse(x_cpu["q"].numpy(), x_cpu["k"].numpy(), kq,
                          x_cpu["k_text"].numpy() if n_text else None, n_text, grid1, grid2, 0.0)
    x = H.to_device(x_cpu)
    k_dev, _ = cq.cq_quantize_kv(lay, x["k"], x["v"])
    got = cq.cq_tau_search(lay, x["q"], x["k"], k_dev, x["k_text"] if n_text else None, n_text, grid1, grid2)
    got = got.cpu().numpy()
    # fp32 logits (about 1e-6 of the largest each), everything after them in fp64
    assert np.abs(got - want).max() <= 1e-4 * np.abs(want).max() and np.isfinite(got).all(), (got, want)
    assert (np.abs(got - want) <= 1e-4 * np.abs(want)).all(), (got, want)
