"""The tile kernel's order of tiles around whole spans of 64: codes, scale bits and minimum bits against the oracle's C++
twin, bit for bit.  (One tensor: its tiles go out in a launch of their own.)"""
import numpy as np
import pytest

import helpers as H
from oracle import cq_oracle_native as N
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

pytestmark = pytest.mark.gpu


# 128 and 256 channels are renumbered, values of 128 channels and 2 bits also by the kernel that knows that every tile is full; 64
# channels and 8 bits keep their order.  The last one's key groups are short tiles of their own.
@pytest.mark.parametrize("tiles", [1, 63, 64, 65, 128, 191])
@pytest.mark.parametrize("d,bits,group,rest", [(128, 1, 128, 0), (128, 2, 32, 32), (128, 2, 128, 0), (128, 4, 64, 64), (256, 1, 64, 64),
                                               (256, 2, 128, 0), (64, 4, 64, 64), (256, 8, 128, 0), (128, 2, 100, 0)])
def test_runs(tiles, d, bits, group, rest):
    n = tiles * (128 if 128 % group == 0 else group) + rest
    w = synth.WORKLOADS[3].replace(batch=1, n_kv_heads=1, n_q_heads=1, head_dim=d, n_vis=n, n_text=0, seed=n + d)
    x = synth.make_inputs(w, "cpu", parts=("k", "v"))
    lay = cq.make_layout(1, 1, 1, d, n, bits, 0, 1, group, d)
    dev = {t: x[t].cuda() for t in x}
    for name, got, axis, size in (("k", cq.cq_quantize_kv(lay, dev["k"], None)[0], 0, group),
                                  ("v", cq.cq_quantize_kv(lay, None, dev["v"])[1], 1, d)):
        ref = N.quantize_tensor(x[name].numpy(), bits, axis, size)
        assert np.array_equal(H.words_of(got.codes), ref["words"]), name
        assert np.array_equal(got.scale.cpu().numpy().view(np.uint32), ref["scale"].view(np.uint32)), name
        assert np.array_equal(got.min.cpu().numpy().view(np.uint16), ref["min"].view(np.uint16)), name
