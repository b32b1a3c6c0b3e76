"""More long groups than the chip has compute units: a workgroup takes its blocks in rounds and asks for the next one's
tokens while it forms codes.  Codes, scale bits and minimum bits against the oracle's C++ twin, bit for bit."""
import numpy as np
import pytest

import helpers as H
from oracle import cq_oracle_native as N
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

pytestmark = pytest.mark.gpu


# 264 to 792 blocks: a last round that few workgroups take, a number of groups that is not a multiple of eight, both
# tensors; the sizes at which the kernel changes, and a last piece of tokens that is nearly empty
@pytest.mark.parametrize("d,bits,rows,group", [(128, 1, 33, 2049), (128, 2, 65, 3072), (128, 2, 33, 3073), (128, 1, 67, 4096),
                                               (64, 2, 67, 2305), (64, 1, 131, 2200), (128, 2, 99, 2050)])
def test_rounds(d, bits, rows, group):
    w = synth.WORKLOADS[3].replace(batch=rows, n_kv_heads=1, n_q_heads=1, head_dim=d, n_vis=group, n_text=0, seed=group + d)
    x = synth.make_inputs(w, "cpu", parts=("k", "v"))
    x["k"][rows - 1, 0, :, 5] = x["k"][0, 0, 0, 5]                       # a constant channel
    lay = cq.make_layout(rows, 1, 1, d, group, bits, 0, 0, group, group)
    got = cq.cq_quantize_kv(lay, x["k"].cuda(), x["v"].cuda())
    for t, name in ((got[0], "k"), (got[1], "v")):
        ref = N.quantize_tensor(x[name].numpy(), bits, 0, group)
        assert np.array_equal(H.words_of(t.codes), ref["words"]), name
        assert np.array_equal(t.scale.cpu().numpy().view(np.uint32), ref["scale"].view(np.uint32)), name
        assert np.array_equal(t.min.cpu().numpy().view(np.uint16), ref["min"].view(np.uint16)), name
