"""Channel-wise groups that one workgroup's registers hold: codes, scale bits and minimum bits against the oracle,
bit for bit."""
import numpy as np
import pytest

import helpers as H
from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

pytestmark = pytest.mark.gpu


# groups that one workgroup's registers hold: the sizes at which the kernel changes, one token either side, a number of
# groups that is not a multiple of eight, both tensors or one
@pytest.mark.parametrize("d,bits", [(64, 1), (128, 1), (128, 2), (256, 2), (128, 4), (64, 8)])
@pytest.mark.parametrize("group", [129, 512, 513, 1025, 1537, 2049, 3072, 3073, 4096, 4097])
def test_groups_held_in_registers(d, bits, group):
    for rows, both in ((3, True), (1, False)):
        w = synth.WORKLOADS[3].replace(batch=1, n_kv_heads=rows, n_q_heads=rows, head_dim=d, n_vis=group, n_text=0, seed=group + d)
        x = synth.make_inputs(w, "cpu", parts=("k", "v"))
        x["k"][0, 0, :, 5] = x["k"][0, 0, 0, 5]                  # a constant channel
        lay = cq.make_layout(1, rows, rows, d, group, bits, 0, 0 if both else 1, group, group if both else d)
        got = cq.cq_quantize_kv(lay, x["k"].cuda(), x["v"].cuda())
        for t, name, axis, size in ((got[0], "k", 0, group), (got[1], "v", lay.v_axis, lay.v_group)):
            ref = O.quantize_tensor(x[name].numpy(), bits, axis, size)
            assert np.array_equal(H.words_of(t.codes), ref["words"]), (name, rows)
            assert np.array_equal(t.scale.cpu().numpy().view(np.uint32), ref["scale"].view(np.uint32)), (name, rows)
            assert np.array_equal(t.min.cpu().numpy().view(np.uint16), ref["min"].view(np.uint16)), (name, rows)
