"""The tile quantizer away from round sizes: head dimensions 64 and 256, token counts that leave a
short tile, groups of any size.  Codes, scale bits and minimum bits against the oracle, bit for bit."""
import pytest
import torch

from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth
import helpers as H

pytestmark = pytest.mark.gpu

# (axis, group, n_vis): a last tile of 32 tokens; long groups one token over a tile, just under two
# tiles, and a multiple of neither; two long groups per row; groups that are one short tile each;
# a last tile of 1 and of 127 tokens
SIZES = [(0, 32, 160), (0, 64, 192), (0, 129, 129), (0, 255, 510), (0, 1003, 1003), (0, 7, 21),
         (0, 127, 127), (1, 32, 129), (1, 64, 255)]


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_short_tiles_and_any_group(d, bits):
    prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_TUNED)      # no fallback to the shape-agnostic kernels
    try:
        for axis, group, n_vis in SIZES + [(1, d, 257)]:
            what = "d %d bits %d axis %d group %d n_vis %d" % (d, bits, axis, group, n_vis)
            print(what, flush=True)
            w = synth.WORKLOADS[4].replace(batch=3, n_kv_heads=1, n_q_heads=1, head_dim=d, n_vis=n_vis,
                                           seed=n_vis + d)
            k = synth.make_inputs(w, "cpu", parts=("k",))["k"]
            k[0, 0, :, 1] = 0.25                               # a constant channel
            k[1, 0, n_vis - 1, 2] = -900.0                     # an extremum in the last token
            k[2, 0, 0, d - 1] = 900.0                          # and in the first
            lay = cq.make_layout(3, 1, 1, d, n_vis, bits, axis, axis, group, group)
            got, _ = cq.cq_quantize_kv(lay, k.cuda(), None)
            torch.cuda.synchronize()
            H.assert_qtensor_equal(got, O.quantize_tensor(k.numpy(), bits, axis, group), what)
    finally:
        cq.cq_bench_set_kernel_path(prev)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits", [1, 8])
def test_keys_and_values_in_one_call(d, bits):
    """Every pair of key and value statistics that one launch takes, and two that it does not, on
    keys and values that differ; a row of 384 tokens is three tiles of each."""
    prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_TUNED)
    try:
        w = synth.WORKLOADS[3].replace(batch=2, n_kv_heads=1, n_q_heads=1, head_dim=d, n_vis=384, seed=d)
        x_cpu = synth.make_inputs(w, "cpu", parts=("k", "v"))
        x = H.to_device(x_cpu)
        for kg in (32, 64, 128, 384, 192):
            for vax, vg in ((1, d), (0, 32), (0, 64), (0, 128), (0, 384), (0, 96)):
                lay = cq.make_layout(2, 1, 1, d, 384, bits, 0, vax, kg, vg)
                k, v = cq.cq_quantize_kv(lay, x["k"], x["v"])
                torch.cuda.synchronize()
                what = "d %d bits %d keys %d values %d/%d" % (d, bits, kg, vax, vg)
                H.assert_qtensor_equal(k, O.quantize_tensor(x_cpu["k"].numpy(), bits, 0, kg), what)
                H.assert_qtensor_equal(v, O.quantize_tensor(x_cpu["v"].numpy(), bits, vax, vg), what)
    finally:
        cq.cq_bench_set_kernel_path(prev)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_both_sides_of_the_shortest_group(d, bits):
    """Channel-wise groups around the length from which the tile kernels are used, keys on one side of it
    and values on the other: bit for bit the same as the oracle, and as the tile kernels wherever
    they can run."""
    n = 16 * 27 * 7
    w = synth.WORKLOADS[4].replace(batch=1, n_kv_heads=2, n_q_heads=2, head_dim=d, n_vis=n, seed=d + bits)
    x_cpu = synth.make_inputs(w, "cpu", parts=("k", "v"))
    x = H.to_device(x_cpu)
    for kg, vg in ((1, 28), (12, 18), (16, 27), (14, 24), (21, 9), (28, 36)):
        lay = cq.make_layout(1, 2, 2, d, n, bits, 0, 0, kg, vg)
        want = [O.quantize_tensor(x_cpu[t].numpy(), bits, 0, g) for t, g in (("k", kg), ("v", vg))]
        for path in (cq.CQ_PATH_AUTO, cq.CQ_PATH_TUNED):
            prev = cq.cq_bench_set_kernel_path(path)
            try:
                got = cq.cq_quantize_kv(lay, x["k"], x["v"])
                torch.cuda.synchronize()
            finally:
                cq.cq_bench_set_kernel_path(prev)
            for g, r, name in zip(got, want, "kv"):
                H.assert_qtensor_equal(g, r, "d %d bits %d groups %d/%d %s path %d" % (d, bits, kg, vg, name, path))


@pytest.mark.parametrize("d", [64, 256])
def test_more_groups_than_blocks_in_a_launch(d):
    """2^24 + 5 groups of one token: more blocks of 256 threads than a launch takes (2^32 - 1 threads), so
    the tile kernels leave them to the others, which take one thread per channel: one launch, or two.  A
    group of one token is its own minimum."""
    n = (1 << 24) + 5
    lay = cq.make_layout(1, 1, 1, d, n, 1, 0, 0, 1, 1)
    x = torch.randn(n, d, device="cuda", dtype=torch.float16, generator=torch.Generator("cuda").manual_seed(1))
    out, _ = cq.cq_quantize_kv(lay, x.view(1, 1, n, d), None)
    torch.cuda.synchronize()
    x.add_(0.0)                                        # a zero minimum is stored as +0
    assert torch.equal(out.min.view(n, d), x)
    for t in (out.codes, out.scale):
        assert int(t.max()) == 0 and int(t.min()) == 0
    del x, out
    torch.cuda.empty_cache()
