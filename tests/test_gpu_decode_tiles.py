"""Decode attention on the tile kernels (head dimensions 64 and 256, token counts and groups of any
size, wide codes with channel-wise values) against the fp64 oracle, at the sizes where blocks, tiles,
head sets and chunks end."""
import numpy as np
import pytest
import torch

from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

import helpers as H

pytestmark = pytest.mark.gpu

# (n_vis, k_group, v_axis, v_group (0: head_dim), q heads of 1 KV head, n_text, calibration)
# whole sequences one token over a block, one under two, long and ragged; groups of 64 in a row that is
# not a multiple of 64 per wave; a group no block or tile size divides; 4, 5 and 9 heads (head sets);
# tails of 0, 1, a block and more; text only; a falling calibration line
CASES = [(129, 129, 0, 129, 4, 1, "dynamic"), (255, 255, 1, 0, 1, 0, "none"),
         (3003, 3003, 0, 3003, 5, 77, "dynamic"), (2112, 64, 0, 64, 4, 256, "dynamic"),
         (1000, 40, 0, 200, 9, 257, "fixed"), (4160, 32, 1, 0, 3, 600, "dynamic"),
         (0, 32, 1, 0, 4, 300, "none"), (17, 17, 0, 17, 2, 3, "falling")]
MODES = {"none": (cq.CQ_CALIB_NONE, 0, 0, 0, 0), "dynamic": (cq.CQ_CALIB_DYNAMIC, 1, 2, 0, 0),
         "fixed": (cq.CQ_CALIB_FIXED, 3, 1, -9, 9), "falling": (cq.CQ_CALIB_FIXED, 0, 3, -1, 1)}


@pytest.fixture
def tile_path():
    """The tile kernels or an error: no other kernels can stand in for them unseen."""
    prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_TILE)
    yield
    cq.cq_bench_set_kernel_path(prev)


def _auto_takes_the_tiles(lay, n_text, calib):
    """Without the switch the tile kernels run as well, unless the tuned ones take the layout."""
    sizes = {}
    for path in (cq.CQ_PATH_TUNED, cq.CQ_PATH_AUTO, cq.CQ_PATH_TILE):
        prev = cq.cq_bench_set_kernel_path(path)
        sizes[path] = cq.cq_decode_workspace_bytes(lay, n_text, calib)
        cq.cq_bench_set_kernel_path(prev)
    return sizes[cq.CQ_PATH_TUNED] or sizes[cq.CQ_PATH_AUTO] == sizes[cq.CQ_PATH_TILE]


def _check(out, ref, what):
    got = out.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all(), what
    err = O.rel_l2(got, ref)
    assert err <= H.REGRESSION_TOL, "%s: rel L2 %.3e" % (what, err)
    H.assert_elementwise_close(got, ref, what)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_tile_decode(d, bits, tile_path):
    for n_vis, kg, vax, vg, g, n_text, calib in CASES:
        vg = vg or d
        what = "d %d bits %d n_vis %d kg %d v %d/%d g %d n_text %d %s" % (d, bits, n_vis, kg, vax, vg, g, n_text, calib)
        print(what, flush=True)
        w = synth.WORKLOADS[2].replace(batch=2, n_kv_heads=2, n_q_heads=2 * g, head_dim=d, n_vis=n_vis,
                                       n_text=n_text + 2, seed=n_vis + d + bits)
        x_cpu = synth.make_inputs(w, "cpu")
        lay = cq.make_layout(2, 2 * g, 2, d, n_vis, bits, 0, vax, kg, vg)
        x = H.to_device(x_cpu)
        kq, vq = H.oracle_quantize(x_cpu, lay)
        kd, vd = cq.cq_quantize_kv(lay, x["k"], x["v"]) if n_vis else (None, None)
        args = MODES[calib]
        assert _auto_takes_the_tiles(lay, n_text, cq.make_calib(*args)), what
        ref = O.decode_attn(x_cpu["q"].numpy(), kq, vq, x_cpu["k_text"].numpy(), x_cpu["v_text"].numpy(),
                            n_text, *args, 0.0)
        out = cq.cq_decode_attn(lay, x["q"], kd, vd, x["k_text"], x["v_text"], n_text, cq.make_calib(*args))
        torch.cuda.synchronize()
        _check(out, ref, what)
        # the tail length on the device, its bound two tokens longer
        n_dev = torch.tensor([n_text], dtype=torch.int32, device="cuda")
        out = cq.cq_decode_attn_devlen(lay, x["q"], kd, vd, x["k_text"], x["v_text"], n_dev, n_text + 2,
                                       cq.make_calib(*args))
        torch.cuda.synchronize()
        _check(out, ref, what + " length on the device")


@pytest.mark.parametrize("d,n_vis,batch", [(64, 640, 2), (128, 4224, 1)])
def test_recorded_step_on_the_tile_kernels(d, n_vis, batch):
    """A growing step (append, attend) recorded once and replayed with eager work and synchronizations
    in between: the count by which the last workgroup of a row is found starts over in every replay.
    (128, 4224 tokens, 2 rows: a layout of the fused kernel that the tile kernels finish sooner.)"""
    w = synth.WORKLOADS[1].replace(batch=batch, n_kv_heads=2, n_q_heads=8, head_dim=d, n_vis=n_vis, n_text=126,
                                   seed=d)
    lay = cq.make_layout(batch, 8, 2, d, n_vis, 1, 0, 1, 64, d)
    x_cpu = synth.make_inputs(w, "cpu")
    x = H.to_device(x_cpu)
    kq, vq = H.oracle_quantize(x_cpu, lay)
    kd, vd = cq.cq_quantize_kv(lay, x["k"], x["v"])
    first, cap = 123, 126
    tails = [x[t].clone() for t in ("k_text", "v_text")]
    length = torch.tensor([first], dtype=torch.int32, device="cuda")
    new = [torch.zeros(batch, 2, 1, d, dtype=torch.float16, device="cuda") for _ in range(2)]
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1, 2)
    ws = torch.empty(cq.cq_decode_workspace_bytes(lay, cap, calib), dtype=torch.uint8, device="cuda")
    assert ws.numel() > 256                             # logits in scratch: not the one-launch kernel
    out = torch.zeros_like(x["q"])

    def step():
        cq.cq_append_text_kv_devlen(lay, *tails, length, *new)
        cq.cq_decode_attn_devlen(lay, x["q"], kd, vd, *tails, length, cap, calib, out=out, workspace=ws)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    length.fill_(first)
    for i in range(3):
        at = first + i
        for t, n in zip(("k_text", "v_text"), new):
            n.copy_(x[t][:, :, at:at + 1])
        out.zero_()
        ws.fill_(255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(length) == at + 1
        ref = O.decode_attn(x_cpu["q"].numpy(), kq, vq, x_cpu["k_text"].numpy(), x_cpu["v_text"].numpy(), at + 1,
                            O.CALIB_DYNAMIC, 1.0, 2.0)
        _check(out, ref, "d %d replay %d" % (d, i))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_values_that_stand_out(d, bits, tile_path):
    """One group of tokens holds values 3e6 times the others' and, for the first query head, weights of 2e-8
    of theirs: both parts count alike in that head's result, and each has to keep fp32's bits.  The
    heads differ in scale, down to one whose weights are all equal (where the outliers are everything), so
    no fixed-point format that the heads share can hold them.  The bar is what rounding the exact
    result to fp16 gives for that head, plus 1e-4: weights are within 17.5 x 2^-22 = 4e-6 (fp32 logits), sums
    of 1000 terms in fp32 within 1e-5."""
    n, group, n_text = 1000, 40, 3
    gen = torch.Generator().manual_seed(d + bits)
    q0 = torch.randn(d, generator=gen)
    q = torch.stack([q0, 0.5 * q0, 0.1 * q0, 0.0 * q0]).half().view(1, 4, d)
    k = 0.05 * torch.randn(1, 1, n, d, generator=gen)
    v = 0.01 * torch.randn(1, 1, n, d, generator=gen)
    out = slice(5 * group, 6 * group)
    k[:, :, out] = -17.5 * d ** 0.5 * q0 / q0.square().sum()
    v[:, :, out] = 30000.0 * torch.randn(1, 1, group, d, generator=gen).clamp(-2, 2)
    kt, vt = 0.05 * torch.randn(1, 1, n_text, d, generator=gen), 0.01 * torch.randn(1, 1, n_text, d, generator=gen)
    x_cpu = {"q": q, "k": k.half(), "v": v.half(), "k_text": kt.half(), "v_text": vt.half()}
    x = H.to_device(x_cpu)
    for vax, vg in ((1, d), (0, group), (0, n)):
        what = "d %d bits %d values %d/%d" % (d, bits, vax, vg)
        print(what, flush=True)
        lay = cq.make_layout(1, 4, 1, d, n, bits, 0, vax, group, vg)
        kq, vq = H.oracle_quantize(x_cpu, lay)
        kd, vd = cq.cq_quantize_kv(lay, x["k"], x["v"])
        ref = O.decode_attn(x_cpu["q"].numpy(), kq, vq, x_cpu["k_text"].numpy(), x_cpu["v_text"].numpy(), n_text,
                            O.CALIB_NONE)
        got = cq.cq_decode_attn(lay, x["q"], kd, vd, x["k_text"], x["v_text"], n_text).cpu().numpy()
        for h in range(4):
            err, least = H.row_rel_l2(got[:, h], ref[:, h]), H.row_rel_l2(ref[:, h].astype(np.float16), ref[:, h])
            assert err <= least + 1e-4, "%s head %d: rel L2 %.3e, fp16 rounding %.3e" % (what, h, err, least)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("level", [150.0, -150.0])
def test_an_empty_tail_of_a_length_on_the_device(d, level, tile_path):
    """No token of the tail yet, its bound larger: the partials of the tail's workgroups are empty, and the merge
    takes its reference from the others.  Logits around 150 and -150, where exp() without a reference leaves
    fp32's range; rows of one and of several chunks."""
    for n_vis, bound in ((512, 1), (2048, 300)):
        gen = torch.Generator().manual_seed(d + n_vis)
        k = 0.5 + 0.1 * torch.randn(1, 2, n_vis, d, generator=gen)
        x_cpu = {"q": (2 * level / d ** 0.5 + torch.randn(1, 4, d, generator=gen)).half(), "k": k.half(),
                 "v": torch.randn(1, 2, n_vis, d, generator=gen).half(),
                 "k_text": torch.zeros(1, 2, bound, d).half(), "v_text": torch.zeros(1, 2, bound, d).half()}
        lay = cq.make_layout(1, 4, 2, d, n_vis, 2, 0, 1, 128, d)
        x = H.to_device(x_cpu)
        kq, vq = H.oracle_quantize(x_cpu, lay)
        kd, vd = cq.cq_quantize_kv(lay, x["k"], x["v"])
        n_dev = torch.zeros(1, dtype=torch.int32, device="cuda")
        for mode in ("none", "dynamic"):
            ref = O.decode_attn(x_cpu["q"].numpy(), kq, vq, None, None, 0, *MODES[mode], 0.0)
            out = cq.cq_decode_attn_devlen(lay, x["q"], kd, vd, x["k_text"], x["v_text"], n_dev, bound,
                                           cq.make_calib(*MODES[mode]))
            torch.cuda.synchronize()
            _check(out, ref, "d %d n_vis %d level %g %s" % (d, n_vis, level, mode))


@pytest.mark.parametrize("d,bits,vax", [(64, 1, 1), (128, 2, 0), (256, 1, 1)])
def test_many_partials(d, bits, vax, tile_path):
    """One row of 32768 tokens is 64 chunks, a tail of 8193 another 33 of 256 tokens (64 of 128 are 8192): the
    last workgroup merges 97 partials in seven batches, and a tail workgroup takes two rounds."""
    n, n_text = 32768, 8193
    w = synth.WORKLOADS[2].replace(batch=1, n_kv_heads=1, n_q_heads=3, head_dim=d, n_vis=n, n_text=n_text, seed=d)
    x_cpu = synth.make_inputs(w, "cpu")
    lay = cq.make_layout(1, 3, 1, d, n, bits, 0, vax, 512, d if vax else 512)
    x = H.to_device(x_cpu)
    kq, vq = H.oracle_quantize(x_cpu, lay)
    kd, vd = cq.cq_quantize_kv(lay, x["k"], x["v"])
    for t in (n_text, 8192, 130):
        ref = O.decode_attn(x_cpu["q"].numpy(), kq, vq, x_cpu["k_text"].numpy(), x_cpu["v_text"].numpy(), t,
                            O.CALIB_DYNAMIC, 1.0, 2.0)
        out = cq.cq_decode_attn(lay, x["q"], kd, vd, x["k_text"], x["v_text"], t, cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1, 2))
        torch.cuda.synchronize()
        _check(out, ref, "d %d bits %d tail %d" % (d, bits, t))


@pytest.mark.parametrize("d,bits,vax", [(64, 1, 0), (128, 8, 1)])
def test_long_runs(d, bits, vax, tile_path):
    """A row of 16.8 million tokens: 1025 value tiles per wave, one more than the int32 digit sums hold, and
    code words beyond 2^31 bytes (128 channels, 8 bits).  With a query of zeros all weights are equal, so the
    result is the mean of the dequantized values, 0.5 on average: formed here in fp64.  fp32 sums of equal
    terms, banked every 1024 tiles, stay far below fp16's rounding."""
    n = 64 * 4 * 64 * 1025
    gen = torch.Generator("cuda").manual_seed(d)
    x = torch.empty(1, 1, n, d, dtype=torch.float16, device="cuda").uniform_(0, 1, generator=gen)
    lay = cq.make_layout(1, 1, 1, d, n, bits, 0, vax, 512, d if vax else n)
    k, v = cq.cq_quantize_kv(lay, x, x)
    q = torch.zeros(1, 1, d, dtype=torch.float16, device="cuda")
    out = cq.cq_decode_attn(lay, q, k, v, None, None, 0)
    torch.cuda.synchronize()
    del x
    total, step = torch.zeros(d, dtype=torch.float64, device="cuda"), n // 64
    shifts = torch.arange(32 - bits, -1, -bits, device="cuda", dtype=torch.int32)
    for t in range(0, n, step):
        words = v.codes[0, 0, t:t + step]
        codes = ((words[:, :, None] >> shifts) & ((1 << bits) - 1)).view(step, d).double()
        if vax:
            total += (codes * v.scale[0, 0, t:t + step].double() + v.min[0, 0, t:t + step].double()).sum(0)
        else:
            total += (codes * v.scale[0, 0].double() + v.min[0, 0].double()).sum(0)
    ref = (total / n).cpu().numpy().reshape(1, 1, d)
    _check(out, ref, "d %d bits %d" % (d, bits))
    del k, v
    torch.cuda.empty_cache()
