"""cq_decode_attn_noalloc (the entry point for callers that cannot allocate) against cq_decode_attn:
same kernels, the library's own per-GPU scratch array instead of a caller's workspace, so the
outputs must agree bit for bit - on two calls in a row, the second with a smaller input (the
array keeps the first call's contents), on split rows (which use the scratch), on whole rows (which
do not) and on the shape-agnostic kernels."""
import numpy as np
import pytest
import torch

from oracle import cq_oracle as O
from paper_2502_14882_amd import binding as cq
from paper_2502_14882_amd import synth

import helpers as H

pytestmark = pytest.mark.gpu


def _inputs(w, lay):
    x_cpu = synth.make_inputs(w, "cpu")
    x = H.to_device(x_cpu)
    k_dev, v_dev = cq.cq_quantize_kv(lay, x["k"], x["v"])
    return x_cpu, x, k_dev, v_dev


def _both(w, lay, calib):
    x_cpu, x, k_dev, v_dev = _inputs(w, lay)
    kt = x["k_text"] if w.n_text > 0 else None
    vt = x["v_text"] if w.n_text > 0 else None
    want = cq.cq_decode_attn(lay, x["q"], k_dev, v_dev, kt, vt, w.n_text, calib)
    torch.cuda.synchronize()
    out = torch.full_like(x["q"], float("nan"))
    cq.cq_decode_attn_noalloc(lay, x["q"], k_dev, v_dev, kt, vt, w.n_text, calib, 0.0, out)
    torch.cuda.synchronize()
    assert torch.equal(out, want), "allocation-free and workspace entry points differ"
    kq, vq = H.oracle_quantize(x_cpu, lay)
    ref = H.oracle_decode(x_cpu, kq, vq, w.n_text, calib.mode, calib.tau1, calib.tau2)
    err = O.rel_l2(out.cpu().numpy().astype(np.float64), ref)
    assert err <= H.REL_L2_TOL, "rel L2 %.3e" % err


def test_two_calls_in_a_row_the_second_smaller():
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)
    # g = 6: two blocks of query heads per KV head, rows run as extrema pass + partial pass +
    # combine through the scratch (chunk extrema and online-softmax partials)
    big = synth.WORKLOADS[4].replace(batch=2, n_kv_heads=2, n_q_heads=12, n_vis=2560, n_text=130)
    small = synth.WORKLOADS[4].replace(batch=1, n_kv_heads=2, n_q_heads=12, n_vis=1280, n_text=70,
                                       seed=4321)
    for w in (big, small):
        lay = H.layout_of(w)
        assert cq.cq_decode_workspace_bytes(lay, w.n_text, calib) > 256, "this case must use scratch"
        _both(w, lay, calib)
    _both(small, H.layout_of(small), cq.make_calib(cq.CQ_CALIB_NONE))


def test_forced_chunks_whole_rows_and_generic_kernels(decode_chunks):
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)
    w = synth.WORKLOADS[1].replace(batch=2, n_kv_heads=2, n_q_heads=8, n_vis=1920, n_text=200)
    lay = H.layout_of(w)
    _both(w, lay, calib)                    # whole rows: the scratch is not touched
    decode_chunks(3)
    _both(w, lay, calib)                    # three chunks per row
    decode_chunks(0)
    prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_GENERIC)
    try:
        ws = cq.cq_decode_workspace_bytes(lay, w.n_text, calib)
        assert 256 < ws <= cq.CQ_NOALLOC_SCRATCH_BYTES
        _both(w, lay, calib)                # shape-agnostic kernels: logits live in the scratch
    finally:
        cq.cq_bench_set_kernel_path(prev)


def test_a_shape_beyond_the_scratch_is_refused():
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)
    w = synth.WORKLOADS[1].replace(batch=4, n_kv_heads=8, n_q_heads=32, head_dim=64, n_vis=16384, n_text=8)
    lay = H.layout_of(w, 1, 128, 64)
    x = synth.make_inputs(w, "cuda")
    k_dev, v_dev = cq.cq_quantize_kv(lay, x["k"], x["v"])
    with pytest.raises(cq.CqError) as e:
        cq.cq_decode_attn_noalloc(lay, x["q"], k_dev, v_dev, x["k_text"], x["v_text"], w.n_text, calib)
    assert e.value.status == cq.CQ_ERR_WORKSPACE


# (batch, q heads, KV heads, head_dim, n_vis, key group, value axis, value group, tails): layouts of the
# tile kernels whose scratch passes the size of the array inside the range of tails, while the
# shape-agnostic kernels would still fit it.  The last one does not fit it with either.
@pytest.mark.parametrize("shape,tails", [
    ((16, 32, 8, 64, 3328, 64, 1, 64), (158, 159, 160, 200, 239)),
    ((8, 32, 8, 128, 3003, 3003, 0, 3003), (2100, 2160, 2800, 3487)),
    ((48, 16, 4, 64, 1024, 64, 1, 64), (800, 1024)),
    ((64, 16, 16, 64, 1024, 1024, 0, 1024), (900, 1014))])
def test_the_same_kernels_on_both_sides_of_the_scratch_limit(shape, tails):
    B, nq, nkv, d, n, kg, vax, vg = shape
    w = synth.WORKLOADS[1].replace(batch=B, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, n_vis=n,
                                   n_text=max(tails), seed=n)
    x = synth.make_inputs(w, "cuda")
    lay = cq.make_layout(B, nq, nkv, d, n, 1, 0, vax, kg, vg)
    k, v = cq.cq_quantize_kv(lay, x["k"], x["v"])
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)

    def agnostic(n_text, size_only=False):
        prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_GENERIC)
        try:
            if size_only:
                return cq.cq_decode_workspace_bytes(lay, n_text, calib)
            return cq.cq_decode_attn(lay, x["q"], k, v, x["k_text"], x["v_text"], n_text, calib)
        finally:
            cq.cq_bench_set_kernel_path(prev)

    for n_text in tails:
        want = cq.cq_decode_attn(lay, x["q"], k, v, x["k_text"], x["v_text"], n_text, calib)
        try:
            got = cq.cq_decode_attn_noalloc(lay, x["q"], k, v, x["k_text"], x["v_text"], n_text, calib)
        except cq.CqError as e:
            assert e.status == cq.CQ_ERR_WORKSPACE
            assert agnostic(n_text, size_only=True) > cq.CQ_NOALLOC_SCRATCH_BYTES, (shape, n_text)
            continue
        torch.cuda.synchronize()
        assert torch.equal(got, want), (shape, n_text)
        err = O.rel_l2(got.cpu().numpy().astype(np.float64), agnostic(n_text).cpu().numpy().astype(np.float64))
        assert err <= 2 * H.REGRESSION_TOL, (shape, n_text, err)      # two fp16 results


@pytest.mark.parametrize("shape,n_text,path", [
    ((1, 32, 8, 128, 3328, 128, 1, 128), 100, cq.CQ_PATH_TUNED),       # one workgroup per row: 256 bytes
    ((1, 12, 2, 128, 2560, 128, 1, 128), 100, cq.CQ_PATH_TUNED),       # split rows: partials
    ((2, 8, 2, 64, 1000, 1000, 0, 1000), 300, cq.CQ_PATH_GENERIC)])    # the shape-agnostic kernels
def test_a_workspace_of_the_size_the_other_kernels_need_is_enough(shape, n_text, path):
    """A program that keeps the size its layout needs without the tile kernels is served by the kernels
    that need no more; a byte block less is refused."""
    B, nq, nkv, d, n, kg, vax, vg = shape
    w = synth.WORKLOADS[1].replace(batch=B, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, n_vis=n, n_text=n_text, seed=n)
    x = synth.make_inputs(w, "cuda")
    lay = cq.make_layout(B, nq, nkv, d, n, 1, 0, vax, kg, vg)
    k, v = cq.cq_quantize_kv(lay, x["k"], x["v"])
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)
    args = (lay, x["q"], k, v, x["k_text"], x["v_text"], n_text, calib)
    prev = cq.cq_bench_set_kernel_path(path)
    try:
        size = cq.cq_decode_workspace_bytes(lay, n_text, calib)
        want = cq.cq_decode_attn(*args)
    finally:
        cq.cq_bench_set_kernel_path(prev)
    assert 0 < size < cq.cq_decode_workspace_bytes(lay, n_text, calib)     # the tile kernels run, with more
    got = cq.cq_decode_attn(*args, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    n_dev = torch.tensor([n_text], dtype=torch.int32, device="cuda")
    dev = cq.cq_decode_attn_devlen(lay, x["q"], k, v, x["k_text"], x["v_text"], n_dev, n_text, calib,
                                   workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(got, want) and torch.equal(dev, want)
    with pytest.raises(cq.CqError) as e:
        cq.cq_decode_attn(*args, workspace=torch.empty(size, dtype=torch.uint8, device="cuda")[:size - 256])
    assert e.value.status == cq.CQ_ERR_WORKSPACE


def test_split_rows_with_a_workspace_for_a_longer_tail():
    """Rows of 45824 tokens are cut into more chunks with a tail of 9386 tokens than with one of 10914, to fill the
    last round of workgroups: the workspace of the latter serves the former, with fewer chunks."""
    n, longest, n_text = 45824, 10914, 9386
    w = synth.WORKLOADS[1].replace(batch=10, n_kv_heads=1, n_q_heads=2, n_vis=n, n_text=longest, seed=3)
    x = synth.make_inputs(w, "cuda")
    lay = cq.make_layout(10, 2, 1, 128, n, 4, 0, 1, 128, 128)
    calib = cq.make_calib(cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)
    k, v = cq.cq_quantize_kv(lay, x["k"], x["v"])
    args = (lay, x["q"], k, v, x["k_text"], x["v_text"], n_text, calib)
    prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_TUNED)
    try:
        size = cq.cq_decode_workspace_bytes(lay, longest, calib)
        assert size < cq.cq_decode_workspace_bytes(lay, n_text, calib)
        want = cq.cq_decode_attn(*args)
        got = cq.cq_decode_attn(*args, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
    finally:
        cq.cq_bench_set_kernel_path(prev)
    err = O.rel_l2(got.cpu().numpy().astype(np.float64), want.cpu().numpy().astype(np.float64))
    assert err <= 2 * H.REGRESSION_TOL, err      # two fp16 results
