"""Sizes of the scratch, on the host: a workspace of the size asked for the largest tail serves every
shorter one.  Nothing is launched: the decode calls below bring a workspace too small for any kernel
and are refused, with the size they need in the message."""
import ctypes
import random
import re

import pytest

from paper_2502_14882_amd import binding as cq

FAKE = 0x10000     # aligned, non-NULL, never touched
DYN = (cq.CQ_CALIB_DYNAMIC, 1.0, 2.0)


def needed(lay, n_text):
    """Bytes that cq_decode_attn itself asks for."""
    t = cq.CqQTensor(FAKE, FAKE, FAKE)
    calib = cq.make_calib(*DYN)
    rc = cq.lib().cq_decode_attn(ctypes.byref(lay), FAKE, ctypes.byref(t), ctypes.byref(t), FAKE, FAKE, n_text,
                                 n_text, ctypes.byref(calib), 0.0, FAKE, FAKE, 0, None)
    assert rc == cq.CQ_ERR_WORKSPACE
    return int(re.search(rb"(\d+) needed", cq.lib().cq_last_error()).group(1))


# where the tail's chunks grow: 64 chunks of 128 tokens are 8192
TAILS = [0, 1, 127, 128, 129, 1000, 4096, 6785, 7493, 8191, 8192, 8193, 8320, 9000, 10000, 16384, 16385, 24576,
         24577, 40000]


@pytest.mark.parametrize("args", [
    (1, 16, 4, 64, 3328, 1, 0, 1, 128, 64),       # a layout only the tile kernels take
    (1, 4, 4, 64, 1024, 1, 0, 1, 64, 64),
    (2, 8, 2, 256, 1003, 4, 0, 0, 1003, 1003),
    (1, 32, 8, 128, 3328, 1, 0, 1, 128, 128),     # layouts that they finish sooner than the fused kernel
    (1, 32, 8, 128, 3328, 1, 0, 1, 64, 128),
    (3, 6, 2, 128, 0, 1, 0, 1, 32, 128),          # a tail and nothing else
    (48, 16, 4, 64, 1024, 1, 0, 1, 64, 64),       # passes 8 MiB inside the range
    (8, 32, 8, 128, 3003, 1, 0, 0, 3003, 3003),
])
def test_the_largest_tail_serves_the_shorter_ones(args):
    lay, calib = cq.make_layout(*args), cq.make_calib(*DYN)
    tails = [t for t in TAILS if args[4] + t > 0]
    sizes = [cq.cq_decode_workspace_bytes(lay, t, calib) for t in tails]
    assert sizes == sorted(sizes), list(zip(tails, sizes))
    for t, size in zip(tails, sizes):
        assert needed(lay, t) <= size, (t, size)


def test_drawn_layouts():
    rng = random.Random(20)
    for _ in range(400):
        d, bits = rng.choice((64, 128, 256)), rng.choice((1, 2, 4, 8))
        n_q, n_kv = rng.choice(((1, 1), (8, 2), (14, 2), (32, 8), (16, 16), (40, 4)))
        n = int(2 ** rng.uniform(0, 14))
        v_axis, v_group = rng.choice(((0, n), (1, d)))
        lay = cq.make_layout(int(2 ** rng.uniform(0, 6)), n_q, n_kv, d, n, bits, 0, v_axis, n, v_group)
        calib = cq.make_calib(*DYN)
        longest = int(2 ** rng.uniform(0, 16))
        top = cq.cq_decode_workspace_bytes(lay, longest, calib)
        for t in [longest] + [rng.randrange(longest) for _ in range(20)]:
            what = ({f: getattr(lay, f) for f, _ in lay._fields_}, longest, t)
            assert cq.cq_decode_workspace_bytes(lay, t, calib) <= top, what
            assert needed(lay, t) <= top, what


def test_tau_search_the_largest_tail_serves_the_shorter_ones():
    """The chunks of the grid kernels are whole rounds of tokens, so their number can fall as the tail grows."""
    rng = random.Random(21)
    t_q = cq.CqQTensor(FAKE, FAKE, FAKE)
    grid = (ctypes.c_float * 4)(0.0, 1.0, 2.0, 3.0)
    for _ in range(400):
        d, n_text = rng.choice((64, 96, 128)), int(2 ** rng.uniform(0, 14))
        n_q, n_kv = rng.choice(((1, 1), (8, 2), (32, 8), (16, 16)))
        n = int(2 ** rng.uniform(0, 14))
        lay = cq.make_layout(int(2 ** rng.uniform(0, 5)), n_q, n_kv, d, n, 1, 0, 0, n, n)
        top = cq.cq_tau_search_workspace_bytes(lay, n_text, 4, 4)
        for t in [n_text] + [rng.randrange(n_text) for _ in range(20)]:
            what = ({f: getattr(lay, f) for f, _ in lay._fields_}, n_text, t)
            assert cq.cq_tau_search_workspace_bytes(lay, t, 4, 4) <= top, what
            rc = cq.lib().cq_tau_search(ctypes.byref(lay), FAKE, FAKE, ctypes.byref(t_q), FAKE, t, t, grid, 4, grid, 4,
                                        0.0, FAKE, FAKE, 0, None)
            assert rc == cq.CQ_ERR_WORKSPACE
            assert int(re.search(rb"(\d+) needed", cq.lib().cq_last_error()).group(1)) <= top, what


def test_no_scratch_for_kernels_that_never_run():
    """Where the tile kernels would finish sooner but no tail is short enough for them to stay within the
    scratch of the allocation-free entry point, the query asks for what the call uses."""
    lay, calib = cq.make_layout(16, 32, 8, 128, 6400, 8, 0, 1, 128, 128), cq.make_calib(*DYN)
    assert 16 * 32 * 6400 * 4 > cq.CQ_NOALLOC_SCRATCH_BYTES            # the logits alone
    for t in (0, 100, 1000):
        assert cq.cq_decode_workspace_bytes(lay, t, calib) == needed(lay, t) < 4 << 20
    # one that fits with a short tail keeps asking for it
    lay = cq.make_layout(16, 32, 8, 128, 2560, 8, 0, 1, 128, 128)
    assert needed(lay, 100) > 4 << 20 and cq.cq_decode_workspace_bytes(lay, 4096, calib) >= needed(lay, 100)


def test_a_long_tail_for_two_head_sets_stays_on_the_streaming_kernels():
    """They read the tail once, the tile kernels once per head set; a shorter tail goes to the tile kernels, and
    the size asked for the long one serves it."""
    lay, calib = cq.make_layout(14, 64, 8, 128, 128, 1), cq.make_calib(*DYN)
    prev = cq.cq_bench_set_kernel_path(cq.CQ_PATH_TUNED)
    tuned = [needed(lay, t) for t in (100, 1000)]
    cq.cq_bench_set_kernel_path(prev)
    assert needed(lay, 1000) == tuned[1] and needed(lay, 100) != tuned[0]
    assert cq.cq_decode_workspace_bytes(lay, 1000, calib) >= needed(lay, 100)


# (layout, tail) of shared rows, and the scratch of one (min, max) pair and one partial per (head, chunk) that
# workspaces for them were first made with
SHARED = [((120, 16, 16, 128, 10752, 8, 0, 1, 128, 128), 0), ((131, 64, 8, 128, 1920, 2, 0, 1, 64, 128), 33),
          ((154, 32, 8, 128, 63744, 4, 0, 1, 64, 128), 0), ((31, 64, 8, 128, 65536, 4, 0, 1, 128, 128), 0),
          ((62, 64, 8, 128, 32448, 1, 0, 1, 64, 128), 221), ((165, 16, 16, 128, 46592, 1, 0, 1, 64, 128), 3485)]
SHARED_BYTES = [2027520, 4426752, 20815872, 8380416, 8380416, 8363520]


@pytest.mark.parametrize("case,size", zip(SHARED, SHARED_BYTES))
def test_words_of_the_exchange_take_no_scratch_of_their_own(case, size):
    args, n_text = case
    assert needed(cq.make_layout(*args), n_text) <= size


@pytest.mark.parametrize("args", [(82, 48, 8, 128, 1024, 2, 0, 1, 32, 128), (20, 64, 8, 128, 3328, 4, 0, 1, 128, 128),
                                  (600, 64, 8, 128, 512, 1, 0, 0, 128, 128)])
def test_whole_rows_of_two_head_sets_take_the_least_scratch(args):
    """One workgroup owns a row (of each set): 256 bytes, also of the entry point that allocates nothing."""
    assert needed(cq.make_layout(*args), 20) == 256


# batch, n_vis, tail; whether the streaming kernels take it: rounds of long tails, rows that are long beside them, 128 rows
# (one round)
SETS = [(64, 768, 1000, True), (53, 768, 804, True), (64, 3328, 128, False), (28, 768, 38, False), (16, 768, 1000, False)]


@pytest.mark.parametrize("batch,n_vis,n_text,streamed", SETS)
def test_two_head_sets_on_chip_unless_rounds_of_a_long_tail(batch, n_vis, n_text, streamed):
    """8 KV heads of 8 query heads.  The streaming kernels keep 16-bit logits in scratch."""
    lay = cq.make_layout(batch, 64, 8, 128, n_vis, 1)
    assert (needed(lay, n_text) > batch * 64 * n_vis * 2) == streamed
