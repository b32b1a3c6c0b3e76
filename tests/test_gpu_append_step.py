"""Append with the length on the device at the sizes where it changes launches (1024 pieces of 16 bytes
per tensor): the new token lands in its slot and nowhere else, the length rises by one; a full tail and
a negative length leave everything alone."""
import pytest
import torch

from paper_2502_14882_amd import binding as cq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,d", [(1, 32), (5, 96), (64, 128), (65, 128), (32, 256), (33, 256)])
def test_append_devlen_sizes(rows, d):
    lay = cq.make_layout(rows, 1, 1, d, 0, v_group=32)
    gen = torch.Generator().manual_seed(rows * d)
    cap = 5
    tails = [torch.randn(rows, 1, cap, d, generator=gen).half() for _ in range(2)]
    new = [torch.randn(rows, 1, 1, d, generator=gen).half() for _ in range(2)]
    for n in (0, 3, 4, 5, 9, -1):
        k, v = (t.cuda() for t in tails)
        length = torch.tensor([n], dtype=torch.int32, device="cuda")
        cq.cq_append_text_kv_devlen(lay, k, v, length, new[0].cuda(), new[1].cuda())
        torch.cuda.synchronize()
        want = [t.clone() for t in tails]
        if 0 <= n < cap:
            for w, x in zip(want, new):
                w[:, :, n] = x[:, :, 0]
        assert int(length) == (n + 1 if 0 <= n < cap else n)
        assert torch.equal(k.cpu(), want[0]) and torch.equal(v.cpu(), want[1]), (rows, d, n)
