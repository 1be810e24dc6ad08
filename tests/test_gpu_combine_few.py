"""The combine where few workgroups run, on either side of that line: bit-exact with the oracle's order.

One vector per thread (up to 256 workgroups of the wider split, 512 with eight choices or more), next
to the wider split: ragged hidden sizes around one and two parts of a row, choices around the batches of
four, slots out of range."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2607_19539_amd import binding as B

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,T,k", [(8, 1, 5), (2048, 3, 8), (2056, 5, 9), (4096, 255, 5), (4104, 7, 17), (7168, 48, 8),
                                   (2048, 511, 6), (2048, 512, 6), (7168, 512, 8), (4096, 16, 4),
                                   # either side of the lines of the split: tokens, choices, a short last part
                                   (2056, 256, 6), (2056, 257, 6), (2056, 257, 8), (7168, 256, 5), (7168, 257, 5),
                                   (7168, 513, 8), (16384, 129, 6), (64, 100, 9), (65536, 3, 3), (8, 70000, 2)])
def test_few_workgroups(H, T, k):
    g = np.random.default_rng(H + T + k)
    rows = T * k + 3
    recv = g.integers(0, 1 << 16, (rows, H), dtype=np.uint16)
    recv &= 0xBFFF                                           # finite: no exponent of all ones
    slot = g.permutation(rows)[:T * k].astype(np.int32).reshape(T, k)
    gate = g.random((T, k), dtype=np.float32)
    d = lambda a, t: torch.from_numpy(np.ascontiguousarray(a).view(t)).cuda()  # noqa: E731
    out = torch.empty((T, H), dtype=torch.int16, device="cuda")
    bad = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.moe_combine(d(recv, np.int16), d(slot, np.int32), d(gate, np.float32), out, bad)
    ref = np.zeros((T, H), np.uint16)
    assert orc.get().combine(recv, slot, gate, ref) == 0
    assert np.array_equal(out.cpu().numpy().view(np.uint16), ref)
    assert int(bad.item()) == 0
    slot2 = slot.copy()
    slot2[0, k - 1] = rows                                   # one past the buffer: skipped and counted
    gate2 = gate.copy()
    gate2[0, k - 1] = 0.0
    B.moe_combine(d(recv, np.int16), d(slot2, np.int32), d(gate, np.float32), out, bad)
    assert int(bad.item()) == 1
    ref_skip = np.zeros((T, H), np.uint16)
    assert orc.get().combine(recv, slot, gate2, ref_skip) == 0  # a zero gate adds +-0 to the same sum
    got = out.cpu().numpy().view(np.uint16)
    same = (got == ref_skip) | (((got | ref_skip) & 0x7FFF) == 0)
    assert same.all()
