"""The single-workgroup device planner and the four-kernel one, on either side of the line between
them: both must build the host's plan, and report the same routing errors.  The line is a capacity
(2048 rows, 64 experts, 1024 (expert, rank) pairs), so the same routing takes either path."""
import numpy as np
import pytest

from paper_2607_19539_amd import binding as B
from tests.test_gpu_devplan import (Case, _expect_device_error, assert_same_plan, check_both_paths, dispatch_routing,
                                    host_tables)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def case(E_l, R, rows, contiguous, seed, me=0):
    rng = np.random.default_rng(seed)
    share = rng.multinomial(rows, rng.dirichlet(np.full(E_l * R, 0.7))).reshape(E_l, R)
    return Case(128, 192, E_l, R, me, *dispatch_routing(rng, share.tolist(), R, contiguous, 9), seed=seed)


@pytest.mark.parametrize("E_l,R,rows,contiguous", [
    (1, 1, 1, True), (1, 3, 2048, False), (2, 4, 255, True), (64, 16, 2048, True), (64, 16, 2047, False),
    (63, 5, 700, False), (8, 2, 2048, True), (2, 40, 300, True),   # 40 ranks: past the table in arguments
])
def test_both_sides_of_the_row_limit(E_l, R, rows, contiguous):
    c = case(E_l, R, rows, contiguous, seed=E_l + R + rows, me=R - 1)
    for max_rows in (2048, 2049):
        for band_rows, mgb in ((0, 1), (16, 3)):
            check_both_paths(c, overlapped=True, max_rows=max_rows, band_rows=band_rows, mgb=mgb)
        check_both_paths(c, overlapped=False, max_rows=max_rows)


@pytest.mark.parametrize("E_l,R", [(65, 2), (64, 17)])
def test_past_the_expert_and_pair_limits(E_l, R):
    check_both_paths(case(E_l, R, 600, True, seed=E_l), overlapped=True)


@pytest.mark.parametrize("max_rows", [2048, 2049])
def test_errors_on_both_sides(max_rows):
    good = case(4, 3, 900, True, seed=5)
    kw = dict(x=good.x, w=(good.w1, good.w3, good.w2))

    def variant(off=None, src=None, slot=None):
        return Case(good.H, good.F, good.E_l, good.R, good.self_rank, good.off if off is None else off,
                    good.src if src is None else src, good.slot if slot is None else slot, good.rr, **kw)

    with B.MoeStage(good.H, good.F, good.E_l, good.R, 0, max_rows, 0, 1, B.MOE_LOCAL_DIRECT, 0, 0) as st:
        off = good.off.copy(); off[1] = off[2] + 1
        _expect_device_error(st, variant(off=off), B.MOE_EROUTING)
        src = good.src.copy(); src[899] = good.R
        _expect_device_error(st, variant(src=src), B.MOE_EROUTING)
        slot = good.slot.copy(); slot[450] = good.rr[good.src[450]]
        _expect_device_error(st, variant(slot=slot), B.MOE_EROUTING, serial=True)
        i, j = 0, next(j for j in range(int(good.off[1]), 900) if good.src[j] == good.src[0])
        slot = good.slot.copy(); slot[j] = slot[i]   # the same (rank, slot) in two experts
        _expect_device_error(st, variant(slot=slot), B.MOE_EROUTING)
        # A good call right after: the header and every table again, and the host-planned run's bytes.
        for overlapped in (False, True):
            good.fill()
            (st.run_devplan if overlapped else st.run_serial_devplan)(*good.dev_args())
            dev_out = good.out()
            st.query()
            assert_same_plan(st.plan(), host_tables(st, good, overlapped), f"overlapped={overlapped}")
            good.fill()
            (st.run if overlapped else st.run_serial)(*good.host_args())
            for r, (a, b) in enumerate(zip(dev_out, good.out())):
                assert np.array_equal(a, b), f"rank {r}, overlapped={overlapped}"
            st.query()
            _expect_device_error(st, variant(src=src), B.MOE_EROUTING, serial=not overlapped)
