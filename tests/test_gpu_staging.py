"""Host-planned runs enqueued faster than the GPU takes them: each plan is read from one of two pinned
halves by its run's reset, so a half may not be written again before the run that uses it has gone."""
import numpy as np
import pytest

from paper_2607_19539_amd import binding as B
from tests.test_gpu_devplan import Case, dispatch_routing

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H, F, E, R = 256, 256, 3, 3


def cases(n):
    out, w = [], None
    for i in range(n):
        rng = np.random.default_rng(100 + i)
        rows = int(rng.integers(20, 700))
        share = rng.multinomial(rows, rng.dirichlet(np.ones(E * R))).reshape(E, R)
        c = Case(H, F, E, R, 0, *dispatch_routing(rng, share.tolist(), R, bool(i % 2), 5), seed=i, w=w)
        w = (c.w1, c.w3, c.w2)
        out.append(c)
    return out


@pytest.mark.parametrize("order", ["host", "host and device"])
def test_runs_queued_behind_other_work_keep_their_own_plans(order):
    cs = cases(7)
    want = []
    for c in cs:
        with B.MoeStage(H, F, E, R, 0, 700, 0, 1, B.MOE_LOCAL_DIRECT | B.MOE_SHARED_CUS, 0, 0) as st:
            c.fill()
            st.run_serial(*c.host_args())
            want.append(c.out())
            st.query()
    busy = torch.randn((4096, 4096), device="cuda")
    stream = torch.cuda.Stream()
    with B.MoeStage(H, F, E, R, 0, 700, 0, 1, B.MOE_LOCAL_DIRECT | B.MOE_SHARED_CUS, 0, 0) as st:
        for c in cs:
            c.fill()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(10):
                busy = busy @ busy * 1e-2       # the runs queue up behind this
            for i, c in enumerate(cs):
                if order != "host" and i % 3 == 1:
                    (st.run_devplan if i % 2 else st.run_serial_devplan)(*c.dev_args())
                else:
                    (st.run if i % 2 else st.run_serial)(*c.host_args())
            st.query()
        for i, (c, ref) in enumerate(zip(cs, want)):
            for r, (a, b) in enumerate(zip(c.out(), ref)):
                assert np.array_equal(a, b), (i, r)


def test_a_refused_call_between_runs_leaves_the_halves_alone():
    a, b = cases(2)
    with B.MoeStage(H, F, E, R, 0, 700, 0, 1, B.MOE_LOCAL_DIRECT, 0, 0) as st:
        outs = []
        for c in (a, b, a):
            c.fill()
            st.run_serial(*c.host_args())
            bad = c.src.copy()
            bad[0] = R
            with pytest.raises(B.MoeError):
                st.run_serial(c.x, c.off, bad, c.slot, c.w1, c.w3, c.w2, c.bufs, c.rr)
            outs.append(c.out())
            st.query()
        assert all(np.array_equal(x, y) for x, y in zip(outs[0], outs[2]))
