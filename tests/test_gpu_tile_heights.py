"""Tile rows of every height the producer computes, at the edges between them.

The producer computes 32, 64, 128, 192 or 256 token rows of a 256-row tile row, whichever holds its
routed rows.  One expert's rows take the counts around each edge (the last tile row of 257 rows
holds one row); hidden and ffn give 7 and 9 K steps, more than the operand rings hold, and columns
that fill no tile; the whole-tile and the K-split launches both run.  The tolerance is the stage's:
each output is one bf16 rounding of an fp32 sum, as the oracle's is."""
import numpy as np
import pytest

from paper_2607_19539_amd import binding as B
from paper_2607_19539_amd.workload import make_workload
from tests.gpu_helpers import DeviceWorkload, compare, log, oracle_bufs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EDGES = (1, 16, 17, 32, 33, 64, 65, 128, 129, 192, 193, 256, 257)


def with_rows(n0, n1, H=448, F=576):
    """Two local experts with n0 and n1 routed rows."""
    full = make_workload("tiny", overrides={"H": H, "F": F, "T_r": 600}, owner=0)
    off = full.expert_offsets
    assert off[1] >= n0 and off[2] - off[1] >= n1
    g = np.random.default_rng(n0 * 1000 + n1)
    return full.subset(np.concatenate([g.choice(int(off[1]), n0, replace=False),
                                       off[1] + g.choice(int(off[2] - off[1]), n1, replace=False)]))


@pytest.mark.timeout(120)
@pytest.mark.parametrize("n", EDGES)
def test_every_height_matches_the_oracle(n):
    wl = with_rows(n, 257 - n if n < 257 else 40)
    ref = oracle_bufs(wl)
    outs = []
    for flags, band_rows, split_k in ((B.MOE_LOCAL_DIRECT, 0, 0),                        # default tail split
                                      (B.MOE_LOCAL_DIRECT | B.MOE_SHARED_CUS, 0, 1),      # whole tiles
                                      (B.MOE_LOCAL_DIRECT, 32, 1)):                       # padding between groups
        dw = DeviceWorkload(torch, wl)
        with B.MoeStage(wl.H, wl.F, wl.E_l, wl.R, wl.self_rank, wl.rows, band_rows, 1, flags, 0, split_k) as st:
            for overlapped in (False, True):
                dw.fill()
                (st.run if overlapped else st.run_serial)(*dw.args())
                st.query()
                worst, rel = compare(dw.host_bufs(), ref)
                outs.append((split_k, [b.clone() for b in dw.bufs]))
    # Heights change neither the order nor the number of an output's products: runs with the same
    # K split agree bit for bit, also where band padding makes every tile row a whole one.
    for k in (0, 1):
        same = [b for s, b in outs if s == k]
        for other in same[1:]:
            assert all(torch.equal(a, b) for a, b in zip(same[0], other)), f"split_k={k}"
    log(f"rows {n}: worst {worst:.2e}, rel {rel:.2e}")


@pytest.mark.timeout(120)
@pytest.mark.parametrize("split_k", [0, 2, 3, 4, 8])
def test_an_earlier_call_s_activations_reach_no_output(split_k):
    """Gate/up stores the activation rows of a tile row's height, a down launch of explicit K parts reads
    all 256: the rest are an earlier call's, NaN here.  They are other token rows, so nothing that is
    stored may see them."""
    big = with_rows(257, 200)
    for n in (1, 33, 65, 192):
        wl = with_rows(n, 40)
        ref = oracle_bufs(wl)
        fresh = None
        for poisoned in (False, True):
            with B.MoeStage(wl.H, wl.F, wl.E_l, wl.R, wl.self_rank, big.rows, 0, 1, B.MOE_LOCAL_DIRECT, 0, split_k) as st:
                if poisoned:
                    dw = DeviceWorkload(torch, big)
                    dw.x.fill_(0x7FC0)
                    st.run_serial(*dw.args())
                    assert all(np.all((b & 0x7F80) == 0x7F80) for b in dw.host_bufs() if b.size)
                for overlapped in (False, True):
                    dw = DeviceWorkload(torch, wl)
                    (st.run if overlapped else st.run_serial)(*dw.args())
                    st.query()
                    compare(dw.host_bufs(), ref)
                    fresh = dw.bufs if fresh is None else fresh
                    assert all(torch.equal(a, b) for a, b in zip(fresh, dw.bufs)), (n, overlapped)
