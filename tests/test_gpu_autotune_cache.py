"""The autotuner's results are shared by plans that search the same forms: two
plans of one grid, source and receiver-node count that differ in a magnetic
receiver on a high wall (which takes the general kernels) or in the kind of
source are timed by themselves; a second plan of the same survey is not."""
import pytest

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")


def tuned(w, zchunk):
    """The plan's ZCHUNK after tuning: the search keeps the plan's own value or
    takes the fused schedule's 2, 4 or 8; a shared result brings its own."""
    p = fw.Plan.from_workload(w, field_dtype="f32", acc_mode="f64")
    p.set_option(fw.FWD_OPT_ZCHUNK, zchunk)
    p.set_model(w.rho)
    p.autotune(steps=8)
    return p.info.n_rec_nodes, p.get_option(fw.FWD_OPT_ZCHUNK)


@pytest.mark.parametrize("order", [2, 4])
def test_wall_receivers_and_source_kinds_are_timed_by_themselves(order):
    w = tiny(seed=61 + order, n=(40, 18, 14), npml=3, ns=1, nr=1, rec_comp=(3,)).replace(
        nt=40, fd_order=order)
    m = w.replace(src_kind=1)
    wall = w.replace(rec_pos=w.rec_pos.copy())
    wall.rec_pos[0, 0] = w.x[-1] - 1e-3 * (w.x[-1] - w.x[-2])
    print(f"autotune cache, order {order}", flush=True)
    (na, a), (nb, b), (nc, c) = tuned(wall, 5), tuned(w, 3), tuned(m, 7)
    assert na == nb == nc
    assert a in (5, 2, 4, 8) and b in (3, 2, 4, 8) and c in (7, 2, 4, 8)
    assert tuned(w, 6) == (nb, b)                # the same survey: found, not timed again
