"""Rows of waves with receivers that the run reaches: every output (receivers,
volume transform, gradient, adjoint receivers) is non-zero, so that the tables
and the block decode of both runs are compared over more than one round of
runs of 128 blocks, and magnetic nodes in the interior and on a high wall.
The residual is of size one, whatever the data."""
import numpy as np
import pytest
import torch

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")


def run(w, dtype, **opt):
    p = fw.Plan.from_workload(w, field_dtype=dtype, acc_mode="f64")
    for k, v in opt.items():
        p.set_option(getattr(fw, "FWD_OPT_" + k.upper()), v)
    p.set_model(w.rho)
    p.basis_build(gamma_rel=1e-12)
    E, vol = p.forward(want_volume=True)
    rng = np.random.default_rng(7)
    r = rng.standard_normal(tuple(E.shape)) + 1j * rng.standard_normal(tuple(E.shape))
    g, Ea = p.adjoint(vol, torch.from_numpy(r).cuda(), want_adjoint_rec=True)
    return [t.cpu().numpy() for t in (E, p.volume_export(vol), g, Ea)]


def near(w, cells):
    """Receivers a few cells from the sources, in other rows and planes too."""
    rng = np.random.default_rng(8)
    h = np.diff(w.x).min()
    for q in range(len(w.rec_pos)):
        w.rec_pos[q] = w.src_pos[q % w.ns] + rng.uniform(-cells, cells, 3) * h
    return w


def same(a, b):
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.abs(x).max() > 0
        assert np.array_equal(x, y)


@pytest.mark.parametrize("order,xcd,ns", [(0, 1, 2), (1, 1, 2), (1, 0, 3), (0, 1, 1)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_decode_of_both_runs(order, xcd, ns, dtype):
    w = near(tiny(seed=71, n=(66, 31, 21), npml=2, ns=ns, moment_dirs=True, nr=6).replace(nt=19), 2.0)
    print(f"decode of both runs, tile order {order} xcd {xcd} ns {ns} {dtype}", flush=True)
    same(run(w, dtype, tile_order=order, xcd_remap=xcd), run(w, dtype, vector=4, vector_h=4))


@pytest.mark.parametrize("src_kind,wall", [(0, False), (1, False), (0, True), (1, True)])
def test_magnetic_nodes_reached(src_kind, wall):
    w = near(tiny(seed=72, n=(70, 10, 9), npml=2, ns=2, moment_dirs=True, nr=4,
                  rec_comp=(0, 3, 4, 5)).replace(nt=33, src_kind=src_kind), 1.0)
    if wall:
        w = w.replace(rec_comp=(3,))
        w.rec_pos[0] = [w.x[-1] - 10.0, w.y[4], w.z[4]]
    print(f"magnetic nodes, source kind {src_kind}, on the wall {wall}", flush=True)
    same(run(w, "f32"), run(w, "f32", schedule=1))
