"""The rows of waves of the fourth-order updates against the general kernels,
bit for bit.  A magnetic receiver on a high wall sends the whole run to the
general kernels, so the same survey with one such receiver more (its residual
zero) has to give the same fields, data and gradient.  Sizes where the rows
can go wrong: fewer cells than the differences reach, one cell before, at and
past a wave's end, a last wave of one and two lanes (images across its edge),
more than two waves, no layers, layers of one cell, layers that end inside a
wave, several sources, both tile orders, magnetic sources."""
import numpy as np
import pytest
import torch

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")


def run(w, dtype, nr, **opt):
    p = fw.Plan.from_workload(w, field_dtype=dtype, acc_mode="f64")
    for k, v in opt.items():
        p.set_option(getattr(fw, "FWD_OPT_" + k.upper()), v)
    p.set_model(w.rho)
    p.basis_build(gamma_rel=1e-12)
    E, vol = p.forward(want_volume=True)
    rng = np.random.default_rng(5)
    shape = tuple(E.shape[:1]) + (nr,) + tuple(E.shape[2:])
    r = np.zeros(tuple(E.shape), dtype=complex)
    r[:, :nr] = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    g, Ea = p.adjoint(vol, torch.from_numpy(r).cuda() * E[:, :nr].abs().max(), want_adjoint_rec=True)
    return [t.cpu().numpy() for t in (E[:, :nr], p.volume_export(vol), g, Ea[:, :nr])]


@pytest.mark.parametrize("n,npml,ns,src_kind,dtype,opt", [
    ((4, 4, 4), 0, 1, 0, "f64", {}),
    ((7, 6, 8), 1, 1, 1, "f32", {}),
    ((63, 10, 10), 3, 2, 0, "f32", {"dft_block": 16}),
    ((64, 11, 10), 3, 1, 1, "f64", {"tile_order": 1}),
    ((65, 9, 9), 2, 2, 0, "f32", {"xcd_remap": 0}),
    ((66, 12, 10), 3, 1, 0, "f64", {"lean": 0}),
    ((130, 11, 12), 3, 2, 1, "f32", {"dft_block": 1}),
    ((200, 13, 14), 4, 1, 0, "f32", {}),
])
def test_bitwise_against_general_kernels(n, npml, ns, src_kind, dtype, opt):
    nr = 4
    w = tiny(seed=44, n=n, npml=npml, ns=ns, moment_dirs=True, nr=nr,
             rec_comp=(3,)).replace(nt=37, src_kind=src_kind, fd_order=4)
    wall = np.array([[w.x[-1] - 1e-3 * (w.x[-1] - w.x[-2]), w.y[1], w.z[1]]])
    v = w.replace(rec_pos=np.concatenate([w.rec_pos, wall]))
    print(f"order-4 rows against the general kernels, grid {n} npml {npml} {dtype} {opt}", flush=True)
    for x, y in zip(run(w, dtype, nr, **opt), run(v, dtype, nr, **opt)):
        assert np.isfinite(x).all() and np.abs(x).max() > 0
        assert np.array_equal(x, y)
