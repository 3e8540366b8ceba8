"""The time-domain adjoint's rows of waves against the general kernels, bit for
bit (16-byte vectors keep the general path; the forward steps are bitwise the
same).  Grids where the rows can go wrong -- one cell before, at and past a
wave's end, a last wave of one lane, more than two waves, no layers, layers
ending where the wave does -- with several sources, electric and magnetic
receivers and sources, and segments of one step, past the run, and that do
not divide it (the last one is kept in the forward run)."""
import numpy as np
import pytest
import torch

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")


def run(w, dtype, segment, **opt):
    p = fw.Plan.from_workload(w, field_dtype=dtype, acc_mode="f64")
    for k, v in opt.items():
        p.set_option(getattr(fw, "FWD_OPT_" + k.upper()), v)
    p.set_model(w.rho)
    E = p.forward()
    rng = np.random.default_rng(6)
    r = rng.standard_normal(tuple(E.shape)) + 1j * rng.standard_normal(tuple(E.shape))
    g = p.adjoint_td(torch.from_numpy(r).cuda() * E.abs().max(), segment=segment)
    return [t.cpu().numpy() for t in (E, g)]


@pytest.mark.parametrize("n,npml,ns,comps,src_kind,dtype,segment,opt", [
    ((4, 4, 4), 0, 1, (0, 1), 0, "f64", 8, {}),
    ((63, 10, 10), 3, 2, (0, 1, 2), 0, "f32", 16, {}),
    ((64, 11, 10), 3, 1, (0, 3), 1, "f64", 33, {"tile_order": 1}),
    ((65, 9, 9), 2, 2, (0, 3, 4, 5), 0, "f32", 1, {"xcd_remap": 0}),
    ((66, 12, 10), 3, 1, (3, 4, 5), 0, "f32", 100, {"lean": 0}),
    ((67, 11, 12), 3, 1, (2,), 1, "f32", 10, {}),
    ((130, 13, 14), 4, 1, (1, 4), 0, "f64", 7, {}),
])
def test_bitwise_against_general_kernels(n, npml, ns, comps, src_kind, dtype, segment, opt):
    w = tiny(seed=46, n=n, npml=npml, ns=ns, moment_dirs=True, nr=5,
             rec_comp=comps).replace(nt=33, src_kind=src_kind)
    print(f"time-domain rows, grid {n} npml {npml} {dtype} segment {segment}", flush=True)
    a = run(w, dtype, segment, **opt)
    b = run(w, dtype, segment, vector=4, vector_h=4, **opt)
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.abs(x).max() > 0
        assert np.array_equal(x, y)
