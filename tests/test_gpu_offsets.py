"""Fields of 2 to 4 GiB a source, where the rows' 32-bit byte offsets pass
2^31, and of more than 4 GiB, where the general kernels run instead: receivers
and the volume transform around a source in the last rows and planes (the
largest offsets), bit for bit against the general kernels (16-byte vectors at
order 2; at order 4 a magnetic receiver more, on a high wall)."""
import numpy as np
import pytest
import torch

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")


def run(w, **opt):
    p = fw.Plan.from_workload(w, field_dtype="f64", acc_mode="f32")
    for k, v in opt.items():
        p.set_option(getattr(fw, "FWD_OPT_" + k.upper()), v)
    p.set_model(w.rho)
    E, vol = p.forward(want_volume=True)
    i = p.info
    return E, p.volume_export(vol), 6 * 8 * i.px * (i.ny + 1) * (i.nz + 1)


@pytest.mark.parametrize("m,order", [(838, 2), (838, 4), (1184, 2)])
def test_large_offsets(m, order):
    print(f"large offsets, 62x{m}x{m} cells, order {order}", flush=True)
    rng = np.random.default_rng(91)
    w = tiny(seed=91, n=(62, 8, 8), npml=2, nr=2, nfreq=1, rec_comp=(3,))
    # the wide grid's axes and model without tiny's random numbers a cell
    y = np.concatenate([[0.0], np.cumsum(100.0 * 1.1 ** rng.uniform(-1, 1, m))])
    rho = np.ones((m, m, 62))
    rho[-20:] = 10.0 ** rng.uniform(0.0, 1.0, (20, m, 62))
    w = w.replace(y=y, z=y.copy(), rho=rho, nt=9, fd_order=order)
    w.src_pos[0] = [w.x[30], y[-7], y[-6]]
    w.rec_pos[:] = w.src_pos[0] + 100.0 * rng.uniform(-1.0, 1.0, (2, 3))
    E, V, size = run(w)
    assert torch.isfinite(V.real).all() and torch.any(E) and torch.any(V)
    assert (2 ** 31 < size < 2 ** 32) if m == 838 else size > 2 ** 32
    if order == 2:
        E2, V2, _ = run(w, vector=4, vector_h=4)
    else:
        wall = [[w.x[-1] - 1e-3 * (w.x[-1] - w.x[-2]), y[4], y[4]]]
        E2, V2, _ = run(w.replace(rec_pos=np.concatenate([w.rec_pos, wall])))
    assert torch.equal(E, E2[:, :2]) and torch.equal(V, V2)
