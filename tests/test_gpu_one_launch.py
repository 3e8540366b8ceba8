"""The one-launch step of schedule 0 (order 2) against the two-kernel form
(16-byte vectors keep that path) bit for bit: receivers, volume transform,
gradient and adjoint receivers, over the sizes where its waves of 64 x nodes
and its skipped high walls can go wrong -- one cell before, at and past a
wave's end, more than two waves, the smallest y and z, layers that end inside
a wave, one that begins in the last wave's first lanes -- with and without
layers, several sources, both precisions, both tile orders, the XCD remap
over more than one run of 128 blocks, and magnetic nodes, also on the high
walls (where the two kernels run instead)."""
import numpy as np
import pytest
import torch

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")


def run(w, dtype, acc, **opt):
    p = fw.Plan.from_workload(w, field_dtype=dtype, acc_mode=acc)
    for k, v in opt.items():
        p.set_option(getattr(fw, "FWD_OPT_" + k.upper()), v)
    p.set_model(w.rho)
    p.basis_build(gamma_rel=1e-12)
    E, vol = p.forward(want_volume=True)
    rng = np.random.default_rng(5)
    r = rng.standard_normal(E.shape) + 1j * rng.standard_normal(E.shape)
    g, Ea = p.adjoint(vol, torch.from_numpy(r).cuda() * E.abs().max(), want_adjoint_rec=True)
    return [t.cpu().numpy() for t in (E, p.volume_export(vol), g, Ea)]


@pytest.mark.parametrize("n,npml,ns,dtype,opt", [
    ((4, 4, 4), 0, 1, "f64", {}),
    ((63, 10, 10), 3, 2, "f32", {"dft_block": 16}),
    ((64, 11, 10), 3, 1, "f64", {"tile_order": 1}),
    ((65, 9, 9), 2, 2, "f32", {"xcd_remap": 0}),
    ((69, 12, 10), 3, 1, "f32", {}),
    ((130, 11, 12), 3, 2, "f32", {"stream_stores": 1}),
    ((129, 9, 9), 0, 1, "f64", {"lean": 0}),
    ((200, 13, 14), 4, 1, "f64", {"stream_stores": 1, "dft_block": 1}),
])
def test_bitwise_against_two_kernels(n, npml, ns, dtype, opt):
    w = tiny(seed=41, n=n, npml=npml, ns=ns, moment_dirs=True, nr=5).replace(nt=37)
    print(f"one launch against two, grid {n} npml {npml} {dtype} {opt}", flush=True)
    a = run(w, dtype, "kahan" if dtype == "f32" else "f64", **opt)
    b = run(w, dtype, "kahan" if dtype == "f32" else "f64", vector=4, vector_h=4, **opt)
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.abs(x).max() > 0
        assert np.array_equal(x, y)


@pytest.mark.parametrize("src_kind,wall", [(0, False), (1, False), (0, True)])
def test_magnetic_nodes_bitwise(src_kind, wall):
    """Magnetic sources and receivers, in the interior and in the last half
    cell below a high wall (their weights then touch the wall's nodes)."""
    w = tiny(seed=42, n=(70, 10, 9), npml=2, ns=2, moment_dirs=True, nr=4,
             rec_comp=(0, 3, 4, 5)).replace(nt=33, src_kind=src_kind)
    if wall:
        w.rec_pos[0] = [w.x[-1] - 10.0, w.y[4], w.z[4]]
        w = w.replace(rec_comp=(3,))
    print(f"magnetic nodes, source kind {src_kind}, on the wall {wall}", flush=True)
    a = run(w, "f32", "f64")
    b = run(w, "f32", "f64", schedule=1)
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.array_equal(x, y)


def test_graph_follows_rebuilt_entry_lists():
    """A captured graph holds the entry lists' addresses: after another
    schedule has rebuilt them, the same configuration runs on the new ones."""
    w = tiny(seed=43, n=(20, 12, 11), npml=3, ns=2).replace(nt=64)
    print("graph after rebuilt entry lists", flush=True)
    p = fw.Plan.from_workload(w, field_dtype="f32", acc_mode="f64")
    p.set_model(w.rho)
    E0 = p.forward().cpu().numpy()
    p.set_option(fw.FWD_OPT_SCHEDULE, 1)
    p.set_option(fw.FWD_OPT_GRAPH_STEPS, 0)
    p.forward()
    hold = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    p.set_option(fw.FWD_OPT_SCHEDULE, 0)
    p.set_option(fw.FWD_OPT_GRAPH_STEPS, 32)
    E1 = p.forward().cpu().numpy()
    del hold
    assert np.abs(E0).max() > 0 and np.array_equal(E0, E1)


@pytest.mark.parametrize("dtype,ns,nf", [("f64", 3, 5), ("f32", 1, 1), ("f64", 8, 3)])
def test_entries_crowded_into_few_rows(dtype, ns, nf):
    """Receivers that share rows, lanes and nodes with each other and with the
    sources, every component, an odd number of frequencies: the rows' tables
    against the lists of the two kernels."""
    w = tiny(seed=47, n=(70, 9, 9), npml=2, ns=ns, moment_dirs=True, nr=9,
             rec_comp=(0, 1, 2, 3, 4, 5)).replace(nt=33)
    w = w.replace(freqs=np.linspace(0.2, 1.0, nf))
    w.rec_pos[:] = w.src_pos[0]
    w.rec_pos[:, 0] += np.linspace(-1.0, 1.0, 9) * 2.2 * np.diff(w.x).min()
    w.rec_pos[-1] = w.rec_pos[0]
    print(f"crowded entries, {dtype} ns {ns} nf {nf}", flush=True)
    a = run(w, dtype, "f64")
    b = run(w, dtype, "f64", vector=4, vector_h=4)
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.abs(x).max() > 0
        assert np.array_equal(x, y)


@pytest.mark.parametrize("order,xcd,ns", [(0, 1, 2), (1, 1, 2), (1, 0, 3), (0, 1, 1)])
def test_decode_over_whole_rounds_of_runs(order, xcd, ns):
    """More than 1024 blocks: runs of 128 blocks an XCD, the blocks past the
    last whole round, both tile orders (the volume holds every row)."""
    w = tiny(seed=48, n=(66, 31, 21), npml=2, ns=ns, moment_dirs=True, nr=4).replace(nt=19)
    print(f"decode over rounds of runs, tile order {order} xcd {xcd} ns {ns}", flush=True)
    a = run(w, "f32", "f64", tile_order=order, xcd_remap=xcd)
    b = run(w, "f32", "f64", vector=4, vector_h=4)
    assert np.abs(a[1]).max() > 0        # the volume; 19 steps may not reach a receiver
    for x, y in zip(a, b):
        assert np.isfinite(x).all() and np.array_equal(x, y)
