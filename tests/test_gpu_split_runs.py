"""Split runs: the step index lives in the workspace, so one plan steps
several of them in turn, a workspace put back by a plain copy continues from
where it then is, a captured call replays from where the last one ended, and
steps past a run's end add nothing.  Each against the uninterrupted run, bit
for bit, on the one-launch step, the rows of waves of order 4 and the general
kernels (16-byte vectors), eager and through the plan's graph."""
import numpy as np
import pytest
import torch

from workloads import tiny

pytestmark = pytest.mark.gpu

fw = pytest.importorskip("paper_2211_16665_amd.fwdem")

FORMS = [
    (2, 0, "f32", {}),
    (2, 1, "f64", {"tile_order": 1}),
    (2, 0, "f32", {"graph_steps": 0}),
    (2, 0, "f32", {"vector": 4, "vector_h": 4}),
    (4, 0, "f64", {}),
    (4, 1, "f32", {"graph_steps": 0}),
]


def plan(order, src_kind, dtype, opt):
    """A plan of 75 steps and its receivers after an uninterrupted run."""
    w = tiny(seed=51, n=(67, 10, 9), npml=2, ns=2, moment_dirs=True, nr=4,
             rec_comp=(0, 2, 4)).replace(nt=75, src_kind=src_kind, fd_order=order)
    p = fw.Plan.from_workload(w, field_dtype=dtype, acc_mode="f64")
    for k, v in opt.items():
        p.set_option(getattr(fw, "FWD_OPT_" + k.upper()), v)
    p.set_model(w.rho)
    E = p.forward().cpu().numpy()
    assert np.isfinite(E).all() and np.abs(E).max() > 0
    return p, E


def buffer(p):
    return torch.empty(p.workspace_size(), dtype=torch.uint8, device="cuda")


def receivers(p):
    return p.run_receivers().cpu().numpy()


def say(what, form):
    print(f"{what}: order {form[0]} source kind {form[1]} {form[2]} {form[3]}", flush=True)


@pytest.mark.parametrize("form", FORMS)
def test_two_workspaces_in_turn(form):
    p, E = plan(*form)
    say("two workspaces in turn", form)
    nt, a, b = p.info.nt, buffer(p), buffer(p)
    p.use_workspace(a)
    p.run_begin()
    p.run_steps(3)
    p.use_workspace(b)
    p.run_begin()
    p.run_steps(2)
    p.use_workspace(a)
    p.run_steps(nt - 3)
    Ea = receivers(p)
    p.use_workspace(b)
    p.run_steps(nt - 2)
    assert np.array_equal(Ea, E) and np.array_equal(receivers(p), E)


@pytest.mark.parametrize("form", FORMS)
def test_full_run_on_another_workspace_between(form):
    p, E = plan(*form)
    say("a full run between", form)
    a, b = buffer(p), buffer(p)
    p.use_workspace(a)
    p.run_begin()
    p.run_steps(6)
    p.use_workspace(b)
    assert np.array_equal(p.forward().cpu().numpy(), E)
    p.use_workspace(a)
    p.run_steps(p.info.nt - 6)
    assert np.array_equal(receivers(p), E)


@pytest.mark.parametrize("form", FORMS)
def test_workspace_put_back_by_a_copy(form):
    p, E = plan(*form)
    say("workspace put back", form)
    a = buffer(p)
    p.use_workspace(a)
    p.run_begin()
    p.run_steps(4)
    saved = a.clone()
    p.run_steps(33)
    a.copy_(saved)
    p.run_steps(p.info.nt - 4)
    assert np.array_equal(receivers(p), E)


@pytest.mark.parametrize("form", [f for f in FORMS if f[3].get("graph_steps") == 0])
def test_captured_call_replayed(form):
    """An odd number of steps, captured by the caller: 25 replays are the run,
    and replays past its end add nothing."""
    p, E = plan(*form)
    say("captured call", form)
    a = buffer(p)
    p.use_workspace(a)
    p.run_begin()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        p.run_steps(3, stream=stream)
    for t in range(25):
        g.replay()
        if t % 8 == 0:                       # eager work of the program between replays
            torch.cuda.synchronize()
            torch.ones(1000, device="cuda").sum().item()
    assert np.array_equal(receivers(p), E)
    g.replay()
    assert np.array_equal(receivers(p), E)


@pytest.mark.parametrize("form", FORMS)
def test_steps_past_the_end_add_nothing(form):
    p, E = plan(*form)
    say("steps past the end", form)
    a, b = buffer(p), buffer(p)
    p.use_workspace(a)
    p.run_begin()
    p.run_steps(p.info.nt)
    p.use_workspace(b)
    p.run_begin()                            # the plan's own count starts again
    p.use_workspace(a)
    p.run_steps(41)
    assert np.array_equal(receivers(p), E)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("between", [2, "full"])
def test_volumes_of_two_workspaces(form, between):
    """The steps that close a transform block follow the workspace: a run with
    a volume left inside a block, another one between, then on to the end."""
    p, _ = plan(*form)
    say(f"volumes of two workspaces, {between} steps between", form)
    nt, ref = p.info.nt, p.volume_buffer()
    p.forward(vol=ref, want_volume=True)
    ref = p.volume_export(ref).cpu().numpy()
    a, b, va, vb = buffer(p), buffer(p), p.volume_buffer(), p.volume_buffer()
    p.use_workspace(a)
    p.run_begin(va)
    p.run_steps(13, va)
    p.use_workspace(b)
    if between == "full":
        p.forward(vol=vb, want_volume=True)
    else:
        p.run_begin(vb)
        p.run_steps(between, vb)
    p.use_workspace(a)
    p.run_steps(nt - 13, va)
    if between != "full":
        p.use_workspace(b)
        p.run_steps(nt - between, vb)
    p.use_workspace(a)
    p.run_flush(va)
    p.use_workspace(b)
    p.run_flush(vb)
    for v in (va, vb):
        assert np.array_equal(p.volume_export(v).cpu().numpy(), ref)


@pytest.mark.parametrize("form", FORMS)
def test_volume_beside_a_run_without(form):
    """Receiver-only steps of another workspace between those of a run with a
    volume."""
    p, E = plan(*form)
    say("a volume beside a run without", form)
    nt, ref = p.info.nt, p.volume_buffer()
    p.forward(vol=ref, want_volume=True)
    a, b, va = buffer(p), buffer(p), p.volume_buffer()
    p.use_workspace(b)
    p.run_begin()
    p.use_workspace(a)
    p.run_begin(va)
    for k in (13, 6, nt - 19):
        p.use_workspace(a)
        p.run_steps(k, va)
        p.use_workspace(b)
        p.run_steps(3)
    p.run_steps(nt - 9)
    assert np.array_equal(receivers(p), E)
    p.use_workspace(a)
    p.run_flush(va)
    assert torch.equal(p.volume_export(va), p.volume_export(ref))
