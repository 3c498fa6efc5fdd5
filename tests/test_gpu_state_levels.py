"""States without the second pair of levels (2D FP32): where memory is short
or the caller asks for it, in batches beside states that have one, in the
server and in the survey calls.  Same bits always."""
from __future__ import annotations

import ctypes

import pytest

import fd_inputs as fi

pytestmark = pytest.mark.gpu


def _problem(nz, nx, nt, seed=4):
    return fi.Problem(name="lv", ndim=2, nz=nz, ny=1, nx=nx, dh=10.0, dt=1e-3, nt=nt, src=(nz // 2, 0, nx // 2),
                      receivers=fi.Receivers(1, 0, 0, 1, 1, nx, 1, 1, 1), f0=30.0, sponge_width=4,
                      sponge_faces=0x3E, velocity_kind="random", velocity_seed=seed)


def _launches(call, copies=False):
    """Nodes (or only the copies) of the graph that `call(stream)` records;
    nothing runs."""
    import torch
    path = next(w for line in open("/proc/self/maps") for w in line.split() if "libamdhip64" in w)
    hip = ctypes.CDLL(path)
    s = torch.cuda.Stream()
    raw = ctypes.c_void_p(s.cuda_stream)
    g, n = ctypes.c_void_p(), ctypes.c_size_t(0)
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(raw, 1) == 0      # thread-local mode
    call(s)
    assert hip.hipStreamEndCapture(raw, ctypes.byref(g)) == 0
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0
    nodes, kind = (ctypes.c_void_p * max(1, n.value))(), ctypes.c_int()
    assert hip.hipGraphGetNodes(g, nodes, ctypes.byref(n)) == 0
    memcpys = 0
    for node in nodes[:n.value]:
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        memcpys += kind.value == 1
    assert hip.hipGraphDestroy(g) == 0
    return memcpys if copies else n.value


def _flight(nz, nx, nt, second_pair=True, seed=4):
    import torch
    from helpers import setup
    model, _, shot = setup(_problem(nz, nx, nt, seed))
    state = model.new_state(second_pair=second_pair)
    state.begin(shot)
    return model, state, shot, torch.empty((shot.nt, shot.nrec), device="cuda")


@pytest.mark.parametrize("storage", [0, 1])
def test_a_device_without_room_for_the_second_pair(monkeypatch, storage):
    import torch
    import paper_2311_05038_amd as fd
    from helpers import setup
    p = _problem(70, 140, 21)
    model, full, shot = setup(p, storage=storage)
    ref = model.run_shot(full, shot)
    least = model.least_state_bytes
    assert least < model.sizes.state if storage == 0 else least == model.sizes.state
    real = fd._alloc

    def short(nbytes, device):
        if nbytes > least or storage != 0:
            raise torch.cuda.OutOfMemoryError("short")
        return real(nbytes, device)
    monkeypatch.setattr(fd, "_alloc", short)
    if storage != 0:    # 16-bit states have no second pair to do without
        with pytest.raises(torch.cuda.OutOfMemoryError):
            model.new_state()
        return
    state = model.new_state()
    assert state.buf.numel() == least
    assert torch.equal(model.run_shot(state, shot), ref)
    assert torch.equal(state.wavefield(0), full.wavefield(0))


@pytest.mark.parametrize("chunk", [1, 2, 3, 13])
def test_a_batch_of_both_kinds(chunk):
    import torch
    import paper_2311_05038_amd as fd
    sizes = [(90, 130, 31, True), (64, 64, 17, False), (200, 70, 40, False), (33, 300, 25, True), (5, 9, 40, True)]
    mixed = [_flight(*a, seed=i) for i, a in enumerate(sizes)]
    while any(f[1].next < f[2].nt for f in mixed):
        fd.step_batch(mixed, chunk)
    for f in mixed:
        st = f[0].new_state()
        tr = f[0].run_shot(st, f[2])
        assert torch.equal(f[3], tr) and torch.equal(st.wavefield(0), f[1].wavefield(0))
        assert torch.equal(st.wavefield(1), f[1].wavefield(1))


def test_a_state_without_a_second_pair_keeps_others_their_launches():
    import paper_2311_05038_amd as fd
    lone = [_flight(256, 256, 200)]
    alone = _launches(lambda s: fd.step_batch(lone, 25, stream=s))
    single = [_flight(200, 300, 200, second_pair=False)]
    steps = _launches(lambda s: fd.step_batch(single, 25, stream=s))
    assert alone < 25 and steps == 25
    both = [_flight(256, 256, 200), _flight(200, 300, 200, second_pair=False)]
    assert _launches(lambda s: fd.step_batch(both, 25, stream=s)) == alone + steps


def test_the_server_within_a_budget_between_the_two_sizes():
    import torch
    import paper_2311_05038_amd as fd
    from helpers import grid_of, receivers_of
    from paper_2311_05038_amd.serve import Request, Scheduler, TorchDevice
    p = _problem(120, 200, 60)

    def inputs(req):
        v = torch.from_numpy(p.velocity().ravel()).cuda()
        return grid_of(p), v, fd.Shot(p.src, torch.from_numpy(p.wavelet()).cuda(), receivers_of(p))
    dev = TorchDevice(inputs, keep_traces=True)
    reqs = [Request(i, 0.0, p.nz, p.nx, p.nt) for i in range(3)]
    full, least = dev.footprint(reqs[0]), dev.least_footprint(reqs[0])
    assert full - least == 2 * 120 * 256 * 4
    out = Scheduler(dev, hbm_budget=(full + least) // 2).run(reqs)
    assert all(o.status == "ok" for o in out.values())
    model = fd.Model(grid_of(p), torch.from_numpy(p.velocity().ravel()).cuda())
    ref = model.run_shot(model.new_state(), inputs(None)[2])
    for o in out.values():
        assert torch.equal(o.result, ref)


@pytest.mark.parametrize("call", ["gradient", "image"])
def test_survey_calls_hold_no_more_than_with_two_levels(call):
    """The second pairs must not add to a survey's peak: the states are given
    back before the work buffers are made."""
    import torch
    import paper_2311_05038_amd as fd
    from helpers import grid_of, receivers_of
    from paper_2311_05038_amd.autograd import l2_misfit_gradient, rtm_image
    p = _problem(600, 640, 24)
    grid = grid_of(p)
    v = torch.from_numpy(p.velocity().ravel()).cuda()
    w = torch.from_numpy(p.wavelet()).cuda()
    shots = [fd.Shot((2, 0, 50 + 60 * i), w, receivers_of(p)) for i in range(4)]
    every = 8
    model = fd.Model(grid, v)
    sz = model.sizes_for(p.nt, every)
    data = torch.zeros((4, p.nt, p.receivers.count), device="cuda")
    torch.cuda.synchronize()
    base = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    if call == "gradient":
        l2_misfit_gradient(v, grid, shots, data, ckpt_every=every)
    else:
        rtm_image(v, grid, shots, data, ckpt_every=every)
    peak = torch.cuda.max_memory_allocated() - base
    least = model.least_state_bytes + sz.checkpoints + sz.adjoint_work
    slack = 4 * data.numel() * 4 + 8 * p.ncells + 2 * sz.model    # traces, sums, the call's own model
    assert peak <= 4 * least + slack
