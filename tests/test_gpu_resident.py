"""The resident time steps (one launch for many steps of a grid that fits the
chip's LDS) where they can go wrong: the smallest grids, tiles of unequal size,
every number of rows per thread, both tile buffer schemes, periodic images that
are the tile itself, more steps than one launch takes, several contexts and
streams at once."""
import time

import numpy as np
import pytest

import harness as hz
from paper_1407_7370_amd import packets

pytestmark = pytest.mark.gpu

C = 137.036
EPS = 2.0 ** -52


def say(msg):
    print(f"[gpu case] {msg}", flush=True)


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def box(nx, ny, bcx, bcy, h=0.1, **kw):
    p = dict(nx=nx, ny=ny, x_min=-0.5 * nx * h, x_max=0.5 * nx * h, y_min=-0.5 * ny * h, y_max=0.5 * ny * h, bc_x=bcx,
             bc_y=bcy, mass=1.0, c=C, charge=-1.0, bz=0.0, pot_kind=0, pot_z=0.0, pot_a=0.0, pulse_kind=0,
             pulse_e=(0.0, 0.0), a0=0.0, omega=0.0, t_pulse=1.0, coef=None)
    p.update(kw)
    return p


FIELDS = dict(bz=0.6, pot_kind=1, pot_z=1.0, pot_a=1.0)


# one tile (also its own periodic neighbour), tiles of four sites, unequal tiles
@pytest.mark.parametrize("nx,ny,bcx,bcy", [(3, 3, 1, 1), (3, 4, 0, 1), (16, 5, 1, 0), (33, 17, 0, 0), (131, 77, 1, 1),
                                           (9, 400, 0, 1), (290, 201, 1, 0)])
@pytest.mark.parametrize("fields", [False, True])
def test_small_grids_vs_oracle(torch_cuda, orc, nx, ny, bcx, bcy, fields):
    """66 steps (a launch takes 64) with a laser pulse, m = 6."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(nx, ny, bcx, bcy, pulse_kind=1, pulse_e=(0.6, 0.8), a0=30.0, omega=1.0, t_pulse=0.02,
               **(FIELDS if fields else {}))
    psi0 = packets.random_spinor(prob, nx) * 1e-2 + packets.gaussian_packet(prob, 1.0, (1.0, -2.0))
    n, dt, m = 66, 1e-4, 6
    say(f"resident {nx}x{ny} bc {bcx}{bcy} fields={fields}")
    prop = Propagator(prob, m, "fp64")
    psi = torch.from_numpy(psi0).cuda()
    st = prop.step(psi, 0.0, dt, n)
    prop.close()
    ref, rst = orc.propagate(prob, psi0, 0.0, dt, n, m)
    assert np.array_equal(st["k_eff"], rst["k_eff"])
    # rounding of the step phase |dt H| per step, 64 roundings of it allowed
    phase = dt * (C * C + 2 * C / 0.1 + 10 * C)
    assert hz.rel_l2(psi.cpu().numpy(), ref) <= 64 * n * phase * EPS
    np.testing.assert_allclose(st["norm2"], rst["norm2"], rtol=64 * n * EPS)


# rows per thread 2, 3, 4 (two tile buffers), 6, 8, 10 (one), and beyond the path
@pytest.mark.parametrize("nx,ny", [(400, 390), (512, 500), (600, 610), (720, 700), (850, 833), (1024, 1024),
                                   (1100, 1050)])
@pytest.mark.parametrize("prec,fields", [("fp64", False), ("fp64", True), ("mixed", False), ("mixed", True)])
def test_rows_per_thread_vs_sweeps(torch_cuda, nx, ny, prec, fields):
    """Against the second-run variant, whose iterations are sweep launches."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(nx, ny, 1, 0, pulse_kind=1, pulse_e=(0.6, 0.8), a0=30.0, omega=1.0, t_pulse=0.02,
               **(FIELDS if fields else {}))
    gen = torch.Generator(device="cuda").manual_seed(nx + ny)
    psi0 = torch.randn((2, ny, nx, 2), generator=gen, dtype=torch.float64, device="cuda")
    psi0 = torch.view_as_complex(psi0).contiguous() / np.sqrt(4.0 * nx * ny)
    n, dt, m = 3, 1e-4, 8
    say(f"resident {nx}x{ny} {prec} fields={fields} against sweeps")
    prop = Propagator(prob, m, prec)
    a, b = psi0.clone(), psi0.clone()
    sa = prop.step(a, 0.0, dt, n)
    sb = prop.step(b, 0.0, dt, n, lowmem=True)
    prop.close()
    dist = float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))
    phase = dt * (C * C + 2 * C / 0.1 + 40 * C)
    tol = 64 * n * phase * EPS
    if prec == "mixed":  # each run lies within its own storage bound
        tol += sa["cum_round_bound"][-1] + sb["cum_round_bound"][-1]
        np.testing.assert_allclose(sa["round_bound"], sb["round_bound"], rtol=1e-6)
    assert dist <= tol
    assert np.array_equal(sa["k_eff"], sb["k_eff"])
    np.testing.assert_allclose(sa["norm2"], sb["norm2"], rtol=64 * n * EPS + (1e-7 if prec == "mixed" else 0.0))


def test_contexts_and_streams_at_once(torch_cuda):
    """Two contexts of different grids on two streams, called from two threads,
    equal their runs alone bit for bit."""
    import threading

    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    grids = [(512, 500), (130, 90)]
    say("resident steps on two streams")
    alone, jobs = [], []
    for nx, ny in grids:
        prob = box(nx, ny, 0, 0, **FIELDS)
        psi0 = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (1.0, 2.0))).cuda()
        stream = torch.cuda.Stream()
        prop = Propagator(prob, 9, "fp64", stream=stream)
        torch.cuda.synchronize()
        ref = psi0.clone()
        torch.cuda.synchronize()
        prop.step(ref, 0.0, 2e-4, 40)
        alone.append(ref)
        jobs.append((prop, psi0))
    out = [None, None]

    def work(i):
        prop, psi0 = jobs[i]
        res = []
        for _ in range(5):
            x = psi0.clone()
            torch.cuda.synchronize()
            prop.step(x, 0.0, 2e-4, 40)
            res.append(x)
        out[i] = res

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert all(torch.equal(x, alone[i]) for x in out[i])
        jobs[i][0].close()


def test_adjoint_without_kept_bases(torch_cuda):
    """One segment too long for its Krylov bases to be kept (400 steps of 512^2,
    m = 12: 37 GB): the backward pass rebuilds them step by step, and loss and
    gradient equal those of short segments bit for bit."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    cfg = packets.fourier_pulse_512()
    psi0 = torch.from_numpy(packets.initial_state(cfg)).cuda()
    prop = Propagator(cfg["problem"], cfg["m"], "fp64")
    res = []
    for ckpt in (400, 50):
        say(f"adjoint 512x512 400 steps, segments of {ckpt}")
        res.append(prop.adjoint(psi0, 0.0, cfg["dt"], 400, ckpt, 9))
    prop.close()
    assert res[0][0] == res[1][0]
    assert np.array_equal(res[0][1], res[1][1])


@pytest.mark.parametrize("steps,ckpts", [(20, (1, 2, 3, 7, 19, 20)), (140, (140, 70, 133))])
def test_adjoint_groups_of_backward_steps(torch_cuda, steps, ckpts):
    """The backward steps of a segment run in groups that double in length, in the
    slots of the steps before them (140: a group longer than a launch): the loss and
    the gradient do not depend on the segments, bit for bit, and agree with those of
    single steps as sweeps."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(120, 100, 1, 0, pulse_kind=2, t_pulse=0.5, coef=np.array([10.0, -5.0, 3.0, 8.0]), **FIELDS)
    psi0 = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (1.0, -2.0))).cuda()
    prop = Propagator(prob, 7, "fp64")
    res = []
    for ckpt in ckpts:
        say(f"adjoint 120x100 {steps} steps, segments of {ckpt}")
        res.append(prop.adjoint(psi0, 0.0, 1e-3, steps, ckpt, 15))
    prop.set_wait(0.0)
    loss, grad = prop.adjoint(psi0, 0.0, 1e-3, steps, ckpts[-1], 15)
    prop.close()
    for r in res[1:]:
        assert r[0] == res[0][0]
        assert np.array_equal(r[1], res[0][1])
    # both ways round like the step phase |dt H| per step, 64 roundings of it allowed,
    # on loss terms of up to |p| ~ 2 and |x| ~ 6 and their gradients
    phase = 1e-3 * (C * C + 2 * C / 0.1 + 10 * C)
    assert abs(loss - res[0][0]) <= 64 * steps * phase * EPS * 10.0
    assert np.max(np.abs(grad - res[0][1])) <= 64 * steps * phase * EPS * max(np.max(np.abs(grad)), 10.0)


def test_adjoint_with_one_slot(torch_cuda):
    """Two segments whose bases fit in the kept store one at a time (512^2, m = 12,
    200 steps: 20 GB each): the second is run again in the slot that the first leaves."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    cfg = packets.fourier_pulse_512()
    psi0 = torch.from_numpy(packets.initial_state(cfg)).cuda()
    prop = Propagator(cfg["problem"], cfg["m"], "fp64")
    res = []
    for ckpt in (200, 50):
        say(f"adjoint 512x512 400 steps, segments of {ckpt}")
        res.append(prop.adjoint(psi0, 0.0, cfg["dt"], 400, ckpt, 9))
    prop.close()
    assert res[0][0] == res[1][0]
    assert np.array_equal(res[0][1], res[1][1])


def test_contexts_on_one_workspace(torch_cuda, orc):
    """Two grids' contexts on the same workspace memory, used in turn: words that
    one leaves in the other's exchange buffers are never taken for its own."""
    from paper_1407_7370_amd import binding
    torch = torch_cuda
    dt, m, n = 1e-4, 6, 3
    probs = [box(64, 60, 1, 1), box(200, 170, 0, 0, **FIELDS)]
    params = [binding.make_params(p, m, binding.DL_PREC_FP64) for p in probs]
    size = max(binding.dirac_lanczos_workspace_bytes(p[0]) for p in params)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    ctxs = [binding.dirac_lanczos_init(p[0], ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream) for p in params]
    psi0 = [packets.random_spinor(p, 3) * 1e-2 + packets.gaussian_packet(p, 1.0, (1.0, -2.0)) for p in probs]
    psi = [torch.from_numpy(p).cuda() for p in psi0]
    for turn in range(4):
        for c, p in zip(ctxs, psi):
            say(f"one workspace, turn {turn}, {tuple(p.shape)}")
            # (synchronous calls: asynchronous ones keep their status in the workspace)
            assert binding.dirac_lanczos_step(c, p.data_ptr(), turn * n * dt, dt, n, (binding.DlStepStat * n)()) == 0
    for c in ctxs:
        binding.dirac_lanczos_destroy(c)
    phase = dt * (C * C + 2 * C / 0.1 + 10 * C)
    for prob, p, p0 in zip(probs, psi, psi0):
        ref, _ = orc.propagate(prob, p0, 0.0, dt, 4 * n, m)
        assert hz.rel_l2(p.cpu().numpy(), ref) <= 64 * 4 * n * phase * EPS


@pytest.mark.parametrize("nx,ny", [(64, 60), (300, 280)])  # sums read directly, and through leaders
@pytest.mark.parametrize("ahead", [1, 2])
@pytest.mark.parametrize("call", ["step", "async", "eigen"])
def test_foreign_words_in_the_workspace(torch_cuda, nx, ny, ahead, call):
    """What another user of the memory left in a workspace between two calls never
    passes for an exchanged word: every word holds the epoch (upper 32 bits) that
    the next launch waits for first or second, and the results stay bit for bit
    those of a fresh workspace."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(nx, ny, 1, 0, **FIELDS)
    psi0 = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (1.0, -2.0))).cuda()

    def run(prop):
        if call == "eigen":
            ev, bd = prop.eigen(psi0, 100, -1e9, 1e9, 4e9, n_wanted=2)
            return torch.tensor(np.concatenate([ev, bd]))
        x = psi0.clone()
        if call == "async":
            prop.step_async(x, 0.0, 1e-4, 5)
            prop.wait()
        else:
            prop.step(x, 0.0, 1e-4, 5)
        return x

    say(f"foreign words {nx}x{ny} ahead {ahead} {call}")
    prop = Propagator(prob, 6, "fp64", k_eigen=100)
    ref = run(prop)
    start = prop.ws_ptr - prop.workspace.data_ptr()
    words = prop.workspace[start:start + prop.ws_bytes // 8 * 8].view(torch.int64)
    sums = words[:7680]  # the workspace starts with the words of the sums: 0 or an epoch
    last = int((sums >> 32).max())
    assert 0 < last < 2 ** 31 - 2
    # (asynchronous calls keep their status in the workspace: there only the sums)
    (sums if call == "async" else words).fill_(((last + ahead) << 32) | 0x3F800000)
    again = run(prop)
    prop.close()
    assert torch.equal(again, ref)


def test_wait_limit_goes_on_in_sweeps(torch_cuda):
    """A resident launch whose workgroups wait longer than the limit (here one tick,
    so no step of it completes) leaves the rest of the call, and later calls, to
    sweeps, with the bits of a context that runs sweeps only; an asynchronous call
    reports it.  A new limit brings the resident launches back."""
    from paper_1407_7370_amd import binding
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(400, 390, 1, 0, pulse_kind=2, t_pulse=0.05, coef=np.array([10.0, -5.0, 3.0, 8.0]), **FIELDS)
    psi0 = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (1.0, -2.0))).cuda()
    n, dt, k = 5, 1e-4, 130

    def run(prop):
        x = psi0.clone()
        st = prop.step(x, 0.0, dt, n)
        ev, bd = prop.eigen(psi0, k, -1e9, 1e9, 4e9, n_wanted=2)
        loss, grad = prop.adjoint(psi0, 0.0, dt, 7, 3, 9)
        return x, st, ev, bd, loss, grad

    def same(a, b):
        assert torch.equal(a[0], b[0])
        for key in ("k_eff", "err_est", "cum_bound", "norm2"):
            assert np.array_equal(a[1][key], b[1][key]), key
        assert all(np.array_equal(p, q) for p, q in zip(a[2:], b[2:]))

    prop = Propagator(prob, 6, "fp64", k_eigen=k)
    say("wait limit: resident")
    resident = run(prop)
    say("wait limit: sweeps only")
    prop.set_wait(0.0)
    sweeps = run(prop)
    assert not torch.equal(sweeps[0], resident[0])  # (another order of the sums)
    calls = [lambda: prop.step(psi0.clone(), 0.0, dt, n), lambda: prop.eigen(psi0, k, -1e9, 1e9, 4e9, n_wanted=2),
             lambda: prop.adjoint(psi0, 0.0, dt, 7, 3, 9)]
    for i, call in enumerate(calls):
        say(f"wait limit: one tick, call {i}")
        prop.set_wait(1e-8)
        call()  # the context runs sweeps after this
        same(run(prop), sweeps)
    prop.set_wait(1e-8)
    same(run(prop), sweeps)
    say("wait limit: one tick, asynchronous")
    prop.set_wait(1e-8)
    x = psi0.clone()
    prop.step_async(x, 0.0, dt, n)
    with pytest.raises(binding.DlError) as ei:
        prop.wait()
    assert ei.value.status == binding.DL_ERR_DEVICE
    assert torch.equal(x, psi0)
    same(run(prop), sweeps)
    say("wait limit: resident again")
    prop.set_wait(20.0)
    same(run(prop), resident)
    for bad in (-1.0, float("nan"), 1e9):
        with pytest.raises(binding.DlError) as ei:
            prop.set_wait(bad)
        assert ei.value.status == binding.DL_ERR_INVALID
    prop.close()


def test_timing_across_the_end_of_resident_steps(torch_cuda):
    """The times of resident steps are kept when the context goes over to sweeps
    while timing is on."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(400, 390, 1, 0, **FIELDS)
    x = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (1.0, -2.0))).cuda()
    prop = Propagator(prob, 9, "fp64")
    say("timing across the end of resident steps")
    prop.step(x, 0.0, 1e-4, 2)
    prop.timing(True)
    prop.step(x, 0.0, 1e-4, 50)
    resident = {k: ms for k, (_, ms) in prop.timing(False).items()}
    prop.timing(True)
    t0 = time.perf_counter()
    prop.step(x, 0.0, 1e-4, 50)
    prop.set_wait(0.0)
    prop.step(x, 0.0, 1e-4, 1)
    wall = 1e3 * (time.perf_counter() - t0)
    both = prop.timing(False)
    prop.close()
    print(resident, both, wall, flush=True)
    assert sum(resident.values()) > 0.5
    # the same fifty resident steps and a step of sweeps, within the wall time
    assert sum(ms for _, ms in both.values()) <= 1.05 * wall
    assert sum(ms for _, ms in both.values()) >= 0.5 * sum(resident.values())
    assert sum(n for n, _ in both.values()) == 51 * (9 + 2)


@pytest.mark.parametrize("call", ["step", "eigen", "adjoint"])
def test_synchronous_calls_report_an_asynchronous_time_out(torch_cuda, call):
    """The next synchronous call reports a time-out of an asynchronous one and does
    nothing else; the call after it runs."""
    from paper_1407_7370_amd import binding
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(400, 390, 1, 0, pulse_kind=2, t_pulse=0.05, coef=np.array([10.0, -5.0, 3.0, 8.0]), **FIELDS)
    psi0 = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (1.0, -2.0))).cuda()
    prop = Propagator(prob, 6, "fp64", k_eigen=70)
    run = {"step": lambda: prop.step(psi0.clone(), 0.0, 1e-4, 2), "eigen": lambda: prop.eigen(psi0, 70, -1e9, 1e9, 4e9),
           "adjoint": lambda: prop.adjoint(psi0, 0.0, 1e-4, 3, 2, 9)}[call]
    say(f"time-out of an asynchronous call reported by {call}")
    prop.set_wait(1e-8)
    x = psi0.clone()
    prop.step_async(x, 0.0, 1e-4, 3)
    with pytest.raises(binding.DlError) as ei:
        run()
    assert ei.value.status == binding.DL_ERR_DEVICE and "asynchronous" in str(ei.value)
    assert torch.equal(x, psi0)
    run()
    prop.close()
