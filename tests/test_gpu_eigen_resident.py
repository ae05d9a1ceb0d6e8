"""The plain eigen mode's resident iterations and its Ritz values on the device
where they can go wrong: tiles of unequal size, every number of rows per thread,
Krylov dimensions about the checkpoints (every 64 iterations, one launch each),
windows with as many values as the device solves and more.

With tol above the spectrum's width all Ritz values of T_j are one cluster: its
mean is tr(T_j) / j and its bound |beta_j|, so the call returns a checkpoint's
trace and beta, to which every site of every iteration contributes."""
import numpy as np
import pytest

import harness as hz
from paper_1407_7370_amd import packets

pytestmark = pytest.mark.gpu

C = 137.036
EPS = 2.0 ** -52
WIDE = 1e9


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


def box(nx, ny, bcx, bcy, fields, h=0.1):
    p = dict(nx=nx, ny=ny, x_min=-0.5 * nx * h, x_max=0.5 * nx * h, y_min=-0.5 * ny * h, y_max=0.5 * ny * h, bc_x=bcx,
             bc_y=bcy, mass=1.0, c=C, charge=-1.0, bz=0.0, pot_kind=0, pot_z=0.0, pot_a=0.0, pulse_kind=0,
             pulse_e=(0.0, 0.0), a0=0.0, omega=0.0, t_pulse=1.0, coef=None)
    if fields:
        p.update(bz=0.6, pot_kind=1, pot_z=1.0, pot_a=1.0)
    return p


def check_traces(torch, orc, prob, psi0, k, n_wanted):
    """The smallest |beta_j| of the checkpoints seen and its block's mean value."""
    from paper_1407_7370_amd.binding import Propagator
    prop = Propagator(prob, 1, "fp64", k_eigen=k)
    ev, bd = prop.eigen(torch.from_numpy(psi0).cuda(), k, -WIDE, WIDE, 4 * WIDE, n_wanted=n_wanted)
    prop.close()
    keff, al, be = orc.lanczos_plain(prob, psi0, k)
    assert keff == k
    marks = [k] if k <= 64 else [64] if n_wanted == 1 else [*range(64, k, 64), k]
    j = min(marks, key=lambda j: be[j - 1])
    # a random start has no converged values in these few iterations, so alpha
    # and beta agree to the rounding of H's norm times a modest growth
    norm = C * C + 2 * C / 0.1 + 20 * C
    assert len(ev) == 1
    assert abs(ev[0] - al[:j].mean()) <= 1e4 * EPS * norm
    assert abs(bd[0] - be[j - 1]) <= 1e4 * EPS * norm


# one tile, unequal tiles, and rows per thread 1, 2, 3, 4 (two tile buffers), 6, 8
@pytest.mark.parametrize("nx,ny,bcx,bcy", [(33, 17, 0, 0), (131, 77, 1, 1), (16, 30, 1, 0), (290, 201, 1, 0), (400, 390, 0, 0),
                                           (512, 500, 0, 1), (600, 610, 1, 1), (720, 700, 0, 0), (850, 833, 1, 0)])
@pytest.mark.parametrize("fields", [False, True])
def test_recurrence_vs_oracle(torch_cuda, orc, nx, ny, bcx, bcy, fields):
    say(f"eigen resident {nx}x{ny} bc {bcx}{bcy} fields={fields}")
    prob = box(nx, ny, bcx, bcy, fields)
    check_traces(torch_cuda, orc, prob, packets.random_spinor(prob, nx), 70, 2)


# dimensions about a checkpoint; up to 64 values are solved on the device (the
# first checkpoint has exactly 64), more on the host
@pytest.mark.parametrize("k,n_wanted", [(1, 1), (2, 1), (63, 1), (64, 1), (65, 1), (65, 2), (66, 2), (128, 2), (129, 2)])
def test_checkpoints_vs_oracle(torch_cuda, orc, k, n_wanted):
    say(f"eigen resident checkpoints k={k} wanted {n_wanted}")
    prob = box(96, 90, 1, 0, True)
    check_traces(torch_cuda, orc, prob, packets.random_spinor(prob, k), k, n_wanted)


@pytest.mark.parametrize("k", [64, 300])
def test_breakdown(torch_cuda, orc, k):
    """A plane wave's Krylov space has two dimensions: both eigenvalues, from the
    host's solve of the last T; and no value of a zero state."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    prob = box(40, 36, 1, 1, False)
    x = np.arange(40)[None, :] * (2 * np.pi * 3 / 40) + np.arange(36)[:, None] * (2 * np.pi * 5 / 36)
    psi0 = np.zeros((2, 36, 40), dtype=np.complex128)
    psi0[0] = np.exp(1j * x)
    say(f"eigen resident breakdown k={k}")
    prop = Propagator(prob, 1, "fp64", k_eigen=k)
    ev, _ = prop.eigen(torch.from_numpy(psi0).cuda(), k, -WIDE, WIDE, 1e-6, n_wanted=8)
    p2 = (np.sin(2 * np.pi * 3 / 40) / 0.1) ** 2 + (np.sin(2 * np.pi * 5 / 36) / 0.1) ** 2
    e = np.sqrt(C ** 4 + C * C * p2)
    assert np.allclose(ev, [-e, e], rtol=64 * EPS, atol=0)
    ev0, _ = prop.eigen(torch.zeros(2, 36, 40, dtype=torch.complex128, device="cuda"), k, -WIDE, WIDE, 1e-6, n_wanted=8)
    assert len(ev0) == 0
    bad = torch.from_numpy(psi0).cuda()
    bad[1, 3, 7] = float("nan")
    with pytest.raises(RuntimeError, match="non-finite"):
        prop.eigen(bad, k, -WIDE, WIDE, 1e-6, n_wanted=8)
    again, _ = prop.eigen(torch.from_numpy(psi0).cuda(), k, -WIDE, WIDE, 1e-6, n_wanted=8)
    prop.close()
    assert np.array_equal(again, ev)


@pytest.mark.parametrize("e_lo,e_hi", [(-1e300, 1e300), (-1e30, 1e30), (0.0, 1e30), (0.0, 1e300), (-1e25, 0.0)])
def test_windows_far_beyond_the_spectrum(torch_cuda, orc, e_lo, e_hi):
    """Finite bounds far outside the spectrum stand for open ends: the values of
    the first checkpoint's T_64 in the window (one cluster each with tol above the
    spectrum's width), as numpy has them for the oracle's T_64, and bit for bit
    those of a window that ends just outside the spectrum."""
    from paper_1407_7370_amd.binding import Propagator
    say(f"eigen window ({e_lo}, {e_hi}]")
    prob = box(96, 90, 1, 0, True)
    psi0 = packets.random_spinor(prob, 11)
    k = 130
    prop = Propagator(prob, 1, "fp64", k_eigen=k)
    psi = torch_cuda.from_numpy(psi0).cuda()
    ev, bd = prop.eigen(psi, k, e_lo, e_hi, 4 * WIDE, n_wanted=1)
    ev2, bd2 = prop.eigen(psi, k, max(e_lo, -WIDE), min(e_hi, WIDE), 4 * WIDE, n_wanted=1)
    prop.close()
    _, al, be = orc.lanczos_plain(prob, psi0, 64)
    w, z = np.linalg.eigh(np.diag(al[:64]) + np.diag(be[:63], 1) + np.diag(be[:63], -1))
    inside = (w > e_lo) & (w <= e_hi)
    # no value of a random start's T_64 has converged: alpha and beta agree to the
    # rounding of H's norm times a modest growth, its eigenvectors to that over the
    # distance of neighbouring values
    err = 1e4 * EPS * (C * C + 2 * C / 0.1 + 20 * C)
    assert len(ev) == 1 and np.abs(w).min() > 1.0
    assert abs(ev[0] - w[inside].mean()) <= err
    assert abs(bd[0] - be[63] * np.linalg.norm(z[-1, inside])) <= err * (1.0 + be[63] / np.diff(w).min())
    assert np.array_equal(ev, ev2) and np.array_equal(bd, bd2)


def test_returns_with_its_work_done(torch_cuda):
    """A checkpoint with more values than the device solves is solved on the host
    beside the next passes; when it has all the wanted values (here the one at 128,
    within about 3 ms, beside 62 passes of about 0.35 ms) and no other checkpoint follows,
    the call still waits for those passes, whose failures would be its own."""
    from paper_1407_7370_amd.binding import Propagator
    torch = torch_cuda
    say("eigen 4096x4096 returns with its work done")
    prob = dict(box(4096, 4096, 0, 0, True), bz=0.0)
    psi = torch.from_numpy(packets.gaussian_packet(prob, 1.0, (0.0, 0.0))).cuda()
    prop = Propagator(prob, 1, "fp64", k_eigen=190)
    prop.eigen(psi, 190, -WIDE, WIDE, 0.15, n_wanted=1)
    ev, _ = prop.eigen(psi, 190, -WIDE, WIDE, 0.15, n_wanted=1)
    done = torch.cuda.current_stream().query()
    at64, _ = prop.eigen(psi, 64, -WIDE, WIDE, 0.15, n_wanted=1)
    prop.close()
    assert len(ev) == 1 and len(at64) == 0
    assert done
