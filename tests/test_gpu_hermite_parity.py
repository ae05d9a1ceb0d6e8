"""The Hermite recurrence in the parity basis (n = 32, 64; n = 16, 48 keep the
plain basis) with a magnetic field, which couples the parities, and the Ritz
values computed on the device: against the oracle, and against the host's Ritz
step where a call is beyond the device's (long recurrences, windows with many
values)."""
import numpy as np
import pytest

import harness as hz
from paper_1407_7370_amd import packets

pytestmark = pytest.mark.gpu

C = 137.036
MC2 = C * C


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


def say(msg):
    print(f"[gpu case] {msg}", flush=True)


def eigen(torch, hp, start, k, lo, hi, tol, wanted=64):
    from paper_1407_7370_amd import binding
    (ev, bd), = binding.hermite_eigen([hp], [torch.from_numpy(start).cuda()], k, [lo], [hi], tol, wanted)
    return ev, bd


@pytest.mark.parametrize("n", [16, 32, 48, 64])
@pytest.mark.parametrize("chirality,bz", [(1, 0.0), (-1, 0.7), (1, -1.3)])
def test_recurrence_vs_oracle(torch_cuda, orc, n, chirality, bz):
    """An off-centre random start vector (all four parity sectors), so that a
    wrong block or a wrong coupling of the parities moves the values."""
    Z = 3.0
    hp = dict(packets.softcore_hermite(Z, n=n, chirality=chirality), bz=bz)
    rng = np.random.default_rng(n)
    start = packets.hermite_packet(hp, 1.0 / Z, (0.4 / Z, 0.25 / Z))
    start = start + 0.05 * (rng.standard_normal(start.shape) + 1j * rng.standard_normal(start.shape)) / n
    start /= np.linalg.norm(start)
    lo, hi, tol, k = MC2 - 0.7 * Z * Z, MC2 - 0.05 * Z * Z, 1e-5, 400
    say(f"hermite recurrence n={n} chirality={chirality} bz={bz}")
    ev, bd = eigen(torch_cuda, hp, start, k, lo, hi, tol)
    rev, rbd, _ = orc.eigen_hermite(hp, start, k, lo, hi, tol)
    print("gpu:", np.round(ev - MC2, 7).tolist(), "oracle:", np.round(rev - MC2, 7).tolist(), flush=True)
    assert len(ev) >= 1
    assert hz.match_converged(ev, bd, rev, rbd, tol) >= 1


def test_device_and_host_ritz_agree(torch_cuda):
    Z = 50.0
    hp = packets.softcore_hermite(Z)
    start = packets.hermite_packet(hp, 1.0 / Z, (0.4 / Z, 0.25 / Z))
    lo, hi, tol = MC2 - 0.6 * Z * Z, MC2 - 0.14 * Z * Z, 1e-5
    say("hermite ritz on the device (K = 2048) and on the host (K = 2049)")
    ev, bd = eigen(torch_cuda, hp, start, 2048, lo, hi, tol)
    hev, hbd = eigen(torch_cuda, hp, start, 2049, lo, hi, tol)
    assert len(ev) >= 6 and hz.match_converged(ev, bd, hev, hbd, tol) == len(ev)
    # a window that holds more values of T than the device keeps per block (most
    # of them not converged)
    say("hermite ritz in a wide window (host)")
    wev, wbd = eigen(torch_cuda, hp, start, 2048, MC2 - 0.6 * Z * Z, MC2 + 3.0 * Z * Z, tol, wanted=256)
    assert len(wev) > len(ev) and hz.match_converged(ev, bd, wev[wev <= hi], wbd[wev <= hi], tol) == len(ev)
    # no value in the window; a single iteration
    say("hermite ritz edge windows")
    none, _ = eigen(torch_cuda, hp, start, 300, -2.0, -1.0, tol)
    assert len(none) == 0
    one, b1 = eigen(torch_cuda, hp, start, 1, 0.0, 2.0 * MC2, 1e9)
    assert len(one) == 1 and b1[0] > 0


@pytest.mark.parametrize("n,k,problems", [(32, 1024, 40), (16, 300, 12), (64, 700, 22)])
def test_many_problems_agree_with_one_at_a_time(torch_cuda, n, k, problems):
    """The Ritz step runs on the device for at least k / 32 problems, on the host for
    fewer, and a block of a device call whose window holds more values than the
    device keeps per block goes to the host by itself (the later blocks of the wide
    windows here)."""
    from paper_1407_7370_amd import binding
    torch = torch_cuda
    tol = 1e-5
    zs = np.linspace(2.0, 40.0, problems)
    hps = [packets.softcore_hermite(float(z), n=n) for z in zs]
    starts = [torch.from_numpy(packets.hermite_packet(h, 1 / z, (0.4 / z, 0.25 / z))).cuda() for h, z in zip(hps, zs)]
    # narrow, wide and empty windows in turn
    lo = [MC2 - 0.7 * z * z for z in zs]
    hi = [MC2 + (-0.14, 3.0, -0.69)[i % 3] * z * z for i, z in enumerate(zs)]
    say(f"hermite {problems} problems n={n} k={k}: together")
    many = binding.hermite_eigen(hps, starts, k, lo, hi, tol, 64)
    say("one at a time")
    found = 0
    for i in range(problems):
        (ev, bd), = binding.hermite_eigen(hps[i:i + 1], starts[i:i + 1], k, lo[i:i + 1], hi[i:i + 1], tol, 64)
        found += hz.match_converged(*many[i], ev, bd, tol)
    assert found >= problems // 3
