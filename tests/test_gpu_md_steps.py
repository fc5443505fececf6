"""Step bookkeeping of the molecular dynamics: the drift of a step runs in the
force kernel of the step before it and alternates between two position arrays,
so odd and even step counts, a single step, a call split in two and lists
rebuilt at every step must all give the same trajectory; the thermostat's
update runs in the start-of-step kernel (up to 16384 atoms) or in its own."""
import numpy as np
import pytest

import synth
from oracle import virial as ov
from tests._cases import announce

pytestmark = pytest.mark.gpu
KE = 1.66053906660e-27 * 1e10 / 1.602176634e-19
KB = 8.617333262e-5


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _start(cells, seed=3):
    import torch
    pos, box = synth.diamond(cells, sigma=0.05, seed=seed)
    m = synth.masses(len(pos), "natural", 1)
    vel = synth.thermal_velocities(m, 300.0, seed)
    return pos, box, m, vel, torch.as_tensor(pos, device="cuda:0").clone(), torch.as_tensor(vel, device="cuda:0").clone()


@pytest.mark.parametrize("skin", [0.0, 1.0])
@pytest.mark.parametrize("pieces,rebuild", [((1,), 0), ((2,), 1), ((5,), 2), ((6,), 0), ((3, 3), 1), ((2, 1, 3), 4)])
def test_nve_step_counts(pieces, rebuild, skin):
    """Against the oracle's integrator (positions 1e-12 A, velocities 1e-12 relative: a few steps of float64)."""
    import torch
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce(f"nve pieces={pieces} rebuild={rebuild} skin={skin}")
    pos, box, m, vel, x, v = _start((2, 2, 2))
    n = sum(pieces)
    ref = ov.md_nve(pos, vel, m, box, ov.tersoff_si(), 1.0, n)
    vir = ModalVirial(m, box, tersoff_si(), max_neighbors=24, skin=skin)
    vir.neighbors(x)
    if skin == 0.0:
        rebuild = 1          # exact lists hold for the positions they were built at
    v32 = torch.empty((n, len(pos), 3), dtype=torch.float32, device="cuda:0")
    at = 0
    for k in pieces:
        vir.md(x, v, 1.0, k, rebuild=rebuild, v32=v32[at:at + k])
        at += k
    torch.cuda.synchronize()
    assert np.abs(ov.min_image(x.cpu().numpy() - ref["pos"][-1], box)).max() <= 1e-12
    assert np.abs(v.cpu().numpy() - ref["vel"][-1]).max() <= 1e-12 * np.abs(ref["vel"][-1]).max()
    assert np.abs(v32.cpu().numpy() - ref["vel"][-n:]).max() <= 2.0 ** -23 * np.abs(ref["vel"]).max()
    vir.close()


@pytest.mark.parametrize("cells", [(2, 2, 2), (10, 10, 10), (13, 13, 13)])
def test_thermostat_update(cells):
    """One step from rest of the thermostat: xi and eta from the kinetic energies
    at entry and at the end (sums of up to 53000 float64 terms: 1e-9 of the
    difference 2K - 3NkT covers their rounding)."""
    import torch
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce(f"thermostat {cells}")
    pos, box, m, vel, x, v = _start(cells)
    vir = ModalVirial(m, box, tersoff_si(), max_neighbors=24, skin=1.0)
    vir.neighbors(x)
    xi, eta = vir.md_nvt(x, v, 1.0, 1, None, 250.0, 80.0)
    torch.cuda.synchronize()
    gkt = 3 * len(pos) * KB * 250.0
    g = lambda w: (float((m[:, None] * w * w).sum()) * KE - gkt) / (gkt * 80.0 ** 2)  # noqa: E731
    half = 0.5 * g(vel)
    want_eta = half
    want_xi = half + 0.5 * g(v.cpu().numpy())
    assert abs(xi - want_xi) <= 1e-9 * abs(want_xi) and abs(eta - want_eta) <= 1e-9 * abs(want_eta)
    vir.close()
