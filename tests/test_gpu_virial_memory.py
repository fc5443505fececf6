"""Device memory of a virial object against the figure its header states, with
few cells and with as many as the atoms allow."""
import os
import re

import numpy as np
import pytest

from tests._cases import announce

pytestmark = pytest.mark.gpu
HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "mhc.h")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("max_nb", [4, 20])
@pytest.mark.parametrize("edge,cells", [(30.0, 10 * 10 * 10), (700.0, 233 * 233 * 116)])   # the last: 6 per atom, of at most 8
def test_device_memory_is_as_stated(edge, cells, max_nb):
    import torch
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce(f"virial memory edge={edge} max_nb={max_nb}")
    with open(HEADER) as fh:
        text = re.sub(r"\s*\n \*\s*", " ", fh.read())
    d, i, j = map(int, re.search(r"Device memory: (?:about )?N \(3 max_neighbors \+ (\d+)\) doubles and "
                                 r"N \((\d+) max_neighbors \+ (\d+)\) ints", text).groups())
    N = 1 << 20
    mass = np.full(N, 28.0)
    stated = N * ((3 * max_nb + d) * 8 + (i * max_nb + j) * 4) + 2 * cells * 4 + 8192
    used = []
    for _ in range(2):                              # the first turn warms the runtime
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        v = ModalVirial(mass, [edge] * 3, tersoff_si(), max_neighbors=max_nb, skin=0.0)
        used.append(free - torch.cuda.mem_get_info()[0])
        v.close()
    assert 0.95 * stated <= used[1] <= stated + (4 << 20), (used, stated)     # allocations come in pieces of 2 MiB


def test_same_bits_however_the_arrays_are_allocated():
    """64000 atoms: one allocation for everything (8 slots), one for each array (24
    slots: more than 64 MB), one because an array alone is larger (64 slots)."""
    import torch
    import synth
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce("virial arrays in one allocation and in many")
    pos, box = synth.diamond((20, 20, 20), sigma=0.05, seed=3)
    mass = synth.masses(len(pos))
    vel = np.random.default_rng(4).normal(0.0, 5e-3, pos.shape)
    out = []
    for max_nb in (8, 24, 64):
        v = ModalVirial(mass, box, tersoff_si(), max_neighbors=max_nb, skin=0.3)
        p, u = (torch.as_tensor(x, device="cuda:0").clone() for x in (pos, vel))
        v.neighbors(p)
        r = dict(v.compute(p))
        v.md(p, u, 1.0, 7, rebuild=3)
        v.neighbors(p)
        counts, lists = v.read_neighbors()
        out.append([r[k].cpu().numpy() for k in sorted(r)] + [p.cpu().numpy(), u.cpu().numpy(), counts, lists[:, :8]])
        v.close()
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))
