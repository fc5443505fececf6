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
