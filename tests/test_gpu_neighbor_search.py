"""Neighbour search at its edges, bit for bit against the oracle's lists: boxes
of one cell along an axis and of exactly three, rows that wrap at either end,
atom counts that are not a multiple of the work-group's 16 atoms, periodic
images of the positions, atoms in random order, and repeated searches (the
cell counts are cleared by the search before)."""
import numpy as np
import pytest

import synth
from tests._cases import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("cells,drop,skin", [((2, 2, 2), 0, 0.0), ((2, 2, 2), 63, 1.0), ((2, 2, 3), 5, 0.0),
                                             ((2, 3, 5), 3, 1.0), ((5, 2, 2), 1, 0.5), ((3, 3, 3), 17, 1.0),
                                             ((2, 2, 9), 0, 0.0)])
def test_lists_at_the_edges(cells, drop, skin):
    import torch
    import oracle.virial as ov
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce(f"neighbour search {cells} drop={drop} skin={skin}")
    pos, box = synth.diamond(cells, sigma=0.08, seed=5)
    rng = np.random.default_rng(6)
    pos = pos[rng.permutation(len(pos))[: len(pos) - drop]]
    v = ModalVirial(synth.masses(len(pos)), box, tersoff_si(), max_neighbors=40, skin=skin)
    for shift in (0, 3):
        p = pos + shift * 0.37 + box * rng.integers(-2, 3, size=pos.shape)
        ref = ov.neighbor_lists(np.mod(p, box), box, 3.0 + skin)
        most = v.neighbors(torch.as_tensor(p, device="cuda:0"))
        counts, lists = v.read_neighbors()
        assert most == max(len(r) for r in ref)
        for i, r in enumerate(ref):
            assert counts[i] == len(r) and np.array_equal(lists[i, : counts[i]], sorted(r)) and (lists[i, counts[i]:] == -1).all()
    v.close()


@pytest.mark.parametrize("cells,keep", [((10, 10, 10), 1000), ((15, 15, 15), 2600), ((19, 19, 19), 5000),
                                        ((20, 20, 20), 5900)])
def test_scan_tiles(cells, keep):
    """Few atoms in many cells: 6, 20, 39 and 46 tiles of the cell scan (its own
    counts up to 40 tiles, 16 at a time; sums of tiles above)."""
    import torch
    import oracle.virial as ov
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce(f"neighbour search {cells} keep={keep}")
    pos, box = synth.diamond(cells, sigma=0.08, seed=7)
    pos = pos[np.random.default_rng(8).permutation(len(pos))[:keep]]
    ref = ov.neighbor_lists(pos, box, 3.0)
    v = ModalVirial(synth.masses(len(pos)), box, tersoff_si(), max_neighbors=8, skin=0.0)
    for _ in range(2):
        assert v.neighbors(torch.as_tensor(pos, device="cuda:0")) == max(len(r) for r in ref)
        counts, lists = v.read_neighbors()
        for i, r in enumerate(ref):
            assert counts[i] == len(r) and np.array_equal(lists[i][: len(r)], r)
    v.close()
