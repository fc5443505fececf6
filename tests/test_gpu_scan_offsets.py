"""The cell scan's last form: more than 2048 tiles of 1024 cells, whose sums one
work-group scans in between (two passes of it at 2.1 million cells), bit for bit
against a search by k-d tree over the same periodic box."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

from tests._cases import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("cells,N", [((127, 127, 129), 270000), ((129, 128, 130), 270000), ((140, 131, 133), 310000)])
def test_search_over_many_cells(cells, N):
    """2032 tiles (each work-group adds the sums before its own), 2097 and 2383 (scanned)."""
    import torch
    from paper_2102_03691_amd import ModalVirial, tersoff_si
    announce(f"neighbour search over {cells} cells")
    assert np.prod(cells) <= 8 * N + 64
    rng = np.random.default_rng(11)
    box = 3.0 * np.array(cells) + 0.5
    pos = rng.uniform(0.0, box, (N, 3))
    pairs = cKDTree(pos, boxsize=box).query_pairs(3.0, output_type="ndarray")
    i, j = np.concatenate([pairs, pairs[:, ::-1]]).T
    order = np.lexsort((j, i))
    i, j = i[order], j[order]
    want = np.bincount(i, minlength=N)
    v = ModalVirial(np.full(N, 28.0), box, tersoff_si(), max_neighbors=24, skin=0.0)
    for _ in range(2):
        assert v.neighbors(torch.as_tensor(pos, device="cuda:0")) == want.max() <= 24
        counts, lists = v.read_neighbors()
        assert np.array_equal(counts, want)
        assert np.array_equal(lists[np.arange(24) < counts[:, None]], j)
    v.close()
