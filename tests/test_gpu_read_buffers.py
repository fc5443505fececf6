"""The pinned read buffers: a small object alone that is read once allocates none
(the process gets no mapping of their 1 MiB), sixteen objects share one
allocation, made with the eighth of them, the last one to go frees it, and every
read gives the same bits whether it came by copy (the first of a small object
alone) or through the buffer (the later ones)."""
import numpy as np
import pytest

import synth
from tests._cases import announce

pytestmark = pytest.mark.gpu
HNEMA, GKMA, DIRECTIONAL = 1, 2, 4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _slabs():
    """Device-visible host mappings of 1 MiB in this process."""
    n = 0
    with open("/proc/self/maps") as fh:
        for line in fh:
            f = line.split()
            a, b = (int(x, 16) for x in f[0].split("-"))
            n += len(f) > 5 and f[5].startswith("/dev/dri") and f[1].startswith("rw") and b - a == 1 << 20
    return n


def _modal(methods, t):
    from paper_2102_03691_amd import ModalHC
    lat = synth.BlochLattice((3, 3, 2))
    h = ModalHC(0)
    h.load_system(synth.masses(lat.n_atoms, "natural", 1), lat.frequencies)
    h.set_bins_uniform(4, 0.0, lat.f_max)
    h.configure(methods=methods, t_block=t, corr_len=6 if methods & GKMA else 0)
    h.load_eigvec_rows(0, lat.eig_rows(0, lat.n_modes))
    h.finalize()
    return h, lat.n_atoms


def _shc(n_atoms=40):
    from paper_2102_03691_amd import ModalSHC
    return ModalSHC(n_atoms, 20, 64), n_atoms


KINDS = {"step": (lambda: _modal(HNEMA, 1), ("read_hnema",)),
         "batch": (lambda: _modal(HNEMA | GKMA, 32), ("read_hnema", "read_gkma")),
         "dir": (lambda: _modal(HNEMA | GKMA | DIRECTIONAL, 32),
                 ("read_hnema", "read_hnema_dir", "read_gkma", "read_gkma_dir")),
         "shc": (_shc, ("read", "read_dir", "spectrum"))}


def _read(h, name):
    r = h.spectrum(np.linspace(0.0, 0.1, 7), 1.0) if name == "spectrum" else getattr(h, name)()
    return [np.asarray(r[k]) for k in sorted(r)] if isinstance(r, dict) else [np.asarray(x) for x in (r if isinstance(r, tuple) else (r,))]


@pytest.mark.parametrize("kind", sorted(KINDS))
def test_reads_by_copy_and_through_the_buffer(kind):
    announce(f"read buffers {kind}")
    make, reads = KINDS[kind]
    for first in reads:
        h, n = make()
        h.push(*synth.gen_steps(2, synth.masses(n), 0, 40))
        by_copy = _read(h, first)
        for name in reads:
            later = [_read(h, name) for _ in range(2)]
            assert all(np.array_equal(a, b) for a, b in zip(*later))
            if name == first:
                assert all(np.array_equal(a, b) for a, b in zip(by_copy, later[0])), name
        h.close()


@pytest.mark.parametrize("kind", ["step", "shc"])
def test_one_read_allocates_no_buffer(kind):
    announce(f"read buffers, one read {kind}")
    make, reads = KINDS[kind]
    grown = []                  # over four turns: the runtime's own allocations come once
    for _ in range(4):
        n0 = _slabs()
        h, n = make()
        h.push(*synth.gen_steps(2, synth.masses(n), 0, 40))
        _read(h, reads[0])
        n1 = _slabs()
        _read(h, reads[0])
        n2 = _slabs()
        h.close()
        grown.append((n1 - n0, n2 - n0, _slabs() - n0))
    one, two, closed = (min(g) for g in zip(*grown))
    assert one == 0, "an object read once allocated pinned memory"
    assert two <= 1 and closed <= 0


def test_objects_share_an_allocation():
    announce("read buffers, 33 objects")
    n = 40
    from paper_2102_03691_amd import ModalSHC
    import torch
    st = torch.cuda.Stream()
    grown = []
    for _ in range(4):
        n0 = _slabs()
        objs = [ModalSHC(n, 20, 64, stream=st.cuda_stream) for _ in range(7)]
        n7 = _slabs()
        objs += [ModalSHC(n, 20, 64, stream=st.cuda_stream) for _ in range(26)]
        n33 = _slabs()
        for h in objs:
            h.push(*synth.gen_steps(2, synth.masses(n), 0, 10))
            _read(h, "read"), _read(h, "read")
        n_read = _slabs()
        for h in objs[::2] + objs[1::2]:
            h.close()
        grown.append((n7 - n0, n33 - n0, n_read - n0, _slabs() - n0))
    seven, all33, read, closed = (min(g) for g in zip(*grown))
    assert seven == 0 and 1 <= all33 <= 3 and read <= 3 and closed <= 0
