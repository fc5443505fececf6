"""Per-step path: steps of one push that share a pass over the basis give the
bits of the same steps pushed one at a time (every per-step binned current and
total, float64 sums of the same float32 modal currents), at step counts around
the group of four, row counts around the work-group's 32 and the smallest
launches that take the grouped kernel.  Sums over steps may be grouped
differently in float64: 2 * 200 additions of 2^-53 each, far below 1e-12."""
import numpy as np
import pytest

import synth
from tests._cases import announce, rel

pytestmark = pytest.mark.gpu
HNEMA, GKMA, DIRECTIONAL = 1, 2, 4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("dims,nb", [((4, 4, 4), 3), ((5, 7, 9), 40)])
@pytest.mark.parametrize("steps", [9, 10, 11, 33, 35, 64, 130])
@pytest.mark.parametrize("methods", [HNEMA, HNEMA | GKMA, HNEMA | DIRECTIONAL])
def test_grouped_steps_equal_single_steps(dims, nb, steps, methods):
    from paper_2102_03691_amd import ModalHC
    announce(f"step groups {dims} steps={steps} methods={methods}")
    lat = synth.BlochLattice(dims)
    m = synth.masses(lat.n_atoms, "natural", 4)
    v, W = synth.gen_steps(8, m, 0, steps)
    out = []
    for piece in (steps, 1):
        h = ModalHC(0)
        h.load_system(m, lat.frequencies)
        h.set_bins_uniform(nb, 0.0, lat.f_max)
        h.configure(methods=methods, t_block=1, corr_len=4 if methods & GKMA else 0)
        h.load_eigvec_rows(0, lat.eig_rows(0, lat.n_modes))
        h.finalize()
        jb = []
        for s0 in range(0, steps, piece):
            h.push(v[s0:s0 + piece], W[s0:s0 + piece])
            if methods & GKMA:
                jb.append(h.read_block_currents(min(piece, steps - s0)))
        out.append((h.read_hnema(), np.concatenate(jb) if jb else None,
                    h.read_hnema_dir()[0] if methods & DIRECTIONAL else None))
        h.close()
    (a, ja, da), (b, jb, db) = out
    assert a[2] == b[2] == steps
    assert rel(a[0], b[0]) <= 1e-12 and rel(a[1], b[1]) <= 1e-12
    if methods & GKMA:
        assert np.array_equal(ja, jb)
    if methods & DIRECTIONAL:
        assert rel(da, db) <= 1e-12


@pytest.mark.parametrize("dims", [(1, 1, 1), (16, 10, 1), (23, 7, 1), (21, 64, 1), (269, 5, 1)])
@pytest.mark.parametrize("methods", [HNEMA, HNEMA | GKMA])
def test_small_step_path_edges(dims, methods):
    """Steps pushed one by one, where the contraction builds its operand itself
    (operand lengths around its padding to 512 and around the longest it takes,
    4096), against one push of the first step count past that path (more than
    4096 waves of 8 rows, or 4096 x 1536 waves x dofs): the same bits per step."""
    from paper_2102_03691_amd import ModalHC
    lat = synth.BlochLattice(dims)
    m = synth.masses(lat.n_atoms, "natural", 4)
    k_pad = -(-96 * -(-lat.n_atoms // 32) // 512) * 512
    steps = min(4096, 4096 * 1536 // k_pad) * 8 // (-(-lat.n_modes // 256) * 256) + 1
    announce(f"small steps {dims} steps={steps} methods={methods}")
    v, W = synth.gen_steps(9, m, 0, steps)
    out = []
    for piece in (steps, 1):
        h = ModalHC(0)
        h.load_system(m, lat.frequencies)
        h.set_bins_uniform(7, 0.0, lat.f_max)
        h.configure(methods=methods, t_block=1, corr_len=4 if methods & GKMA else 0)
        for r0 in range(0, lat.n_modes, 512):
            h.load_eigvec_rows(r0, lat.eig_rows(r0, min(512, lat.n_modes - r0)))
        h.finalize()
        jb = []
        for s0 in range(0, steps, piece):
            h.push(v[s0:s0 + piece], W[s0:s0 + piece])
            if methods & GKMA:
                jb.append(h.read_block_currents(min(piece, steps - s0)))
        out.append((h.read_hnema(), np.concatenate(jb) if jb else None))
        h.close()
    (a, ja), (b, jb) = out
    assert a[2] == b[2] == steps
    assert rel(a[0], b[0]) <= 1e-12 and rel(a[1], b[1]) <= 1e-12
    if methods & GKMA:
        assert np.array_equal(ja, jb)
