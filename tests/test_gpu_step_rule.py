"""Per-step path, pushes of several steps: which kernel takes them (rounds of one
wave per SIMD, one wave per 8 modes and step; operand length; modes), and the
same bits per step as the steps pushed one at a time, whichever it is.  The
operand (4320 dofs, padded to 4608) is longer than the one-launch kernel takes."""
import numpy as np
import pytest

import synth
from tests._cases import announce

pytestmark = pytest.mark.gpu
HNEMA, GKMA = 1, 2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("modes,steps,kernel", [(300, 5, "k_gemv_f32"), (1000, 8, "k_gemv_f32"),
                                                (1000, 9, "k_gemv_f32"), (1000, 12, "k_gemv_f32"),
                                                (1000, 16, "k_gemv_f32"), (1000, 17, "k_gemv_steps"),
                                                (128, 64, "k_gemv_f32"), (128, 65, "k_gemv_steps"),
                                                (128, 130, "k_gemv_steps"), (3072, 2, "k_gemv_f32"),
                                                (3072, 3, "k_gemv_steps"), (4320, 1, "k_gemv_f32"),
                                                (4320, 2, "k_gemv_steps"), (4320, 5, "k_gemv_steps")])
def test_kernel_of_a_push(modes, steps, kernel):
    from paper_2102_03691_amd import ModalHC
    announce(f"step rule modes={modes} steps={steps}")
    lat = synth.BlochLattice((12, 12, 10))
    m = synth.masses(lat.n_atoms, "natural", 4)
    v, W = synth.gen_steps(8, m, 0, steps)
    out = []
    for piece in (steps, 1):
        h = ModalHC(0)
        h.load_system(m, lat.frequencies[:modes])
        h.set_bins_uniform(7, 0.0, lat.f_max)
        h.configure(methods=HNEMA | GKMA, t_block=1, corr_len=4)
        for r0 in range(0, modes, 1440):
            h.load_eigvec_rows(r0, lat.eig_rows_torch(r0, min(1440, modes - r0), device="cuda:0"))
        h.finalize()
        jb = []
        for s0 in range(0, steps, piece):
            h.push(v[s0:s0 + piece], W[s0:s0 + piece])
            jb.append(h.read_block_currents(min(piece, steps - s0)))
        assert h.last_kernel() == (kernel if piece == steps else "k_gemv_f32")
        out.append(np.concatenate(jb))
        h.close()
    assert np.array_equal(out[0], out[1])
