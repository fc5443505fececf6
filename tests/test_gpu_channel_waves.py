"""The contraction with one channel per wave (small systems) at the edges of
its tiles: one row block and one t-block, k shorter than its staging, ragged
modes, the pieces of a split tile, the direction split, and whole rounds of
tiles followed by a rest that runs channel by channel.  Against the plane-wave
(FFT) form of the oracle; tolerances as for every other batched contraction
(relative L2: FP32 1e-5, split-BF16 1e-4, e4m3 hi/lo 1e-2)."""
import numpy as np
import pytest

import oracle
import synth
from tests._cases import announce, log, rel

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]
HNEMA, GKMA, DIRECTIONAL = 1, 2, 4
TOL = {0: 1e-5, 1: 1e-4, 3: 1e-2}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("prec", [0, 1, 3])
@pytest.mark.parametrize("dims,T,methods", [((1, 1, 1), 32, HNEMA), ((2, 3, 2), 32, GKMA), ((3, 3, 4), 64, HNEMA | DIRECTIONAL),
                                            ((7, 5, 9), 96, HNEMA | GKMA), ((11, 9, 8), 128, HNEMA),
                                            ((14, 14, 14), 512, HNEMA)])
def test_channel_waves(dims, T, methods, prec):
    from paper_2102_03691_amd import ModalHC
    announce(f"channel waves {dims} T={T} methods={methods} prec={prec}")
    lat = synth.BlochLattice(dims)
    m = synth.masses(lat.n_atoms, "natural", 2)
    nb, L, S = 5, 9, T if T > 256 else T + 11
    v, W = synth.gen_steps(3, m, 0, S)
    h = ModalHC(0)
    h.load_system(m, lat.frequencies)
    h.set_bins_uniform(nb, 0.0, lat.f_max)
    h.configure(methods=methods, precision=prec, t_block=T, corr_len=L if methods & GKMA else 0)
    for r0 in range(0, lat.n_modes, 2048):
        h.load_eigvec_rows(r0, lat.eig_rows_torch(r0, min(2048, lat.n_modes - r0), device="cuda:0"))
    h.finalize()
    h.push(v, W)
    kb = oracle.bin_of_mode(lat.kpoint_frequencies().ravel(), nb, 0.0, lat.f_max).reshape(lat.dims)
    Jb = oracle.binned_current_fft(lat.dims, m, v, W, kb, nb)
    err = {}
    if methods & HNEMA:
        err["hnema"] = rel(h.read_hnema()[0], oracle.hnema_average(Jb))
    if methods & DIRECTIONAL:
        err["sum_over_directions"] = rel(h.read_hnema_dir()[0].sum(axis=2), oracle.hnema_average(Jb))
    if methods & GKMA:
        Jt = oracle.total_heat_current(v, W)
        err["corr"] = rel(h.read_gkma()["corr"], oracle.gkma_correlation(Jb, Jt, L))
    h.close()
    log(f"channel_waves_{dims}_T{T}_m{methods}_p{prec}", **err)
    assert max(err.values()) <= TOL[prec], err
