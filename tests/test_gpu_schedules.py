"""A schedule that the caller names runs the kernel it names, and AUTO's kernel
for few tiles (one channel per wave) gives that kernel's bits: whole tiles, the
pieces of split tiles (three and more to a tile), whole rounds of tiles followed
by a rest, and the direction split, slot-major (HNEMA only) and step-major."""
import numpy as np
import pytest

import synth
from tests._cases import announce

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]
HNEMA, GKMA, DIRECTIONAL = 1, 2, 4
AUTO, TILES, STREAMK, SPLIT = 0, 1, 2, 3


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(lat, m, v, W, methods, prec, T, sched):
    from paper_2102_03691_amd import ModalHC
    L = 9
    h = ModalHC(0)
    h.load_system(m, lat.frequencies)
    h.set_bins_uniform(5, 0.0, lat.f_max)
    h.configure(methods=methods, precision=prec, t_block=T, corr_len=L if methods & GKMA else 0, schedule=sched)
    for r0 in range(0, lat.n_modes, 2048):
        h.load_eigvec_rows(r0, lat.eig_rows_torch(r0, min(2048, lat.n_modes - r0), device="cuda:0"))
    h.finalize()
    h.push(v, W)
    out = list(h.read_hnema()[:2])
    if methods & DIRECTIONAL:
        out += h.read_hnema_dir()[:2]
    if methods & GKMA:
        out.append(h.read_gkma()["corr"])
    ran = h.last_schedule(), h.last_kernel()
    h.close()
    return out, *ran


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("dims,T", [((1, 1, 1), 32), ((8, 8, 4), 64), ((12, 12, 8), 32), ((12, 12, 8), 128),
                                    ((9, 8, 8), 96), ((14, 14, 14), 512)])
@pytest.mark.parametrize("methods", [HNEMA, HNEMA | GKMA])
def test_named_schedule_runs_its_kernel(dims, T, methods, prec):
    announce(f"schedules {dims} T={T} methods={methods} prec={prec}")
    lat = synth.BlochLattice(dims)
    m = synth.masses(lat.n_atoms, "natural", 2)
    v, W = synth.gen_steps(3, m, 0, T if T > 256 else T + 11)
    ref, sums, kernel = _run(lat, m, v, W, methods, prec, T, AUTO)
    for asked in (TILES, STREAMK, SPLIT):
        if T > 256 and asked != sums:
            continue
        out, ran, named = _run(lat, m, v, W, methods, prec, T, asked)
        assert named == ("k_gemm_split" if ran == SPLIT else "k_gemm"), (asked, ran, named)
        assert asked != TILES or ran == TILES
        if ran == sums:
            assert all(np.array_equal(a, b) for a, b in zip(ref, out)), (asked, kernel)
    if 1 < lat.n_atoms and T <= 128:   # (one atom: two k-stages, a tile is as short)
        assert kernel == "k_gemm_chan"


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("dims,T", [((12, 12, 8), 32), ((7, 5, 9), 64), ((9, 8, 8), 96), ((11, 9, 8), 128)])
@pytest.mark.parametrize("methods", [HNEMA, HNEMA | GKMA])
def test_named_schedule_runs_the_direction_tiles(dims, T, methods, prec):
    announce(f"schedules, direction split {dims} T={T} methods={methods} prec={prec}")
    lat = synth.BlochLattice(dims)
    m = synth.masses(lat.n_atoms, "natural", 2)
    v, W = synth.gen_steps(3, m, 0, T + 11)
    ref, _, kernel = _run(lat, m, v, W, methods | DIRECTIONAL, prec, T, AUTO)
    assert kernel == "k_gemm_chan"
    for asked in (TILES, STREAMK, SPLIT):
        out, _, named = _run(lat, m, v, W, methods | DIRECTIONAL, prec, T, asked)
        assert named == "k_gemm_dir", asked
        assert all(np.array_equal(a, b) for a, b in zip(ref, out)), asked
