"""Read-outs at the edges of the finishing kernels and of the pinned buffer.

The GKMA finisher works on tiles of 64 series (9 bins + 9) x 64 lags; small
read-outs go through 64 KB of pinned host memory, larger ones through device
memory.  Correlations are held to the oracle at the bounds of the FP32 path
(1e-5, the float64 total 1e-12); the
running integral to the trapezoid rule over the correlation read (L additions of
2^-53 each, L <= 200: below 1e-13 of the largest value); results read in pieces
to the same bits as in one."""
import numpy as np
import pytest

import synth
from tests._cases import TOL, Case, announce, rel, run_library

pytestmark = pytest.mark.gpu
HNEMA, GKMA, FP32 = 1, 2, 0


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("nb,L,S", [(6, 2, 5), (6, 63, 70), (7, 64, 70), (7, 65, 70), (13, 129, 40), (20, 200, 250),
                                      (1500, 960, 70)])     # the last: correlation tiles of 64 lags
def test_gkma_finish_tiles(nb, L, S):
    announce(f"gkma read-out nb={nb} L={L} S={S}")
    case = Case((3, 3, 2), S, "natural", 5)
    out = run_library(case, nb, HNEMA | GKMA, FP32, 64, corr_len=L, dt=0.5, splits=[S // 2, S - S // 2])
    want = case.oracle(nb, corr_len=L, dt=0.5)
    c = out["corr"]
    assert rel(c, want["corr"]) <= TOL[FP32] and rel(out["hcacf"], want["hcacf"]) <= 1e-12
    run = np.zeros_like(c)
    run[1:] = np.cumsum(0.25 * (c[1:] + c[:-1]), axis=0)
    assert np.abs(out["integral"] - run).max() <= 1e-13 * np.abs(run).max()
    assert not out["corr"][S:].any()


@pytest.mark.parametrize("nb", [2729, 2730])      # 3 nb + 3 doubles: 64 KB, and just above
def test_hnema_read_around_the_pinned_size(nb):
    announce(f"hnema read-out nb={nb}")
    case = Case((3, 3, 2), 6, "natural", 6)
    out = run_library(case, nb, HNEMA, FP32, 64)
    want = case.oracle(nb)
    assert rel(out["hnema"], want["hnema"]) <= TOL[FP32]
    assert rel(out["hnema_total"], want["hnema_total"]) <= 1e-12


@pytest.mark.parametrize("n_lags", [910, 911])    # 9 n_lags doubles: 64 KB, and just above
def test_shc_reads_around_the_pinned_size(n_lags):
    from paper_2102_03691_amd import ModalSHC
    announce(f"shc read-out n_lags={n_lags}")
    N, S = 40, 130
    m = synth.masses(N, "natural", 7)
    v, W = synth.gen_steps(9, m, 0, S)
    s = ModalSHC(N, n_lags, 64)
    s.push(v, W)
    K, n = s.read()
    Kd, nd = s.read_dir()
    assert n == nd == S
    assert np.array_equal(K, (Kd[..., 0] + Kd[..., 1]) + Kd[..., 2])
    w = np.linspace(0.1, 30.0, 2049)
    for f in (s.spectrum, s.spectrum_dir):
        whole = f(w, 0.01)
        parts = np.concatenate([f(w[a:a + 700], 0.01) for a in range(0, 2049, 700)])
        assert np.array_equal(whole, parts)
    s.reset()
    K0, n0 = s.read()
    assert n0 == 0 and not K0.any()
    s.push(v, W)
    assert np.array_equal(s.read()[0], K)
    s.close()


@pytest.mark.parametrize("atoms", [[40], [70, 40, 130, 40, 33], [40] * 16, [30 + k % 7 for k in range(70)]])
@pytest.mark.parametrize("steps", [64, 100])
def test_shc_group_work_group_orders(atoms, steps):
    """Systems of a group on any XCD and in any order of the launch (one, mixed
    lengths, equal lengths, more systems than a wave has lanes) give the bits
    of their own pushes."""
    import torch
    from paper_2102_03691_amd import ModalSHC, SHCGroup
    announce(f"shc group n={len(atoms)} steps={steps}")
    ins = [synth.gen_steps(k, synth.masses(N, "natural", k), 0, steps) for k, N in enumerate(atoms)]
    stream = torch.cuda.Stream()
    got = [ModalSHC(N, 70, 64, stream=stream.cuda_stream) for N in atoms]
    group = SHCGroup(got)
    group.push([v for v, _ in ins], [W for _, W in ins])
    for N, (v, W), s in zip(atoms, ins, got):
        one = ModalSHC(N, 70, 64)
        one.push(v, W)
        assert np.array_equal(one.read()[0], s.read()[0])
        one.close()
    group.close()
    for s in got:
        s.close()
