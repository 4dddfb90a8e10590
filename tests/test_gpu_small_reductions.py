"""The reductions around the chunk kernel at the edges of their blocks, against FP64
references: the exact mean pre-pass (64 pixels and 16 frame groups of 8 loads per
block), the tiled ring store (1 KiB of pixels by up to 16 frames), finalize and the
detector sums (1024 pixels per block), the D_p correction and the partial reduce
(8 slots per block), each on a second pass over the same plan too."""

import numpy as np
import pytest
import torch

import oracle as O
import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


def check(plan, host, L, H, window, masks, push, param=None, passes=2):
    P, NT, ny, nx = host.shape
    psi = host.cuda()
    So, Spo = O.tacaw_spectra(host.numpy(), L, H, O.window(window, L, param), fft=True)
    want = So, O.detector_spectra(So, masks), np.transpose(O.detector_spectra(Spo, masks), (1, 0, 2))
    for k in range(passes):
        plan.reset()
        for f in range(0, NT, push):
            plan.push(psi[:, f:f + push])
        S = plan.finalize().cpu().numpy().reshape(L, -1)
        D, Dp = plan.detector_spectra(per_probe=True)
        got = S, D.cpu().numpy(), Dp.cpu().numpy()
        err = [rel(g, w) for g, w in zip(got, want)]
        print(f"pass {k}: S {err[0]:.1e} D {err[1]:.1e} Dp {err[2]:.1e}", flush=True)
        assert max(err) <= 1e-5
        # D is the probe mean of D_p, both FP64 sums of the same spectra
        assert rel(got[2].mean(axis=1), got[1]) <= 1e-12


@pytest.mark.parametrize("ny,nx", [(1, 1), (7, 9), (8, 8), (5, 13), (32, 32), (25, 41)])
@pytest.mark.parametrize("NT,dtype", [(64, "c64"), (128 + 15, "c128"), (64 * 17 + 3, "c64")])
def test_exact_mean_pre_pass(ny, nx, NT, dtype):
    from paper_2607_02236_amd import tacaw

    L, H, P = 64, 32, 3
    host = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=NT + nx, model="lines", n_terms=8))
    m = np.stack([np.ones((ny, nx)), np.random.default_rng(nx).random((ny, nx))])
    with tacaw.Plan(P, ny, nx, NT, L, H, window="tukey", window_param=0.4, in_dtype=dtype,
                    masks=torch.from_numpy(m).cuda()) as plan:
        check(plan, host, L, H, "tukey", m, NT, 0.4)


@pytest.mark.parametrize("ny,nx,dtype", [(1, 3, "c64"), (1, 127, "c64"), (8, 16, "c64"), (3, 43, "c128"),
                                         (9, 29, "c64")])
@pytest.mark.parametrize("L,push", [(200, 100), (64, 17), (256, 128), (1024, 500)])
def test_tiled_ring_store(ny, nx, dtype, L, push):
    from paper_2607_02236_amd import tacaw

    H, P, NT = L // 2, 2, 3 * L + 50
    host = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=L + nx, model="lines", n_terms=8))
    m = np.stack([np.ones((ny, nx))])
    with tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype, masks=torch.from_numpy(m).cuda(), ring_frames=2 * L,
                    tiled_ring=True) as plan:
        check(plan, host, L, H, "hann", m, push)


@pytest.mark.parametrize("P,ny,nx", [(1, 1, 5), (9, 16, 16), (3, 33, 31), (33, 40, 52)])
@pytest.mark.parametrize("n_det,window", [(1, "hann"), (8, "rect")])
def test_probe_and_detector_reductions(P, ny, nx, n_det, window):
    from paper_2607_02236_amd import tacaw

    L, H, NT = 64, 64, 150
    host = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype="c64", seed=P + nx, model="lines", n_terms=8))
    rng = np.random.default_rng(P)
    m = rng.random((n_det, ny, nx)) * (rng.random((n_det, ny, 1)) > 0.3)  # some tiles without a mask
    with tacaw.Plan(P, ny, nx, NT, L, H, window=window, masks=torch.from_numpy(m).cuda()) as plan:
        check(plan, host, L, H, window, m, NT)
