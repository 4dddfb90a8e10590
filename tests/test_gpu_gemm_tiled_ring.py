"""bf16 DFT-GEMM form fed through the tiled ring by pushes: its tiles are 128 pixels,
1 or 2 KiB a row, so that a block of the ring store (1 KiB of pixels) takes a whole
tile row of complex64 and half of one of complex128. One tile, whole tiles, and a
last tile with pixels in its first half only and in both."""

import numpy as np
import pytest
import torch

import oracle as O
import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("ny,nx,stride", [(5, 13, 13), (16, 16, 16), (17, 17, 17), (17, 21, 24)])
@pytest.mark.parametrize("L,push", [(128, 50), (1024, 256)])
def test_tiled_ring_pushes_match_oracle(dtype, ny, nx, stride, L, push):
    from paper_2607_02236_amd import tacaw

    H, P, NT = L // 2, 2, 3 * L + 40
    host = T.generate(T.SeriesSpec(P, NT, ny, stride, dtype=dtype, seed=L + nx, model="lines", n_terms=8))
    x = host.cuda()[:, :, :, :nx]
    m = np.stack([np.ones((ny, nx)), np.random.default_rng(nx).random((ny, nx))])
    with tacaw.Plan(P, ny, nx, NT, L, H, transform="gemm_bf16x3", in_dtype=dtype, k_row_stride=stride,
                    masks=torch.from_numpy(m).cuda(), ring_frames=2 * L, tiled_ring=True) as plan:
        for f in range(0, NT, push):
            plan.push(x[:, f:f + push])
        S = plan.finalize().cpu().numpy().reshape(L, -1)
        D, Dp = plan.detector_spectra(per_probe=True)
        D, Dp = D.cpu().numpy(), Dp.cpu().numpy()
    So, Spo = O.tacaw_spectra(np.ascontiguousarray(host.numpy()[:, :, :, :nx]), L, H, O.window("hann", L), fft=True)
    eS, eD = rel(S, So), rel(D, O.detector_spectra(So, m))
    eDp = rel(Dp, np.transpose(O.detector_spectra(Spo, m), (1, 0, 2)))
    print(f"L={L} {dtype} {ny}x{nx}: S {eS:.1e} D {eD:.1e} Dp {eDp:.1e}", flush=True)
    assert max(eS, eD, eDp) <= 1e-4  # bf16 hi + lo operands: about 16 bits
