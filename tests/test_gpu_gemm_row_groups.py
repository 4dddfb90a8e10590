"""DFT-GEMM form at the edges of its row blocks (32 GEMM rows, 16 output rows, at most 8
blocks per workgroup) and pixel tiles (128): one block, one row into the next block, 8, 9
and 17 blocks, which such small grids spread one to a group; with waves that only
stage, detector partials and several probes. (Groups of 8: test_gpu_gemm_full_groups.py.)"""

import numpy as np
import pytest
import torch

import oracle as O
import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


# output rows 2 M + 1: 15, 17 (1 and 2 blocks), 127, 129 (8 and 9), 257 (17)
@pytest.mark.parametrize("M", [7, 8, 63, 64, 128])
@pytest.mark.parametrize("form,dtype,ny,nx", [("gemm_bf16x3", "c64", 11, 12), ("gemm_bf16x3", "c128", 8, 16),
                                              ("gemm_f16x3", "c64", 3, 43)])
def test_row_groups_match_oracle(form, dtype, ny, nx, M):
    from paper_2607_02236_amd import tacaw

    L, H, P = 512, 256, 2
    NT = 2 * L + 40
    spec = T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=M + nx, model="lines", n_terms=8)
    host = T.generate(spec)
    m = np.stack([np.ones((ny, nx)), np.random.default_rng(M).random((ny, nx))])
    plan = tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype, transform=form, omega_half=M,
                      masks=torch.from_numpy(m).cuda())
    for _ in range(2):  # the second pass finds the first one's sums in the buffers
        plan.reset()
        plan.push(host.cuda())
        S = plan.finalize().cpu().numpy().reshape(2 * M + 1, -1)
        D, Dp = plan.detector_spectra(per_probe=True)
    rows = np.mod(np.arange(-M, M + 1), L)
    So, Spo = O.tacaw_spectra(host.numpy(), L, H, O.window("hann", L), fft=True)
    So, Spo = So[rows], Spo[:, rows]
    eS, eD = rel(S, So), rel(D.cpu().numpy(), O.detector_spectra(So, m))
    eDp = rel(Dp.cpu().numpy(), np.transpose(O.detector_spectra(Spo, m), (1, 0, 2)))
    plan.close()
    print(f"{form} {dtype} {ny}x{nx} M={M}: S {eS:.1e} D {eD:.1e} Dp {eDp:.1e}", flush=True)
    assert eS <= 1e-5 and eD <= 1e-5 and eDp <= 1e-5


# 257 tiles, one more than a round of workgroups: 8, 9 and 17 blocks in groups of 4, 5 and 6;
# against the FFT form
@pytest.mark.parametrize("M", [63, 64, 128])
@pytest.mark.parametrize("form", ["gemm_bf16x3", "gemm_f16x3"])
def test_full_row_groups_match_fft_form(form, M):
    from paper_2607_02236_amd import tacaw

    L, H, P, ny, nx = 512, 256, 1, 128, 257
    NT = 2 * L + 40
    psi = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype="c64", seed=M, model="lines", n_terms=8), device="cuda")
    masks = torch.rand(1, ny, nx, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(M))
    out = []
    for f in (form, "fft"):
        plan = tacaw.Plan(P, ny, nx, NT, L, H, in_dtype="c64", transform=f, omega_half=M, masks=masks)
        plan.push(psi)
        S = plan.finalize().cpu().numpy()
        D, Dp = plan.detector_spectra(per_probe=True)
        out.append((S, D.cpu().numpy(), Dp.cpu().numpy()))
        plan.close()
    for x, y in zip(*out):
        assert rel(x, y) <= 1e-5
