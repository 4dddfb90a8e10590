"""DFT-GEMM form with all eight waves of a workgroup at work: 256 tiles are one workgroup
for each CU, so the row-group rule leaves 8 row blocks (127 output rows) in one group. The
last tile holds 50 pixels; several probes, one mask that is zero on most tiles."""

import numpy as np
import pytest
import torch

import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


@pytest.mark.parametrize("form,dtype", [("gemm_bf16x3", "c64"), ("gemm_bf16x3", "c128"),
                                        ("gemm_f16x3", "c64"), ("gemm_f16x3", "c128")])
@pytest.mark.parametrize("L,H", [(256, 128), (512, 512)])
def test_eight_blocks_in_one_group_match_fft_form(form, dtype, L, H):
    from paper_2607_02236_amd import tacaw

    M, P, ny, nx = 63, 2, 10, 3269
    NT = 2 * L + 8
    psi = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=L, model="lines", n_terms=8), device="cuda")
    gen = torch.Generator("cuda").manual_seed(L)
    masks = torch.rand((2, ny, nx), dtype=torch.float64, device="cuda", generator=gen)
    masks[1, 1:] = 0.0
    out = []
    for f in (form, "fft"):
        with tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype, transform=f, omega_half=M, masks=masks) as plan:
            plan.push(psi)
            S = plan.finalize()
            D, Dp = plan.detector_spectra(per_probe=True)
            out.append([t.cpu().numpy() for t in (S, D, Dp)])
    for name, x, y in zip(("S", "D", "Dp"), *out):
        # and output row by row (each is one row of one wave's block): the operands' 16 bits
        # leave a row of 1e-4 of the strongest one's power an error of 2^-16 / 1e-2
        axis = 0 if name == "S" else -1
        n = [np.linalg.norm(np.take(y, r, axis)) for r in range(2 * M + 1)]
        e = max(rel(np.take(x, r, axis), np.take(y, r, axis)) for r in range(2 * M + 1) if n[r] >= 1e-4 * max(n))
        print(f"{form} {dtype} L={L}: {name} {rel(x, y):.1e}, worst row {e:.1e}", flush=True)
        assert rel(x, y) <= 1e-5 and e <= 1e-2
