"""At L = 1024 a pushed series has the bits of one push too: every variant that a chunk of
it can take folds its four column quarters in the same order, with the same twiddle row."""

import numpy as np
import pytest
import torch

import tacaw_synth as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("first,step", [(1024, 1024), (1025, 515), (511, 256), (1536, 2049)])
def test_pushed_series_equals_one_push(dtype, full, first, step):
    from paper_2607_02236_amd import tacaw

    L, P, NT, ny, nx = 1024, 2, 4437, 5, 7
    H = L if full else L // 2
    psi = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=H, model="lines", n_terms=8)).cuda()
    masks = torch.ones((1, ny, nx), dtype=torch.float64, device="cuda")
    out = []
    for cuts in ([0, *range(first, NT, step), NT], [0, NT]):
        with tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype, masks=masks) as plan:
            for f, g in zip(cuts, cuts[1:]):
                plan.push(psi[:, f:g])
            S = plan.finalize()
            D, Dp = plan.detector_spectra(per_probe=True)
            out.append([t.cpu().numpy() for t in (S, D, Dp)])
    for name, g, o in zip(("S", "D", "Dp"), *out):
        e = float(np.linalg.norm(g - o) / np.linalg.norm(o))
        print(f"{dtype} H={H} {first}+{step}: {name} {e:.1e}", flush=True)
        assert e <= 1e-12  # the FP64 sums are grouped by launch
