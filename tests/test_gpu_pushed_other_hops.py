"""Series pushed in pieces at hops other than L and L/2 (the general kernel): the frames
before a push come from the ring, whose rows wrap anywhere in a chunk, in immediate mode
(depth L) and in deferred mode (deeper, every frame from the ring). Against the FP64
oracle and against the whole series in one push."""

import numpy as np
import pytest
import torch

import oracle as O
import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


def reduce(tacaw, psi, L, H, masks, step, dtype, ring=0):
    P, NT, ny, nx = psi.shape
    with tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype, masks=masks, ring_frames=ring) as plan:
        for f in range(0, NT, step):
            plan.push(psi[:, f:f + step])
        S = plan.finalize().cpu().numpy().reshape(L, -1)
        D, Dp = plan.detector_spectra(per_probe=True)
        return S, D.cpu().numpy(), Dp.cpu().numpy()


@pytest.mark.parametrize("ring_chunks,step", [(0, "L//3"), (0, "L-1"), (0, "2*L+3"), (1.5, "L//2"), (2, "7*L//8")])
@pytest.mark.parametrize("L,H,dtype", [(64, 48, "c64"), (64, 1, "c64"), (128, 50, "c64"), (128, 127, "c128"),
                                       (200, 66, "c64"), (256, 64, "c128"), (512, 170, "c64"), (1024, 700, "c64")])
def test_pushed_series_matches_oracle_and_one_push(L, H, dtype, ring_chunks, step):
    from paper_2607_02236_amd import tacaw

    P, NT, ny, nx = 2, 3 * L + L // 3, 5, 7
    host = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=L + H, model="lines", n_terms=8))
    psi = host.cuda()
    m = np.stack([np.ones((ny, nx)), np.random.default_rng(L).random((ny, nx))])
    masks = torch.from_numpy(m).cuda()
    got = reduce(tacaw, psi, L, H, masks, eval(step, {"L": L}), dtype, int(ring_chunks * L))
    one = reduce(tacaw, psi, L, H, masks, NT, dtype)
    So, Spo = O.tacaw_spectra(host.numpy(), L, H, O.window("hann", L), fft=True)
    want = So, O.detector_spectra(So, m), np.transpose(O.detector_spectra(Spo, m), (1, 0, 2))
    for name, g, o, w in zip(("S", "D", "Dp"), got, one, want):
        e, e1 = rel(g, w), rel(g, o)
        print(f"L={L} H={H} {dtype} ring {ring_chunks} step {step}: {name} vs oracle {e:.1e}, vs one push {e1:.1e}",
              flush=True)
        assert e <= 1e-5 and e1 <= 1e-12  # the same FP32 transform of the same chunks
