"""Series pushed in pieces whose boundaries fall anywhere in a chunk: the launch's
first chunk takes its earlier frames from the ring and the rest from the push
(row groups before, after and across the boundary), every later chunk from the push.
S, D and D_p against the FP64 oracle and against the whole series in one push."""

import numpy as np
import pytest
import torch

import oracle as O
import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


def reduce(tacaw, psi, L, H, masks, pieces, dtype, row_stride=0):
    P, NT, ny, nx = psi.shape
    plan = tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype, masks=masks, k_row_stride=row_stride)
    f = 0
    for n in pieces:
        plan.push(psi[:, f:f + n])
        f += n
    assert f == NT
    S = plan.finalize().cpu().numpy().reshape(L, -1)
    D, Dp = plan.detector_spectra(per_probe=True)
    out = S, D.cpu().numpy(), Dp.cpu().numpy()
    plan.close()
    return out


def pieces_of(NT, first, step):
    out, f = [min(first, NT)], min(first, NT)
    while f < NT:
        out.append(min(step, NT - f))
        f += out[-1]
    return out


# (first piece, later pieces) as functions of L: boundaries on a row group, one frame
# off it, inside the first chunk's first half, and a push that completes two chunks
@pytest.mark.parametrize("first,step", [("L", "L"), ("L+1", "L//2+3"), ("L//2-1", "L//4"), ("L+L//2", "2*L+1")])
@pytest.mark.parametrize("L,full,dtype", [(64, False, "c64"), (128, True, "c64"), (200, False, "c64"),
                                          (200, True, "c128"), (256, False, "c128"), (512, False, "c64"),
                                          (512, True, "c64"), (1024, False, "c64"), (1024, False, "c128")])
def test_pushed_series_matches_oracle_and_one_push(L, full, dtype, first, step):
    from paper_2607_02236_amd import tacaw

    H = L if full else L // 2
    P, NT, ny, nx = 2, 4 * L + L // 3, 5, 7
    spec = T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=L + H, model="lines", n_terms=8)
    host = T.generate(spec)
    psi = host.cuda()
    m = np.stack([np.ones((ny, nx)), np.random.default_rng(L).random((ny, nx))])
    masks = torch.from_numpy(m).cuda()
    pieces = pieces_of(NT, eval(first, {"L": L}), eval(step, {"L": L}))
    got = reduce(tacaw, psi, L, H, masks, pieces, dtype)
    one = reduce(tacaw, psi, L, H, masks, [NT], dtype)
    So, Spo = O.tacaw_spectra(host.numpy(), L, H, O.window("hann", L), fft=True)
    want = So, O.detector_spectra(So, m), np.transpose(O.detector_spectra(Spo, m), (1, 0, 2))
    for name, g, o, w in zip(("S", "D", "Dp"), got, one, want):
        e, e1 = rel(g, w), rel(g, o)
        print(f"L={L} H={H} {dtype} {pieces[:3]}: {name} vs oracle {e:.1e}, vs one push {e1:.1e}", flush=True)
        assert e <= 1e-5
        # the same FP32 transform of the same chunks (the twiddle rows of L = 1024 may round apart)
        assert e1 <= 1e-6 if L == 1024 else e1 <= 1e-12


def test_pushed_k_space_window_in_place():
    # pixel rows of a wider grid: the push is strided, the ring contiguous
    from paper_2607_02236_amd import tacaw

    L, H, P, NT, ny, nx = 256, 128, 2, 900, 6, 9
    spec = T.SeriesSpec(P, NT, ny, 16, dtype="c64", seed=3, model="lines", n_terms=8)
    psi = T.generate(spec).cuda()
    cut = psi[:, :, :, 2:2 + nx]
    masks = torch.ones((1, ny, nx), dtype=torch.float64, device="cuda")
    got = reduce(tacaw, cut, L, H, masks, [300, 77, 523], "c64", row_stride=16)
    want = reduce(tacaw, cut.contiguous(), L, H, masks, [NT], "c64")
    for g, w in zip(got, want):
        assert rel(g, w) <= 1e-12
