"""The adjoint where one workgroup takes several probes (grids of 512 tiles or more: all of
them; smaller ones: a share, the last one less): the prefetch across the change of
probe, the carried half gradient, per-probe weights and every mean term. Bit for bit
against one call per probe, and (L = 64) against the FP64 oracle. And its scratch: calls with fewer
probes fit what a larger one made, and the fixed scratch falls back to one share."""

import numpy as np
import pytest
import torch

import oracle as O
import tacaw_synth as T

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((np.asarray(a) - np.asarray(b)).ravel()) / np.linalg.norm(np.asarray(b).ravel()))


# (ny, nx, P): 576 tiles of 16 pixels, 3 probes a workgroup; 200 tiles, shares 2, 2, 1
@pytest.mark.parametrize("ny,nx,P", [(96, 96, 3), (50, 64, 5)])
@pytest.mark.parametrize("L,H,mode,window,r,dtype", [
    (64, 32, "global", "hann", 1.0, "c64"),          # mean term from the bin sums
    (64, 32, "global", "hann_width", 1.0, "c64"),
    (64, 64, "global", "hann_width", 1.0, "c128"),
    (64, 32, "global", "hann_width", 1.1, "c64"),    # mean term in a second pass
    (64, 64, "global", "tukey", 0.3, "c64"),
    (64, 32, "global", "hann", 1.0, "c128"),
    (64, 32, "per_segment", "hann", 1.0, "c64"),
    (64, 64, "per_segment", "hann", 1.0, "c64"),
    (64, 32, "none", "hann", 1.0, "c64"),
    (256, 128, "global", "hann", 1.0, "c64"),
    (256, 128, "global", "hann", 1.0, "c128"),
    (512, 256, "global", "hann", 1.0, "c64"),
])
def test_probe_loop_matches_oracle_and_single_calls(ny, nx, P, L, H, mode, window, r, dtype):
    from paper_2607_02236_amd import tacaw

    NT = 2 * L + L // 2 + 5
    x = T.generate(T.SeriesSpec(P, NT, ny, nx, dtype=dtype, seed=L + H + P, model="lines", n_terms=4), device="cuda")
    rng = np.random.default_rng(P)
    m = rng.random((2, ny, nx)) * (rng.random((2, ny, 1)) > 0.3)
    gS, gD, gP = rng.random((L, ny * nx)) * 0.1, rng.random((2, L)), rng.random((2, P, L)) * 0.3
    dev = [torch.from_numpy(v).cuda() for v in (gS.reshape(L, ny, nx), gD, gP)]
    with tacaw.Plan(P, ny, nx, NT, L, H, window=window, window_param=r, mean_mode=mode, in_dtype=dtype,
                    masks=torch.from_numpy(m).cuda()) as plan:
        plan.push(x)
        plan.finalize()
        g, gw = plan.backward(x, gS=dev[0], gD=dev[1], gDp=dev[2])
        one, w1 = [], 0.0
        for p in range(P):
            gp, wp = plan.backward(x[p:p + 1], probe0=p, gS=dev[0], gD=dev[1], gDp=dev[2])
            one.append(gp)
            w1 += float(wp)
        one = torch.cat(one)
        assert torch.equal(torch.view_as_real(g), torch.view_as_real(one))
    if L > 64:
        return  # the single calls stand in for the oracle
    w = O.window(window, L, r)
    dw = O.window_width_derivative(L, r) if window == "hann_width" else None
    Mf = m.reshape(2, -1)
    want, dr, lval = O.spectra_vjp(x.cpu().numpy(), L, H, w, gS + np.einsum("jm,jk->mk", gD, Mf),
                                   np.einsum("jpm,jk->pmk", gP, Mf), mode, dw=dw)
    e = rel(g.cpu().numpy(), want)
    print(f"L={L} H={H} {mode} {window} {dtype} {ny}x{nx} P={P}: {e:.1e}", flush=True)
    assert e <= 1e-5
    if dw is not None:
        assert float(gw) == pytest.approx(dr, rel=2e-5, abs=1e-9 * abs(lval))
        assert w1 == pytest.approx(float(gw), rel=1e-9, abs=1e-12 * abs(lval))


def test_scratch_does_not_grow_for_fewer_probes():
    # one tile: 600 probes are evened out to 300 shares of 2, 512 probes to 512 of 1
    from paper_2607_02236_amd import tacaw

    L, P = 64, 600
    x = T.generate(T.SeriesSpec(P, L, 1, 1, dtype="c64", seed=1, model="lines", n_terms=2)).cuda()
    with tacaw.Plan(P, 1, 1, L, L, L) as plan:
        plan.push(x)
        S = plan.finalize()
        plan.backward(x, gS=S)
        size = plan.info()["device_bytes"]
        for n in (599, 512, 300, 7):
            plan.backward(x[:n], gS=S)
            assert plan.info()["device_bytes"] == size


def test_fixed_scratch_falls_back_to_one_share():
    # 256 probes x 4095 pixels in 256 tiles: the fixed 16 MiB hold one partial per tile, not two
    from paper_2607_02236_amd import tacaw

    L, P, ny, nx = 64, 256, 63, 65
    gen = torch.Generator("cuda").manual_seed(3)
    x = torch.complex(torch.randn((P, L, ny, nx), device="cuda", generator=gen),
                      torch.randn((P, L, ny, nx), device="cuda", generator=gen))
    with tacaw.Plan(P, ny, nx, L, L, L, window="hann_width", window_param=1.1) as plan:
        plan.push(x)
        S = plan.finalize()
        g0, w0 = plan.backward(x, gS=S)
        g1, w1 = plan.backward(x, gS=S, static_scratch=True)
        assert torch.equal(torch.view_as_real(g0), torch.view_as_real(g1))
        assert float(w1) == pytest.approx(float(w0), rel=1e-9)
