"""Large inputs in whole cache lines are loaded past the caches; the same series at an
address 8 or 16 bytes off a line takes the ordinary loads. The arithmetic is the same,
so the sums are too, bit for bit (each value of S is summed by one thread, in order).
A corner of the grid is also checked against a transform in FP64."""

import pytest
import torch

pytestmark = pytest.mark.gpu

LINE = 128


def reduce_S(tacaw, psi, L, H, dtype):
    P, NT, ny, nx = psi.shape
    plan = tacaw.Plan(P, ny, nx, NT, L, H, in_dtype=dtype)
    plan.push(psi)
    S = plan.finalize().clone()
    plan.close()
    return S


@pytest.mark.parametrize("L,full,dtype", [(64, False, "c64"), (128, True, "c64"), (200, False, "c64"), (256, False, "c128"),
                                          (512, True, "c64"), (512, False, "c128"), (1024, True, "c128")])
def test_loads_past_the_caches_give_the_same_sums(L, full, dtype):
    from paper_2607_02236_amd import tacaw

    H = L if full else L // 2
    ct = torch.complex64 if dtype == "c64" else torch.complex128
    esz = 8 if dtype == "c64" else 16
    ny, nx, P = 64, 96, 2
    s = -(-((512 << 20) // (P * ny * nx * esz) + 1 - L) // H) + 1  # chunks: at least 512 MiB
    NT = (s - 1) * H + L
    assert NT * P * ny * nx * esz >= 512 << 20
    buf = torch.empty(P * NT * ny * nx + 1, dtype=ct, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(L)
    torch.view_as_real(buf).normal_(generator=g)
    aligned = buf[:-1].view(P, NT, ny, nx)
    assert aligned.data_ptr() % LINE == 0
    S = reduce_S(tacaw, aligned, L, H, dtype)
    off = torch.empty_like(buf)
    off[1:] = buf[:-1]
    shifted = off[1:].view(P, NT, ny, nx)
    assert shifted.data_ptr() % LINE == esz
    assert torch.equal(S, reduce_S(tacaw, shifted, L, H, dtype))
    del off, shifted

    # a corner of the grid by torch in FP64: mean removed, Hann window, every chunk
    z = aligned[:, :, :2, :5].reshape(P, NT, 10).to(torch.complex128)
    z = z - z.mean(dim=1, keepdim=True)
    w = torch.hann_window(L, periodic=True, dtype=torch.float64, device="cuda")
    ref = torch.zeros(L, 10, dtype=torch.float64, device="cuda")
    for i in range(s):
        ref += torch.fft.fft(z[:, i * H:i * H + L] * w[None, :, None], dim=1).abs().square().sum(0)
    got = S.reshape(L, ny, nx)[:, :2, :5].reshape(L, 10)
    got, ref = got / got.sum(), ref / ref.sum()
    # FP32 transform: each |X|^2 within a few 1e-7 of itself, the sums as well
    assert float((got - ref).norm() / ref.norm()) < 2e-6
