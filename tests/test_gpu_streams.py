"""A plan on another stream than the one that makes its inputs: a plan's creation waits
for the work enqueued on the device before it, so frames and masks made just before
it, on any stream, are whole when the plan's stream reads them, and what the current
stream still uses is not written over."""

import contextlib

import pytest
import torch

import tacaw_synth as T

pytestmark = pytest.mark.gpu

L, H, P, NT, NY, NX = 128, 64, 2, 640, 24, 20


def busy():
    # some tens of milliseconds of work on the current stream
    a = torch.ones((8192, 8192), device="cuda")
    for _ in range(12):
        a = torch.mm(a, a).clamp_(max=1.0)


@pytest.mark.parametrize("made_on", ["default", "side"])
@pytest.mark.parametrize("with_masks", [False, True])
@pytest.mark.parametrize("kept", [False, True])
def test_inputs_made_just_before_on_the_current_stream(made_on, with_masks, kept):
    from paper_2607_02236_amd import tacaw

    src = T.generate(T.SeriesSpec(P, NT, NY, NX, dtype="c64", seed=5, model="lines", n_terms=8)).cuda()
    msrc = torch.from_numpy(T.standard_masks(NY, NX, scale=0.15)).cuda()
    want = tacaw.spectra(src, L, H, masks=msrc, per_probe=True)
    x, m = torch.full_like(src, float("nan")), torch.full_like(msrc, float("nan"))
    busy()  # (the library and the matrix product are warm)
    plan_stream, maker = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(maker) if made_on == "side" else contextlib.nullcontext():
        busy()
        x.copy_(src)
        m.copy_(msrc)
        masks = m if with_masks else None
        if kept:
            plan = tacaw.Plan(P, NY, NX, NT, L, H, masks=masks, stream=plan_stream)
            plan.push(x)
            S = plan.finalize()
            got = (S, *plan.detector_spectra(per_probe=True)) if with_masks else (S,)
            plan_stream.synchronize()
            plan.close()
        else:
            got = tacaw.spectra(x, L, H, masks=masks, per_probe=with_masks, stream=plan_stream)
            got = got if with_masks else (got,)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0])
    for g, w in zip(got[1:], want[1:]):  # FP64 atomic sums: their order may vary
        assert float((g - w).norm() / w.norm()) <= 1e-13
