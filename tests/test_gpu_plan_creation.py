"""What a plan's creation leaves behind: no host copies of its tables."""

import os

import pytest
import torch

pytestmark = pytest.mark.gpu


def resident_bytes():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * os.sysconf("SC_PAGE_SIZE")


def test_plans_keep_no_host_copy_of_their_tables():
    # the DFT matrix of L = 1024 with all bins is 16.8 MB; 12 open plans would hold 200 MB
    from paper_2607_02236_amd import tacaw

    def make():
        return tacaw.Plan(1, 2, 2, 1024, 1024, 512, transform="gemm_bf16x3")

    keep = [make(), make()]
    torch.cuda.synchronize()
    before = resident_bytes()
    keep += [make() for _ in range(12)]
    grown = resident_bytes() - before
    print(f"12 plans: {grown / 1e6:.1f} MB of host memory", flush=True)
    for p in keep:
        p.close()
    assert grown < 12 * 16.8e6 / 4
