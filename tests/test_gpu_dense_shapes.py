"""Launch shapes of plain FP32 plans whose length has no radix FFT along the sweep (they take the dense
product, frame by frame), and the narrow column tiles at N = 2048."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from test_gpu_render import FP32_BAR, SPLIT_BAR, random_case, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N", [(24, 128), (60, 64), (300, 32)])
def test_tuning_of_the_dense_form_changes_speed_not_results(gpu_lib, T, N, tmp_path):
    """Frames per chunk, column and depth workgroups, the tuner's pick and its file: the same bits."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=1700 + T)
    fr = torch.from_numpy(frames).cuda()
    print(f"\n[gpu] dense tuning T={T} N={N}", flush=True)
    plan = Plan(T, N)
    V0 = plan.render(fr, lam, 12e-6, 0.3).clone()
    assert rel_l2(V0.cpu().numpy(), O.render(frames, lam, 12e-6, 0.3)) <= FP32_BAR
    for tuning in ([1, 0, 0], [3, 7, 5], [T, 1024, 64], [0, 0, 4096, 0]):
        plan.set_tuning(tuning)
        assert torch.equal(plan.render(fr, lam, 12e-6, 0.3), V0), tuning
    plan.set_tuning([0, 0, 0])
    cache = str(tmp_path / "tuning.json")
    choice = plan.tune(fr, lam, 12e-6, 0.3, cache_path=cache)
    V = plan.render(fr, lam, 12e-6, 0.3)
    if choice[8] == 0:
        assert torch.equal(V, V0), choice
    else:                                   # the other radix order of the column transforms rounds differently
        assert rel_l2(V.cpu().numpy(), V0.cpu().numpy()) <= 2e-6, choice
    assert Plan(T, N).tune(fr, lam, 12e-6, 0.3, cache_path=cache) == choice
    plan.close()


@pytest.mark.parametrize("N", [32, 64, 128, 512, 1024])
def test_radix_orders_of_the_dense_form(gpu_lib, N):
    """Both radix orders of the column transforms in front of the dense FP32 product (T = 24)."""
    from paper_2003_08960_amd.api import Plan
    T = 24
    frames, lam = random_case(T, N, seed=1800 + N)
    fr = torch.from_numpy(frames).cuda()
    print(f"\n[gpu] dense radix orders N={N}", flush=True)
    ref = O.render(frames, lam, 20e-6, 0.05)
    plan = Plan(T, N, precision="fp32")
    for radix in (0, 1):
        plan.set_tuning([0, 0, 0, 0, 0, 0, 0, 0, radix])
        assert rel_l2(plan.render(fr, lam, 20e-6, 0.05).cpu().numpy(), ref) <= FP32_BAR, radix
    plan.close()


@pytest.mark.parametrize("precision,T,eq6", [("fp32", 2, False), ("bf16_split", 3, True), ("fp32_fft", 16, True)])
def test_narrowest_column_tile_at_2048(gpu_lib, precision, T, eq6):
    """Column tiles of 2 (the default's exchange buffer holds 8) in both radix orders, with and without
    the Eq. 6 factor."""
    from paper_2003_08960_amd.api import Plan
    N = 2048
    frames, lam = random_case(T, N, seed=1900 + T)
    fr = torch.from_numpy(frames).cuda()
    bar = SPLIT_BAR if precision.endswith("split") else FP32_BAR
    print(f"\n[gpu] narrowest column tile {precision} T={T}", flush=True)
    ref = O.render(frames, lam, 12e-6, 0.6, eq6_phase=eq6)
    plan = Plan(T, N, precision=precision, eq6_phase=eq6)
    for tile, radix in ((2, 0), (2, 1), (4, 1), (0, 1)):
        plan.set_tuning([0, 0, 0, 1, 0, tile, 0, 0, radix])
        assert rel_l2(plan.render(fr, lam, 12e-6, 0.6).cpu().numpy(), ref) <= bar, (tile, radix)
    plan.close()
