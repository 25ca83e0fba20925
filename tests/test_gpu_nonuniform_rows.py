"""The paired rows of the depth matrix of a sweep not linear in k: bins about the centre (T - 1) / 2,
half-integer for even T and integer for odd T, with the rest of the phase carried by the frames."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from paper_2003_08960_amd import synth
from test_gpu_render import FP32_BAR, SPLIT_BAR, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bar", [("fp32", FP32_BAR), ("bf16_split", SPLIT_BAR), ("fp16_split", SPLIT_BAR)])
@pytest.mark.parametrize("T", [2, 3, 31, 32, 257, 300])
def test_every_row_pair(gpu_lib, T, precision, bar):
    """Dispersion and a gate on top (the same per-frame phase and amplitude), Fresnel and angular
    spectrum; lengths around the 32-row blocks of the matrix and beyond one slab of it."""
    from paper_2003_08960_amd.api import Plan
    N = 16
    frames = synth.random_frames(T, N, seed=T)
    lam = synth.sweep_wavelengths(T, 870e-9, 800e-9, bend=0.2)
    rng = np.random.default_rng(T)
    disp, gate = rng.uniform(-3, 3, T), rng.uniform(0.2, 1.0, T)
    fr = torch.from_numpy(frames).cuda()
    print(f"\n[gpu] nonuniform rows T={T} {precision}", flush=True)
    plan = Plan(T, N, precision=precision, nonuniform_k=True)
    plan.set_gate(gate)
    V = plan.render(fr, lam, 20e-6, 0.05, disp)
    assert rel_l2(V.cpu().numpy(), O.render(frames, lam, 20e-6, 0.05, disp, gate=gate, nonuniform_k=True)) <= bar
    plan = Plan(T, N, precision=precision, nonuniform_k=True, angular_spectrum=True)
    V = plan.render(fr, lam, 20e-6, 0.01, disp)
    assert rel_l2(V.cpu().numpy(), O.render_as(frames, lam, 20e-6, 0.01, disp, nonuniform_k=True)) <= bar
