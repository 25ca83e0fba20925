"""The plain FP32 form takes the radix FFT along the sweep where the length has one."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from test_gpu_render import FP32_BAR, random_case, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N", [(16, 16), (16, 32), (32, 64), (64, 128), (128, 32), (256, 64), (16, 2048), (256, 512)])
def test_fp32_equals_the_fft_form(gpu_lib, T, N):
    """Depth-first, frame order (dispersion), |V|, exact chirp, with dense-product shapes a user may have
    stored: the same volumes as SSOCT_DEPTH_FFT bit for bit, from the smaller workspace."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=700 + T + N)
    fr = torch.from_numpy(frames).cuda()
    disp = np.linspace(-2, 2, T) ** 2
    print(f"\n[gpu] fp32 route T={T} N={N}", flush=True)
    for kw, d in (({}, None), ({}, disp), ({"write_abs": True}, None), ({"exact_chirp": True}, None)):
        a, b = Plan(T, N, precision="fp32", **kw), Plan(T, N, precision="fp32_fft", **kw)
        assert a.workspace.numel() <= b.workspace.numel()
        V = b.render(fr, lam, 12e-6, 0.3, d).clone()
        assert torch.equal(a.render(fr, lam, 12e-6, 0.3, d), V), kw
        a.set_tuning([1, 0, 512, 0])            # one frame per chunk, dense workgroups, frame order
        assert torch.equal(a.render(fr, lam, 12e-6, 0.3, d), V), kw
        a.close(), b.close()
    if T * N * N <= 1 << 19:
        V = Plan(T, N).render(fr, lam, 12e-6, 0.3)
        assert rel_l2(V.cpu().numpy(), O.render(frames, lam, 12e-6, 0.3)) <= FP32_BAR


def test_fp32_route_without_allocation(gpu_lib):
    """render_noalloc where the static array leaves fewer frames per chunk than the default."""
    from paper_2003_08960_amd.api import Plan
    for T, N in ((16, 1024), (64, 512), (32, 128)):
        frames, lam = random_case(T, N, seed=710 + T)
        fr = torch.from_numpy(frames).cuda()
        print(f"\n[gpu] fp32 noalloc T={T} N={N}", flush=True)
        plan = Plan(T, N)
        V = plan.render(fr, lam, 12e-6, 0.3).clone()
        assert torch.equal(plan.render_noalloc(fr, lam, 12e-6, 0.3), V)
        assert torch.equal(plan.render_noalloc(fr, lam, 12e-6, 0.3), V)
