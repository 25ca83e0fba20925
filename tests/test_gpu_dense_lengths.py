"""Dense depth product at the lengths where its tile hand-over, operand packing and K chunk change: one,
two, four and eight waves of 32 rows, tiles of 32 to 256 frames, full and part-filled, several chunks."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from test_gpu_render import FP32_BAR, SPLIT_BAR, random_case, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,bar", [("fp32", FP32_BAR), ("bf16_split", SPLIT_BAR), ("fp16_split", SPLIT_BAR),
                                           ("fp16", None), ("bf16", None)])
@pytest.mark.parametrize("T", [1, 2, 31, 33, 60, 64, 65, 100, 127, 128, 129, 200, 257, 300])
def test_lengths(gpu_lib, T, precision, bar):
    """Each form against the oracle (the unsplit 16-bit ones, which have no bar, against their own split
    form: one rounding of 2^-9 or 2^-12 per operand); one workgroup walking every tile, three, and half
    the K chunk where there is one: the same bits."""
    from paper_2003_08960_amd import native
    from paper_2003_08960_amd.api import Plan
    if precision == "fp32" and T in (64, 128):
        pytest.skip("a radix FFT length: no dense FP32 product")
    N = 32
    frames, lam = random_case(T, N, seed=1500 + T)
    fr = torch.from_numpy(frames).cuda()
    print(f"\n[gpu] dense lengths {precision} T={T}", flush=True)
    plan = Plan(T, N, precision=precision)
    V0 = plan.render(fr, lam, 12e-6, 0.3).clone()
    if bar is not None:
        assert rel_l2(V0.cpu().numpy(), O.render(frames, lam, 12e-6, 0.3)) <= bar
    else:
        ref = Plan(T, N, precision=precision + "_split").render(fr, lam, 12e-6, 0.3).cpu().numpy()
        assert rel_l2(V0.cpu().numpy(), ref) <= 2 * 2.0 ** (-9 if precision == "bf16" else -12)
    kc = 32
    while kc < T and kc < 256:
        kc *= 2
    for tuning in ([0, 0, 1], [0, 0, 3], [0, 0, 0, 1, 0, 0, 0, kc // 2], [0, 0, 3, 1, 0, 0, 0, kc // 2]):
        if len(tuning) > 3 and kc // 2 < 32:
            with pytest.raises(native.SsoctError):
                plan.set_tuning(tuning)
            continue
        plan.set_tuning(tuning)
        assert torch.equal(plan.render(fr, lam, 12e-6, 0.3), V0), tuning
    plan.close()


def test_magnitude_and_gradient_of_a_ragged_length(gpu_lib):
    """The |V| epilogue and the Gamma pass with its adjoint over several tiles per workgroup."""
    from paper_2003_08960_amd.api import Plan
    for T in (60, 100, 200):
        N = 32
        frames, lam = random_case(T, N, seed=1600 + T)
        fr = torch.from_numpy(frames).cuda()
        print(f"\n[gpu] dense magnitude and gradient T={T}", flush=True)
        ref = O.render(frames, lam, 12e-6, 0.3)
        plan = Plan(T, N, precision="fp32", write_abs=True)
        plan.set_tuning([0, 0, 3])
        assert rel_l2(plan.render(fr, lam, 12e-6, 0.3).cpu().numpy(), np.abs(ref)) <= FP32_BAR
        plan = Plan(T, N, precision="fp32", backward=True)
        plan.set_tuning([0, 0, 3])
        g = plan.backward_sharpness(fr, lam, 12e-6, 0.3).cpu().numpy()
        L, dz, dc, _ = O.sharpness_grad(frames, lam, 12e-6, 0.3)
        assert abs(g[0] - L) <= FP32_BAR * L and abs(g[1] - dz) <= 1e-4 * abs(dz) and rel_l2(g[2:17], dc) <= 1e-4
