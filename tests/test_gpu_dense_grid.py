"""Dense depth product on any number of workgroups (tuning entry 2), down to fewer than the row slabs of
256 rows that the matrix of a long sweep is split into: every bin is computed, whatever the count."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from paper_2003_08960_amd import synth
from test_gpu_render import FP32_BAR, SPLIT_BAR, random_case, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,T,slabs,nonuniform", [
    ("fp32", 20, 1, False), ("fp32", 100, 1, False), ("fp32", 300, 2, False), ("bf16_split", 300, 2, False),
    ("fp32", 600, 3, False), ("fp32", 1024, 4, False), ("bf16", 256, 2, True), ("bf16_split", 257, 3, True),
    ("bf16_split", 1024, 8, True), ("fp32", 300, 2, True)])
def test_dense_workgroups_change_no_bit(gpu_lib, precision, T, slabs, nonuniform):
    """1, 2, 3, fewer than the slabs, one more, a multiple of 8 slabs (slabs of one XCD) and more than
    the tiles: the volume of the default count bit for bit, into a buffer of NaN."""
    from paper_2003_08960_amd.api import Plan
    N = 32
    frames, lam = random_case(T, N, seed=1200 + T)
    if nonuniform:
        lam = synth.sweep_wavelengths(T, 870e-9, 800e-9, bend=0.2)
    fr = torch.from_numpy(frames).cuda()
    plan = Plan(T, N, precision=precision, nonuniform_k=nonuniform)
    V0 = plan.render(fr, lam, 12e-6, 0.3).clone()
    if precision != "bf16":
        ref = O.render(frames, lam, 12e-6, 0.3, nonuniform_k=nonuniform)
        assert rel_l2(V0.cpu().numpy(), ref) <= (SPLIT_BAR if "split" in precision else FP32_BAR)
    out = torch.empty_like(V0)
    for grid in sorted({1, 2, 3, max(1, slabs - 1), slabs, slabs + 1, 8 * slabs, 16 * slabs, 4096}):
        print(f"\n[gpu] dense workgroups {precision} T={T} grid={grid}", flush=True)
        plan.set_tuning([0, 0, grid])
        out.fill_(complex(float("nan"), float("nan")))
        assert torch.equal(plan.render(fr, lam, 12e-6, 0.3, out=out), V0), grid
    plan.close()


@pytest.mark.parametrize("T", [100, 300, 600])
def test_gradients_on_any_number_of_dense_workgroups(gpu_lib, T):
    """The Gamma pass and the adjoint product take the same count.  The loss is one FP64 partial per
    workgroup, so its sum of T N^2 terms of one sign runs in another order: at most T N^2 2^-53 apart."""
    from paper_2003_08960_amd.api import Plan
    N = 32
    frames, lam = random_case(T, N, seed=1300 + T)
    fr = torch.from_numpy(frames).cuda()
    rng = np.random.default_rng(T)
    G = torch.from_numpy((rng.standard_normal((T, N, N)) + 1j * rng.standard_normal((T, N, N))).astype(np.complex64)).cuda()
    disp, zern = rng.uniform(-1, 1, T), rng.normal(0, 0.3, 15)
    plan = Plan(T, N, precision="fp32", backward=True)
    g0 = plan.backward_sharpness(fr, lam, 12e-6, 0.3, disp, zern).clone()
    v0 = plan.backward(fr, lam, 12e-6, 0.3, G, disp, zern).clone()
    L, dz, dc, dphi = O.sharpness_grad(frames, lam, 12e-6, 0.3, disp, zern)
    g = g0.cpu().numpy()
    assert abs(g[0] - L) <= FP32_BAR * L and abs(g[1] - dz) <= 1e-4 * abs(dz) and rel_l2(g[17:], dphi) <= 1e-4
    for grid in (1, 2, 3, 5, 24, 1000):
        print(f"\n[gpu] gradient on dense workgroups T={T} grid={grid}", flush=True)
        plan.set_tuning([0, 0, grid])
        plan.workspace.fill_(255)               # NaN in every stack
        g = plan.backward_sharpness(fr, lam, 12e-6, 0.3, disp, zern)
        assert torch.equal(g[1:], g0[1:]), grid
        assert abs(float(g[0] - g0[0])) <= T * N * N * 2.0 ** -53 * float(g0[0]), grid
        plan.workspace.fill_(255)
        assert torch.equal(plan.backward(fr, lam, 12e-6, 0.3, G, disp, zern), v0), grid
    plan.close()
