"""Row groups and chunks that follow the launch size: the forward, bin-pair, angular-spectrum and
adjoint row passes give every CU work also when a launch has few rows, and the depth-first order
keeps the two real bins in one plane, so chunks of planes of any size have to land in the volume."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from test_gpu_render import FP32_BAR, random_case, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eq6,aberr", [(False, False), (True, True)])
@pytest.mark.parametrize("T,N,F", [(16, 32, 0), (16, 64, 0), (32, 128, 6), (64, 128, 64), (32, 512, 10), (16, 1024, 2)])
def test_depth_first_planes_in_any_chunk(gpu_lib, T, N, F, eq6, aberr):
    """Chunks of F/2 planes: one row per group with the two transforms split (small launches) up to
    the default 4 rows, plane 0 (bins 0 and T/2) in the first chunk, a ragged last chunk; the volume is
    the same for every chunking and row group."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=900 + T + N)
    zern = np.random.default_rng(T).normal(0, 0.3, 15) if aberr else None
    fr = torch.from_numpy(frames).cuda()
    print(f"\n[gpu] planes T={T} N={N} F={F} eq6={eq6} aberr={aberr}", flush=True)
    plan = Plan(T, N, precision="fp32_fft", eq6_phase=eq6)
    V0 = plan.render(fr, lam, 12e-6, 0.3, None, zern).clone()
    assert rel_l2(V0.cpu().numpy(), O.render(frames, lam, 12e-6, 0.3, zernike_coeffs=zern, eq6_phase=eq6)) <= FP32_BAR
    for rpg in (0, 2, 8):
        plan.set_tuning([F, 0, 0, 1, rpg])
        assert torch.equal(plan.render(fr, lam, 12e-6, 0.3, None, zern), V0), rpg


@pytest.mark.parametrize("T,N", [(1, 16), (3, 32), (5, 64), (2, 128), (9, 256), (3, 512), (17, 512), (5, 1024), (2, 2048)])
def test_row_groups_of_small_launches(gpu_lib, T, N):
    """Frame order (aberrated) and angular spectrum where the row passes take 1, 2 or 4 rows per group."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=950 + T + N)
    fr = torch.from_numpy(frames).cuda()
    zern = np.random.default_rng(N).normal(0, 0.3, 15)
    print(f"\n[gpu] row groups T={T} N={N}", flush=True)
    V = Plan(T, N, precision="fp32").render(fr, lam, 12e-6, 0.3, None, zern)
    assert rel_l2(V.cpu().numpy(), O.render(frames, lam, 12e-6, 0.3, zernike_coeffs=zern)) <= FP32_BAR
    V = Plan(T, N, precision="fp32", angular_spectrum=True).render(fr, lam, 12e-6, 0.01)
    assert rel_l2(V.cpu().numpy(), O.render_as(frames, lam, 12e-6, 0.01)) <= FP32_BAR


@pytest.mark.parametrize("T,N", [(3, 32), (5, 64), (16, 64), (9, 128), (16, 256), (5, 512)])
def test_adjoint_row_groups(gpu_lib, T, N):
    """Sharpness gradient where the adjoint row pass takes 1, 2 or 4 rows per group: loss within the
    FP32 bar, gradients within 1e-4 (the bar of every gradient test: the moments cancel)."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=980 + T + N)
    fr = torch.from_numpy(frames).cuda()
    zern = np.random.default_rng(T).normal(0, 0.3, 15)
    disp = np.linspace(-1, 1, T) ** 2
    print(f"\n[gpu] adjoint row groups T={T} N={N}", flush=True)
    plan = Plan(T, N, precision="fp32", backward=True)
    g = plan.backward_sharpness(fr, lam, 12e-6, 0.3, disp, zern).cpu().numpy()
    ref = O.sharpness_grad(frames, lam, 12e-6, 0.3, disp, zern)
    assert abs(g[0] - ref[0]) <= FP32_BAR * abs(ref[0])
    assert abs(g[1] - ref[1]) <= 1e-4 * abs(ref[1])
    assert rel_l2(g[2:17], ref[2]) <= 1e-4
    assert rel_l2(g[17:], ref[3]) <= 1e-4


@pytest.mark.parametrize("precision,T", [("fp32", 2), ("bf16_split", 3), ("fp32_fft", 16)])
def test_two_columns_per_thread_at_2048(gpu_lib, precision, T):
    """N = 2048: the default column tile takes two adjacent columns per thread with 16-byte accesses;
    a volume at an odd complex64 of its allocation takes one column per thread; the narrower tiles do
    too.  All within the bar of the form, in both radix orders, and the gradient as well."""
    from paper_2003_08960_amd.api import Plan
    from test_gpu_render import SPLIT_BAR
    N = 2048
    frames, lam = random_case(T, N, seed=990 + T)
    fr = torch.from_numpy(frames).cuda()
    bar = SPLIT_BAR if precision.endswith("split") else FP32_BAR
    print(f"\n[gpu] two columns per thread T={T} {precision}", flush=True)
    ref = O.render(frames, lam, 12e-6, 0.6)
    plan = Plan(T, N, precision=precision, backward=True)
    odd = torch.empty(T * N * N + 1, dtype=torch.complex64, device="cuda")[1:].view(T, N, N)
    assert odd.data_ptr() % 16 == 8
    for out in (None, odd):
        for tile, radix in ((0, 0), (0, 1), (4, 0), (8, 0)):
            plan.set_tuning([0, 0, 0, 1, 0, tile, 0, 0, radix])
            assert rel_l2(plan.render(fr, lam, 12e-6, 0.6, out=out).cpu().numpy(), ref) <= bar, (tile, radix)
    if T == 2:
        g = plan.backward_sharpness(fr, lam, 12e-6, 0.6).cpu().numpy()
        L, dz, dc, dphi = O.sharpness_grad(frames, lam, 12e-6, 0.6)
        assert abs(g[0] - L) <= FP32_BAR * L and abs(g[1] - dz) <= 1e-4 * abs(dz) and rel_l2(g[2:17], dc) <= 1e-4


@pytest.mark.parametrize("gated,absolute", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("T,N", [(16, 16), (32, 32), (16, 64), (256, 64), (64, 512), (16, 2048)])
def test_gate_and_magnitude_depth_first(gpu_lib, T, N, gated, absolute):
    """A gate weighs the frames before their depth transform and |V| is written by the column pass; with
    the Eq. 6 factor (whose amplitude shares the gate's table entry), a zero first weight and negative
    ones.  Both evaluation orders meet the bar."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=1000 + T + N)
    fr = torch.from_numpy(frames).cuda()
    gate = np.sin(np.pi * np.arange(T) / T) ** 2 - 0.2 * (np.arange(T) % 3 == 1) if gated else None
    print(f"\n[gpu] gate and magnitude T={T} N={N}", flush=True)
    ref = O.render(frames, lam, 12e-6, 0.6, eq6_phase=True, gate=gate)
    ref = np.abs(ref) if absolute else ref
    plan = Plan(T, N, precision="fp32_fft", write_abs=absolute, eq6_phase=True)
    plan.set_gate(gate)
    for order in (1, 0):
        plan.set_tuning([0, 0, 0, order])
        assert rel_l2(plan.render(fr, lam, 12e-6, 0.6).cpu().numpy(), ref) <= FP32_BAR, order
    plan.set_gate(None)                         # and back to the rectangular gate of a fresh plan
    plan.set_tuning([0, 0, 0, 1])
    V = plan.render(fr, lam, 12e-6, 0.6).clone()
    assert torch.equal(V, Plan(T, N, precision="fp32_fft", write_abs=absolute, eq6_phase=True).render(fr, lam, 12e-6, 0.6))


@pytest.mark.parametrize("T,N", [(16, 64), (16, 512), (16, 1024), (32, 256), (32, 512), (64, 256), (64, 512), (128, 256),
                                 (128, 512)])
def test_tiles_per_workgroup_of_the_first_stage(gpu_lib, T, N):
    """Depth-first stage 1 with 1, 256/T and a quarter of 256/T tiles per workgroup (by launch size),
    tiles of one workgroup in one row and across rows: sampled pixel columns against the direct sums,
    and Parseval over the whole volume (the bar of the FP32 forms)."""
    from paper_2003_08960_amd.api import Plan
    frames, lam = random_case(T, N, seed=1100 + T + N)
    fr = torch.from_numpy(frames).cuda()
    print(f"\n[gpu] stage 1 tiles T={T} N={N}", flush=True)
    V = Plan(T, N, precision="fp32_fft").render(fr, lam, 12e-6, 0.3)
    rng = np.random.default_rng(T + N)
    pix = [(int(u), int(v)) for u, v in rng.integers(0, N, (6, 2))] + [(0, 0), (N - 1, N - 1)]
    got = np.stack([V[:, u, v].cpu().numpy() for u, v in pix], axis=1)
    assert rel_l2(got, O.render_columns(frames, lam, 12e-6, 0.3, pix)) <= FP32_BAR
    s = lam / lam.max()
    energy = sum(float(np.sum(O.rescale(frames[t], s[t]) ** 2)) for t in range(T)) * T * N * N
    assert abs(float((V.abs().double() ** 2).sum()) - energy) <= 2 * FP32_BAR * energy


@pytest.mark.parametrize("order", [0, 1])
def test_gated_stream_equals_the_gated_render(gpu_lib, order):
    """Host-fed streams of a gated FFT-form plan: chunk graphs (frame order) and the whole-volume graph
    (depth first), several sweeps through the same graphs."""
    from paper_2003_08960_amd.api import Plan, Stream
    T, N = 16, 128
    sweeps = [random_case(T, N, seed=760 + i) for i in range(3)]
    lam = sweeps[0][1]
    print(f"\n[gpu] gated stream order={order}", flush=True)
    plan = Plan(T, N, precision="fp32_fft")
    plan.set_tuning([0, 0, 0, order])
    plan.set_gate(np.hanning(T + 2)[1:-1])
    refs = [plan.render(torch.from_numpy(f).cuda(), lam, 12e-6, 0.3).clone() for f, _ in sweeps]
    st = Stream(plan, lam, 12e-6, 0.3, slots=2)
    for i, (f, _) in enumerate(sweeps):
        for a in range(0, T, 5):
            assert st.push_frames(np.ascontiguousarray(f[a:a + 5]), i * T + a) == 0
        r = st.pop(wait=True)
        assert r["seq"] == i and torch.equal(st.slot_volume(r["slot"]), refs[i])
    st.close(), plan.close()
