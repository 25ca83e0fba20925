"""Host-fed sweeps that take several chunks of the frame order: the Fresnel stage of a chunk starts when
the chunk has landed, also for plans whose renders take the depth-first order (a gate, plain FP32)."""
import numpy as np
import pytest
import torch

from oracle import ssoct_oracle as O
from paper_2003_08960_amd import native
from test_gpu_render import FP32_BAR, random_case, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,gated", [("fp32", False), ("fp32", True), ("fp32_fft", True)])
@pytest.mark.parametrize("F", [0, 5])
def test_chunks_start_while_frames_arrive(gpu_lib, precision, gated, F):
    """T = 32, N = 1024: two default chunks of 16 frames, or seven of 5 (the last one ragged).  The volume
    of a host-fed sweep has the frame order's bits, so its chunks ran one by one; a device-filled slot,
    where every frame is there at once, the depth-first order's.  A sweep is cut short after its
    first chunk, then the same slot is host-fed, device-filled and host-fed again."""
    from paper_2003_08960_amd.api import Plan, Stream
    T, N = 32, 1024
    sweeps = [random_case(T, N, seed=1400 + i)[0] for i in range(3)]
    lam = random_case(T, N, seed=1400)[1]
    gate = np.hanning(T + 2)[1:-1] if gated else None
    print(f"\n[gpu] stream chunks {precision} gated={gated} F={F}", flush=True)
    frame_order = Plan(T, N, precision="fp32_fft")
    frame_order.set_tuning([0, 0, 0, 0])
    frame_order.set_gate(gate)
    plan = Plan(T, N, precision=precision)
    plan.set_tuning([F])
    plan.set_gate(gate)
    dev = [torch.from_numpy(f).cuda() for f in sweeps]
    want = [frame_order.render(f, lam, 12e-6, 0.3).cpu() for f in dev]
    eager = [plan.render(f, lam, 12e-6, 0.3).cpu() for f in dev]
    pix = [(3, 5), (512, 512), (700, 1), (1023, 1023)]
    ref = O.render_columns(sweeps[0], lam, 12e-6, 0.3, pix, gate=gate)
    for V in (want[0], eager[0]):
        got = np.stack([V[:, u, v].numpy() for u, v in pix], axis=1)
        assert rel_l2(got, ref) <= FP32_BAR
    assert not torch.equal(want[0], eager[0])      # the two orders round differently
    st = Stream(plan, lam, 12e-6, 0.3, slots=1)

    def popped():
        r = st.pop(wait=True)
        return r["seq"], st.slot_volume(r["slot"]).cpu()

    assert st.push_frames(sweeps[0][:20], 0) == native.OK               # a chunk of it runs
    assert st.push_frames(sweeps[0][21:], 21) == native.EDROPPED
    for i in (1, 2):
        for a in range(0, T, 9):
            assert st.push_frames(np.ascontiguousarray(sweeps[i][a:a + 9]), i * T + a) == native.OK
        seq, V = popped()
        assert seq == i and torch.equal(V, want[i]), i
        slot, buf = st.acquire()
        buf.copy_(dev[0])
        torch.cuda.synchronize()
        st.submit(slot, 100 + i)
        seq, V = popped()
        assert seq == 100 + i and torch.equal(V, eager[0]), i
    assert st.stats()["dropped_sweeps"] == 1 and st.stats()["done"] == 4
    st.close(), plan.close(), frame_order.close()


@pytest.mark.parametrize("precision,order", [("bf16_split", 1), ("fp32_fft", 0), ("fp32_4step", 1)])
def test_ragged_chunks_and_a_discarded_sweep_in_the_frame_order(gpu_lib, precision, order):
    """Forms that render frame by frame, five frames per chunk (T = 32: six chunks and a ragged one): the
    chunk graphs of a sweep that is then discarded do not disturb the next one in the same slot, and every
    volume has the bits of the plan's render."""
    from paper_2003_08960_amd.api import Plan, Stream
    T, N = 32, 128
    sweeps = [random_case(T, N, seed=1450 + i)[0] for i in range(3)]
    lam = random_case(T, N, seed=1450)[1]
    print(f"\n[gpu] stream ragged chunks {precision}", flush=True)
    plan = Plan(T, N, precision=precision)
    plan.set_tuning([5, 0, 0, order])
    want = [plan.render(torch.from_numpy(f).cuda(), lam, 12e-6, 0.3).clone() for f in sweeps]
    st = Stream(plan, lam, 12e-6, 0.3, slots=1)
    assert st.push_frames(sweeps[0][:23], 0) == native.OK               # chunks 0 to 3 start
    assert st.push_frames(sweeps[0][24:], 24) == native.EDROPPED
    for i, cuts in ((1, (0, 7, 19, 32)), (2, tuple(range(0, 33, 3)) + (32,))):
        for a, b in zip(cuts[:-1], cuts[1:]):
            assert st.push_frames(np.ascontiguousarray(sweeps[i][a:b]), i * T + a) == native.OK
        r = st.pop(wait=True)
        assert r["seq"] == i and torch.equal(st.slot_volume(r["slot"]), want[i]), i
    assert st.stats()["dropped_sweeps"] == 1 and st.stats()["done"] == 2
    st.close(), plan.close()
