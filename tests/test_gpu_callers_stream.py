"""Work on a caller's stream: what the host changes or reads in between finds the
steps enqueued there done."""
import numpy as np
import pytest

from paper_2609_02675_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_02675_amd as P
    if P.device_count() < 1:
        pytest.fail("no HIP device visible")
    return P


@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_scenes_come_and_go_under_steps_on_a_callers_stream(P, prec):
    """Admissions and releases right behind steps that a caller's stream still runs
    (no read in between) change nothing of those steps."""
    import torch
    st = torch.cuda.Stream()

    def run(stream):
        b = P.Batch(8, 1 << 28, prec)
        keep = [b.admit(S.pile(300, 1, precision=prec), 40), b.admit(S.linkage("slider", drive_amp_deg=60.0, precision=prec), 40),
                b.admit(S.chain(30, tilt_deg=20.0, precision=prec), 40)]
        gone = b.admit(S.pile(40, 2, precision=prec), 40)
        for k in range(8):
            b.step(stream=stream, nsteps=4)
            if k == 1:  # the wave table shrinks, grows and moves to a larger allocation
                b.release(gone)
            if k in (2, 4):
                keep.append(b.admit(S.chain(200 * k, tilt_deg=20.0, precision=prec), 40))
            if k == 5:
                keep.append(b.admit(S.pile(900, 3, precision=prec), 40))
            if k == 6:
                b.set_schedule(contact_lanes=8)
        out = [b.state(s) + (np.array([b.residual(s)]),) for s in keep]
        b.close()
        return out

    for x, y in zip(run(None), run(st.cuda_stream)):
        for p, q in zip(x, y):
            assert np.array_equal(p, q)


def test_a_read_waits_for_replays_of_a_callers_graph(P):
    """Steps captured in a caller's graph: every read after a replay, the second and
    later ones too, finds that replay's steps done."""
    import torch
    sc = S.chain(200, tilt_deg=30.0, precision=S.PREC_FP64)
    want, g = P.Scene(sc), P.Scene(sc)
    st = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(st), torch.cuda.graph(graph, stream=st):
        g.step(100, stream=st.cuda_stream)
    for _ in range(5):
        with torch.cuda.stream(st):
            graph.replay()
        got = g.state()
        want.step(100)
        for p, q in zip(got, want.state()):
            assert np.array_equal(p, q)
        torch.zeros(1000, device="cuda").add_(1).sum().item()
