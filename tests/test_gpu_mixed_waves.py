"""Many small scenes on a batch's flat path share wavefronts; few have wavefronts of
their own.  Either way a scene's bits are its own."""
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


def _kinds(prec):
    """Scenes of the flat path beside each other: variable and driven joints, quadratic
    chains beyond a tile (whose last wave holds one body and six), contacts between."""
    return [S.linkage("slider", drive_amp_deg=60.0, precision=prec), S.mass_ratio_chain(19, precision=prec),
            S.chain(65, tilt_deg=20.0, precision=prec), S.spring_net(5, order=4, precision=prec),
            S.linkage("four_bar", drive_amp_deg=40.0, precision=prec), S.pile(20, 4, precision=prec),
            S.chain(70, tilt_deg=30.0, precision=prec), S.slider_pair(precision=prec)]


@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_shared_waves_do_not_change_a_scenes_bits(P, prec):
    kinds = _kinds(prec)
    steps = [3 + k % 4 for k in range(len(kinds))]  # scenes end between others that go on

    def run(rounds):
        b = P.Batch(rounds * len(kinds) + 8, 1 << 28, prec)
        slots = [b.admit(kinds[k], steps[k]) for _ in range(rounds) for k in range(len(kinds))]
        assert None not in slots
        b.step()
        if rounds > 1:  # holes in the range of bodies, and other scenes in their place
            for k in (3, 10, 17, 30):
                b.release(slots[k])
            slots[10] = b.admit(kinds[10 % len(kinds)], steps[10 % len(kinds)])
        b.step(nsteps=4)
        b.step()
        b.step()
        last = len(slots) - len(kinds)
        got = [[b.state(slots[at + k]) + (np.array([b.residual(slots[at + k])]),) for k in range(len(kinds))]
               for at in sorted({0, last // 2 // len(kinds) * len(kinds), last}) if at != 0 or rounds == 1]
        back = b.state(slots[10]) if rounds > 1 else None
        b.close()
        return got, back

    (alone,), _ = run(1)
    many, back = run(40)  # 360 waves of scenes without contacts
    assert len(many) == 2
    for got in many:
        for sc, x, y in zip(kinds, alone, got):
            for p, q in zip(x, y):
                assert np.array_equal(p, q), sc.name
    for p, q in zip(alone[10 % len(kinds)], back):  # admitted a step later, done all the same
        assert np.array_equal(p, q)
