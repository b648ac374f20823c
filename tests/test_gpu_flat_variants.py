"""The flat iteration has two variants, picked by the number of waves in a launch
(few waves: everything loaded at the start; many: fewer registers).  They form
the same sums in the same order, so a scene keeps its bits whether it runs alone
or beside a scene large enough to change the variant."""
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


def _touching(n, prec):
    """n boxes close enough to touch, the lowest at the ground, spinning."""
    side = max(1, round(n ** (1 / 3)))
    sc = S.box_drop(side, layers=-(-n // side ** 2), seed=n, spacing=1.3, base_height=-0.7, precision=prec)
    k = np.arange(n)
    rng = np.random.Generator(np.random.PCG64(n))
    fields = ("shape", "shape_param", "density", "flags", "group", "c0", "A0", "v0")
    sc = sc.copy(**{f: getattr(sc, f)[k] for f in fields}, w0=rng.uniform(-1, 1, (n, 3)))
    sc.flags[n // 2] |= S.FLAG_PINNED
    return sc


@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_launch_size_does_not_change_a_scenes_bits(P, prec, lanes):
    # ends per body around and beyond a round of the latency variant, a pinned
    # body among them; joints beyond a tile; variable and driven joints
    scenes = [_touching(67, prec), _touching(200, prec), S.chain(67, tilt_deg=20.0, precision=prec),
              S.spring_net(5, order=4, precision=prec), S.linkage("slider", drive_amp_deg=60.0, precision=prec)]
    filler = S.chain(64 * 1024 + 1, tilt_deg=5.0, precision=prec)  # more waves than the latency variant takes
    got = []
    for beside in ([], [filler]):
        b = P.Batch(8, 1 << 30, prec)
        b.set_schedule(contact_lanes=lanes)
        slots = [b.admit(s, 6) for s in scenes]
        assert all(b.admit(s, 6) is not None for s in beside)
        for _ in range(8):  # two steps more than the scenes take: those change nothing
            b.step()
        got.append([b.state(k) + (np.array([b.residual(k)]),) for k in slots])
        b.close()
    for sc, x, y in zip(scenes, *got):
        for p, q in zip(x, y):
            assert np.array_equal(p, q), sc.name
