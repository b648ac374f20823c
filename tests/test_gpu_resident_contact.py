"""Contact scenes beside the sizes at which one workgroup takes their steps, and at
which its size changes: the same bits as the flat kernels, which run a scene while
every iteration's residual is recorded."""
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


def _heap(n, prec):
    """n boxes and spheres that touch, the lowest in the ground, one of them pinned:
    more contacts per body than a lane's registers hold."""
    rng = np.random.Generator(np.random.PCG64(n))
    side = max(1, round(n ** (1 / 3)))
    sc = S.box_drop(side, layers=-(-n // side ** 2), seed=n, spacing=1.25, base_height=-0.7, precision=prec)
    k = np.arange(n)
    fields = ("shape", "shape_param", "density", "flags", "group", "c0", "A0", "v0")
    sc = sc.copy(**{f: getattr(sc, f)[k] for f in fields}, w0=rng.uniform(-1, 1, (n, 3)))
    sc.shape[k % 4 == 1] = S.SHAPE_SPHERE
    sc.shape_param[k % 4 == 1] = [0.5, 0.0, 0.0]
    sc.flags[n // 2] |= S.FLAG_PINNED
    return sc


def _chain_on_the_ground(n, prec, augmented):
    sc = (S.mass_ratio_chain(n, tilt_deg=90.0, ratio=2.0, precision=prec) if augmented
          else S.chain(n, tilt_deg=90.0, precision=prec))
    return sc.copy(flags=np.zeros(n, np.uint8), group=np.ones(n, np.int32), c0=sc.c0 + [0.0, 0.52, 0.0],
                   density=np.full(n, 1000.0), contact_enable=1, planes=np.array([[0.0, 1.0, 0.0, 0.0]]),
                   v0=np.random.Generator(np.random.PCG64(n)).uniform(-0.3, 0.3, (n, 3)))


def _robots(k, prec):
    """k robots of 13 bodies with driven joints, a sphere each, on the ground."""
    one = S.granular_bed_quadruped(nx=1, nz=1, ny=1, precision=prec)
    many = [one.copy(c0=one.c0 + [2.0 * i, -0.02, 0.0]) for i in range(k)]
    return S.merge(many).copy(planes=np.array([[0.0, 1.0, 0.0, 0.0]]))


@pytest.mark.parametrize("n", [16, 17, 63, 64, 65, 127, 128, 129, 191, 192, 193])
@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_workgroup_and_flat_kernels_give_the_same_bits(P, prec, n):
    scenes = [_heap(n, prec), _chain_on_the_ground(n, prec, False), _chain_on_the_ground(n, prec, True)]
    if n in (64, 128):
        scenes.append(_robots(n // 14, prec))
    for sc in scenes:
        print(f"[case] {sc.name} n={sc.n_bodies} prec={prec}", flush=True)
        g, f = P.Scene(sc), P.Scene(sc)
        g.step(4)
        f.set_debug(2)
        f.step(4)
        assert g.contacts()["i"].size > 0
        for p, q in zip(g.state(), f.state()):
            assert np.isfinite(p).all() and np.array_equal(p, q), sc.name
        assert g.residual() == pytest.approx(f.residual(), rel=1e-12), sc.name
        assert g.polar_fallbacks() == f.polar_fallbacks(), sc.name
