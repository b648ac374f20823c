"""The variants of the body iteration form the same sums in the same order, so a
scene's bits do not depend on which of them runs it: the flat kernels' two
variants, picked by the number of waves in a launch (few waves: everything loaded
at the start; many: fewer registers), the resident kernels' workgroup sizes and
their lanes per body, picked by the scene's size, and the tile kernels' lanes per
body, picked by the number of tiles."""
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


def _moving(sc, seed):
    """The scene with every body turned, moving and spinning in all directions."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n = sc.n_bodies
    R = S.rot_axis(rng.normal(size=3), 1.0)
    return sc.copy(c0=sc.c0 @ R.T, A0=R @ sc.A0, v0=rng.uniform(-0.5, 0.5, (n, 3)), w0=rng.uniform(-2, 2, (n, 3)))


def _joint_scenes(prec):
    star = S.spring_net(3, order=4, precision=prec)  # one hub with more ends than LDS holds
    extra = {k: np.concatenate([getattr(star, k), np.repeat(getattr(star, k)[:1], 12, axis=0)])
             for k in ("bond_type", "x_i", "x_j", "kappa", "rest_len", "drive", "order")}
    star = star.copy(bond_i=np.concatenate([star.bond_i, np.zeros(12, np.int32)]),
                     bond_j=np.concatenate([star.bond_j, 1 + np.arange(12, dtype=np.int32) % 8]), **extra)
    quad = star.copy(bond_type=np.zeros(star.n_bonds, np.int32))
    hung = S.chain(9, tilt_deg=40.0, precision=prec, pin_top=False)  # from a world point, by a second end or a third
    hung = hung.copy(bond_i=np.r_[hung.bond_i, 0, 4].astype(np.int32), bond_j=np.r_[hung.bond_j, -1, -1].astype(np.int32),
                     bond_type=np.zeros(10, np.int32), x_i=np.r_[hung.x_i, [[0, 0.5, 0], [0.5, 0, 0]]],
                     x_j=np.r_[hung.x_j, [[0, 0.5, 0], [3.0, -1, 1]]], kappa=np.full(10, 1e5), rest_len=np.r_[np.zeros(9), 0.2],
                     drive=np.zeros((10, 13)), order=np.full(10, 2, np.int32))
    return star, quad, hung


@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_resident_workgroup_size_does_not_change_a_scenes_bits(P, prec):
    """A plain scene (resident kernels, several steps per launch) against the same
    scene with the recording of every residual on, which the flat kernels do, a
    step at a time: sizes at and beside each workgroup's edge, bonds within and
    beyond what it holds, with and without rest lengths, to the world and to
    pinned bodies, and contact piles at theirs."""
    chains = [S.chain(n, tilt_deg=20.0, precision=prec)
              for n in (1, 2, 16, 17, 64, 65, 128, 129, 255, 256, 257, 512, 513, 1024)]
    nets = [S.spring_net(n, order=p, precision=prec)
            for n, p in ((2, 12), (4, 2), (8, 2), (8, 4), (11, 2), (12, 2), (16, 6), (17, 2), (23, 4))]
    star, quad, hung = _joint_scenes(prec)
    other = [S.mass_ratio_chain(precision=prec), S.slider_pair(precision=prec), S.slider_rod(precision=prec),
             S.linkage("slider", drive_amp_deg=60.0, precision=prec), S.general_inertia_chain(precision=prec),
             S.polar_fallback_body("flip", precision=prec), S.world_pendulum(theta0_deg=50.0, precision=prec), star, quad,
             hung]
    scenes = [_moving(s, k) for k, s in enumerate(chains + nets)] + other + [_touching(n, prec) for n in (2, 16, 17, 64)]
    for sc in scenes:
        if sc.n_bodies > (1024 if prec == S.PREC_FP32 else 512):
            continue
        g, f = P.Scene(sc), P.Scene(sc)
        g.step(3)
        g.step(4)
        f.set_debug(2)
        f.step(7)
        for p, q in zip(g.state(), f.state()):
            assert np.array_equal(p, q), sc.name
        assert g.residual() == pytest.approx(f.residual(), rel=1e-12), sc.name
        assert g.polar_fallbacks() == f.polar_fallbacks(), sc.name


@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("tile", [32, 64, 128])
def test_number_of_tiles_does_not_change_a_scenes_bits(P, prec, tile):
    """Scenes in a few tiles (a quad of lanes per body) and beside enough others
    to change the kernel (one lane per body): one body, full tiles, bonds to the
    world, with rest lengths, beyond the two in registers, a body turned inside
    out, scenes that finish inside a launch."""
    _, quad, hung = _joint_scenes(prec)
    scenes = [S.chain(n, tilt_deg=20.0, precision=prec) for n in (1, 2, 31, 32)] + [quad, hung]
    scenes += [S.spring_net(5, precision=prec), S.general_inertia_chain(precision=prec)]
    scenes = [_moving(s, k) for k, s in enumerate(scenes)]
    scenes += [S.world_pendulum(theta0_deg=50.0, precision=prec), S.polar_fallback_body("flip", precision=prec)]
    scenes += [_moving(S.chain(n, tilt_deg=20.0, precision=prec), n) for n in (64, 128) if n <= tile]
    filler = S.chain(tile - 3, tilt_deg=5.0, precision=prec)
    got = []
    for extra in (0, 800):
        b = P.Batch(len(scenes) + extra, (64 << 20) + extra * 2 * P.scene_bytes(filler), prec)
        b.set_tile(tile)
        slots = [b.admit(s, 7 + k % 3) for k, s in enumerate(scenes)]
        for _ in range(extra):
            assert b.admit(filler, 9) is not None
        b.step(nsteps=5)
        b.step(nsteps=6)
        got.append([b.state(k) + (b.residual(k), b.polar_fallbacks(k)) for k in slots])
        b.close()
    for sc, x, y in zip(scenes, *got):
        for p, q in zip(x[:4], y[:4]):
            assert np.array_equal(p, q), sc.name
        assert x[4:] == y[4:], sc.name


@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_two_phase_kernels_match_the_flat_ones(P, prec):
    """The resident kernels that form the ends first and add them afterwards, against
    the flat kernels as above: ends beyond what registers hold and beyond what LDS
    holds, many driven and sliding joints around the change from four lanes per
    body to one, and a driven point on a free body, whose block is factored again."""
    driven = S.linkage("slider", drive_amp_deg=60.0, precision=prec)
    free = driven.copy(bond_j=np.where(driven.bond_type == S.BOND_DRIVEN, 2, driven.bond_j).astype(np.int32))
    many = [S.merge([driven, free] * k) for k in (1, 8, 9, 33)]
    nets = [S.spring_net(n, order=4, precision=prec) for n in (9, 19, 22)]
    for sc in many + nets:
        g, f = P.Scene(sc), P.Scene(sc)
        g.step(3)
        g.step(4)
        f.set_debug(2)
        f.step(7)
        for p, q in zip(g.state(), f.state()):
            assert np.isfinite(p).all() and np.array_equal(p, q), (sc.name, sc.n_bodies)
        assert g.residual() == pytest.approx(f.residual(), rel=1e-12), sc.name
