"""State read-back: every value of every body, whichever outputs are asked for,
after steps on the handle's own stream and on a caller's."""
import ctypes as C

import numpy as np
import pytest

from paper_2609_02675_amd import _lib, scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_02675_amd as P
    if P.device_count() < 1:
        pytest.fail("no HIP device visible")
    return P


def _spread(n, prec):
    """n free bodies, every component of every body's state a value of its own."""
    rng = np.random.Generator(np.random.PCG64(n))
    sc = S.chain(n, precision=prec, pin_top=False)
    return sc.copy(c0=rng.uniform(-9, 9, (n, 3)), A0=S.random_rotations(rng, n), v0=rng.uniform(-1, 1, (n, 3)),
                   w0=rng.uniform(-1, 1, (n, 3)))


@pytest.mark.parametrize("n", [1, 2, 43, 7300])  # one workgroup's values and beside it; beyond one MiB of them
@pytest.mark.parametrize("prec", [S.PREC_FP32, S.PREC_FP64], ids=["fp32", "fp64"])
def test_a_read_returns_what_was_uploaded(P, prec, n):
    sc = _spread(n, prec)
    b = P.Batch(2, 1 << 27, prec)
    b.admit(_spread(3, prec), 1)  # the scene read does not start the arrays
    slot = b.admit(sc, 1)
    # an FP32 position is the sum of two floats (48 bits at least), the rest one float
    c_tol, tol = (9 * 2.0 ** -48, 2.0 ** -24) if prec == S.PREC_FP32 else (0.0, 0.0)
    for st in (P.Scene(sc).state(), b.state(slot)):
        for x, y, t in zip(st, (sc.c0, sc.A0, sc.v0, sc.w0), (c_tol, tol, tol, tol)):
            assert np.abs(x - y).max() <= t
    g = P.Scene(sc)
    whole = g.state()
    for k in range(4):  # any output may be left out
        one = np.full(whole[k].shape, np.nan)
        ptr = [None] * 4
        ptr[k] = one.ctypes.data_as(C.c_void_p)
        assert _lib.lib().pabd_scene_read_state(g._h, *ptr) == _lib.PABD_OK
        assert np.array_equal(one, whole[k])


def test_a_read_waits_for_steps_on_a_callers_stream(P):
    import torch
    sc = S.chain(60, tilt_deg=30.0, precision=S.PREC_FP64)
    want = P.Scene(sc)
    want.step(400)
    ref = want.state()
    g, b = P.Scene(sc), P.Batch(2, 1 << 26, S.PREC_FP64)
    b.set_tile(32)  # 60 bodies: the flat path, many launches
    slot = b.admit(sc, 400)
    st = torch.cuda.Stream()
    for _ in range(4):
        g.step(50, stream=st.cuda_stream)
        b.step(nsteps=50, stream=st.cuda_stream)
    half = g.state(), b.state(slot)
    st.synchronize()
    for x, y in zip(half, (g.state(), b.state(slot))):
        assert all(np.array_equal(p, q) for p, q in zip(x, y))
    st.synchronize()
    g.step(200)
    for _ in range(4):
        b.step(nsteps=50)
    for got in (g.state(), b.state(slot)):
        assert all(np.array_equal(p, q) for p, q in zip(got, ref))


def test_threads_read_the_scenes_of_one_batch(P):
    """Reads of different scenes at the same time: each returns its own scene."""
    from concurrent.futures import ThreadPoolExecutor
    scs = [_spread(n, S.PREC_FP64) for n in (400, 900, 1300, 700)]
    b = P.Batch(len(scs), 1 << 27, S.PREC_FP64)
    slots = [b.admit(s, 1) for s in scs]

    def read(k):
        for _ in range(100):
            for x, y in zip(b.state(slots[k]), (scs[k].c0, scs[k].A0, scs[k].v0, scs[k].w0)):
                if not np.array_equal(x, y):
                    return False
        return True

    with ThreadPoolExecutor(len(scs)) as pool:
        assert all(pool.map(read, range(len(scs))))


@pytest.mark.parametrize("n", [8, 200, 1000])
def test_an_error_the_caller_left_behind_is_not_this_calls(P, n):
    """A caller's own failed HIP call does not fail the step or the read after it."""
    sc = S.chain(n, tilt_deg=20.0, precision=S.PREC_FP32)
    want, g = P.Scene(sc), P.Scene(sc)
    want.step(4)
    ref = want.state()
    hip = _lib.lib()  # its symbols include those of the HIP runtime it is linked to
    assert hip.hipSetDevice(9999) != 0
    g.step(4)
    assert hip.hipSetDevice(9999) != 0
    got = g.state()
    hip.hipGetLastError()
    for p, q in zip(got, ref):
        assert np.array_equal(p, q)
