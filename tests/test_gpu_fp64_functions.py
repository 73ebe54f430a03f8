"""Each elementary function of the FP64 walks against its exact value (80-bit
arithmetic) over the arguments that a walk gives it, random ones and the ends of
the ranges. The bounds are those of a replay of the functions in C with exact
fused operations over 2e7 arguments (0.81, 0.50, 1.82, 0.89 and 0.87), rounded
up: the hardware's reciprocal and root seeds are corrected to far below them."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import build as B  # noqa: E402

LN, SQRT, TURN, SINCOS, EXP = range(5)
N = 1 << 20


def on_gpu(function, x):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert os.path.exists(B.PROBE_LIB)
    lib = ctypes.CDLL(B.PROBE_LIB)
    t = torch.as_tensor(x.view(np.int32) if x.dtype == np.uint32 else x).cuda()
    out = torch.empty((2, len(x)), dtype=torch.float64, device="cuda")
    assert lib.probe_fp64_math(ctypes.c_int(function), ctypes.c_void_p(t.data_ptr()), ctypes.c_longlong(len(x)),
                               ctypes.c_void_p(out[0].data_ptr()), ctypes.c_void_p(out[1].data_ptr())) == 0
    return out.cpu().numpy()


def long(x):
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no 80-bit arithmetic")
    return x.astype(np.longdouble)


def ulps(got, want):
    return float(np.max(np.abs(got - want) / np.spacing(np.abs(want).astype(np.float64))))


def words():
    edges = [np.arange(2000), 2 ** 32 - 1 - np.arange(2000)]
    edges += [k * 2 ** 29 + np.arange(-500, 500) for k in range(1, 8)]
    return np.concatenate([np.random.default_rng(1).integers(0, 2 ** 32, N)] + edges).astype(np.uint32)


def test_logarithm():
    w = words()
    want = -2 * np.log((long(w) + np.longdouble(0.5)) * np.longdouble(2.0) ** -32)
    assert ulps(on_gpu(LN, w)[0], want) <= 1.0


def test_square_root():
    rng = np.random.default_rng(2)
    x = np.concatenate([2.0 ** rng.uniform(-32, 6, N), 2.0 ** -32 * (1 + np.arange(100)), 4.0 ** np.arange(-16.0, 3.0)])
    assert ulps(on_gpu(SQRT, x)[0], np.sqrt(long(x))) <= 0.52


def test_turn():
    w = words()
    q = ((w.astype(np.int64) + 2 ** 29) >> 30)
    r = long(w.astype(np.int64) - (q << 30)) + np.longdouble(0.5)
    a = r * (2 * np.longdouble("3.14159265358979323846264338327950288") * np.longdouble(2.0) ** -32)
    s, c = np.sin(a), np.cos(a)
    want = [np.choose(q & 3, v) for v in ([s, c, -s, -c], [c, -s, -c, s])]
    got = on_gpu(TURN, w)
    assert max(ulps(g, v) for g, v in zip(got, want)) <= 2.0


@pytest.mark.parametrize("most", [np.pi / 4, 100.0, 2 * np.pi * 2.0 ** 25])
def test_sine_and_cosine(most):
    rng = np.random.default_rng(3)
    x = np.concatenate([rng.uniform(-most, most, N), [0.0, most, -most, 1e-300, -1e-20],
                        np.rint(rng.uniform(-most, most, 10000) / (np.pi / 2)) * (np.pi / 2)])
    x = x[np.abs(x) <= most]
    got, want = on_gpu(SINCOS, x), [np.sin(long(x)), np.cos(long(x))]
    assert max(float(np.max(np.abs(g - v))) for g, v in zip(got, want)) <= 2.0 ** -53
    if most < 1.0:
        nz = x != 0.0
        assert max(ulps(g[nz], v[nz]) for g, v in zip(got, want)) <= 1.0
        assert got[0][~nz].tolist() == [0.0] * int(np.sum(~nz))


def test_exponential():
    x = np.concatenate([np.random.default_rng(4).uniform(0, 40, N), [0.0, 1e-300, 1e-17, 24.953298500158186, 300.0]])
    assert ulps(on_gpu(EXP, x)[0], np.exp(-long(x))) <= 1.0
