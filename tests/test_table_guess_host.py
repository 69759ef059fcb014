"""The sampled noise curve's guessed interval against bisection, on the host
build of the kernels' code: the same interval and arithmetic, so the values
are equal bit for bit, on every spacing of the samples (even in ln f, in f, in
neither, nearly even, rounded as in a file), every size from two samples, and
at the samples themselves, their neighbouring doubles and the range's ends."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "model_host")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("table") / "libtable_host.so")
    subprocess.check_call(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                           os.path.join(HERE, "table_host.hip"), "-o", lib], stderr=subprocess.DEVNULL)
    return ctypes.CDLL(lib)


def _psd(host, tf, tS, kind, f, guess):
    P = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    out = np.zeros(len(f))
    found = host.table_psd_host(ctypes.c_int64(len(tf)), P(tf), P(tS), ctypes.c_int(kind), ctypes.c_double(2.7e-5),
                                ctypes.c_int64(len(f)), P(f), ctypes.c_int(guess), P(out))
    return out, found


def _curves(rng):
    for n in (2, 3, 4, 5, 6, 64, 2001):
        yield "log", np.geomspace(1.0, 4000.0, n)
        yield "lin", np.linspace(5.0, 2048.0, n)
    g = np.geomspace(2.0, 3000.0, 900)
    yield "rounded", np.unique(np.round(g, 3))
    jitter = g.copy()
    jitter[1:-1] *= np.exp(rng.uniform(-0.4, 0.4, len(g) - 2) * np.log(g[1] / g[0]))
    yield "jittered", jitter
    yield "two halves", np.concatenate([np.geomspace(1.0, 30.0, 200), np.linspace(31.0, 4000.0, 800)])
    yield "random", np.sort(rng.uniform(1.0, 4000.0, 700))
    shifted = g.copy()                   # even in ln f at the three samples looked at, not between
    shifted[300:400] = g[300] * (g[400] / g[300]) ** (np.linspace(0.0, 1.0, 100, endpoint=False) ** 3)
    yield "bent", shifted


@pytest.mark.parametrize("kind", [1, 2])
def test_guess_equals_bisection(host, kind):
    rng = np.random.default_rng(3)
    kinds = set()
    for name, tf in _curves(rng):
        tf = np.ascontiguousarray(tf)
        tS = rng.uniform(0.5, 2.0, len(tf))
        f = np.concatenate([tf, np.nextafter(tf, 0.0), np.nextafter(tf, 1e9), rng.uniform(0.5 * tf[0], 1.2 * tf[-1], 3000),
                            np.exp(rng.uniform(np.log(tf[0]), np.log(tf[-1]), 3000))])
        a, found = _psd(host, tf, tS, kind, f, 1)
        b, _ = _psd(host, tf, tS, kind, f, 0)
        kinds.add(found)
        assert np.array_equal(a, b, equal_nan=True), (name, len(tf))
        inside = (f >= tf[0]) & (f <= tf[-1])
        np.testing.assert_allclose(a[inside], np.interp(f[inside], tf, tS if kind == 1 else tS ** 2), rtol=1e-12)
        if len(tf) >= 4:
            assert {"log": found == 1, "lin": found == 2}.get(name, True), (name, len(tf), found)
    assert kinds == {0, 1, 2}
