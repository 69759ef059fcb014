"""The strain kernels' parts of a grid, on the host build of their code: every
point in exactly one part, whole runs of 256 points from a line of eight columns
on, lengths that differ by no more than a run, no part for nothing, up to the
longest grid an int32 holds."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "model_host")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("wave") / "libwave_host.so")
    subprocess.check_call(["/opt/rocm/bin/hipcc", "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                           os.path.join(HERE, "wave_part_host.hip"), "-o", lib], stderr=subprocess.DEVNULL)
    return ctypes.CDLL(lib)


def _parts(host, n, sh, parts, share, longest):
    k = np.zeros((parts, 2), dtype=np.int32)
    assert host.wave_parts_host(n, sh, parts, share, longest, k.ctypes.data_as(ctypes.c_void_p)) == 0
    return k.astype(np.int64)


def test_parts_cover_the_grid(host):
    rng = np.random.default_rng(5)
    big = 2 ** 31 - 1
    ns = [1, 2, 7, 8, 249, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 4096, 4097, 20000, big, big - 1, big - 255,
          big - 256, big - 300, *np.exp(rng.uniform(0, np.log(big), 60)).astype(int)]
    for n in ns:
        for sh in range(8):
            for parts, share, longest in ((1, 1, 4), (2, 1, 16), (3, 1, 16), (7, 1, 16), (9, 1, 4), (16, 1, 4), (2, 2, 16),
                                          (10, 10, 16), (41, 10, 16), (32, 32, 4), (64, 64, 4), (64, 64, 16)):
                k = _parts(host, int(n), sh, parts, share, longest)
                has = k[:, 1] > k[:, 0]
                m = int(has.sum())
                runs = (n + sh + 255) // 256
                assert has[:m].all()                              # the first parts, no gaps
                assert m == min(parts, max(min(runs, share), -(-runs // longest), 1))
                assert k[0, 0] == -sh and k[m - 1, 1] == n
                assert np.array_equal(k[1:m, 0], k[:m - 1, 1])
                assert np.all((k[1:m, 0] + sh) % 256 == 0)
                length = -(-(k[:m, 1] - k[:m, 0]) // 256)
                assert length.max() - length.min() <= 1


def test_lengths_that_are_none(host):
    for n in (0, -1, -5000, -2 ** 31):
        k = _parts(host, n, 3, 4, 2, 16)
        assert np.all(k[:, 1] <= 0)
