"""The nonlocal-means kernel's choice of output rows per lane and waves per tile,
compiled for the host, at measured sizes: in FP64 no shape is chosen that ran
slower than four-wave blocks of one row a wave (but 6% at windows of radius 1
and 2) or much slower than the best; FP32 goes by tile counts alone."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SHAPES = (11, 21, 14, 24, 28)  # rows * 10 + waves

# distance, height, width, radius; us of each shape; of the four-wave blocks
MEASURED = [
    ("bhattacharyya", 550, 173, 1, [13.9, 15.3, 15.9, 17.2, 31.2], 14.8),
    ("bhattacharyya", 674, 231, 1, [18.6, 22.3, 22.7, 24.3, 46.9], 17.5),
    ("bhattacharyya", 173, 585, 5, [93.2, 97.6, 79.0, 86.2, 121.1], 106.3),
    ("bhattacharyya", 256, 256, 5, [57.8, 97.3, 47.6, 50.2, 66.8], 67.0),
    ("bhattacharyya", 128, 128, 11, [212.4, 377.8, 63.7, 106.7, 91.8], 256.4),
    ("bhattacharyya", 768, 768, 2, [97.7, 103.0, 117.5, 117.6, 183.9], 94.4),
    ("bhattacharyya", 768, 768, 8, [822.1, 861.8, 816.7, 793.4, 1087.8], 824.6),
    ("bhattacharyya", 1024, 1024, 5, [643.2, 627.8, 675.6, 625.3, 984.0], 626.4),
    ("bhattacharyya", 1500, 1500, 3, [629.2, 599.0, 700.9, 648.0, 859.6], 608.3),
    ("bhattacharyya", 2000, 40, 5, [88.2, 94.9, 83.8, 87.2, 127.0], 96.6),
    ("kl", 550, 173, 1, [12.4, 12.8, 17.7, 15.5, 28.4], 15.9),
    ("kl", 680, 189, 2, [20.4, 22.6, 31.9, 24.1, 34.4], 20.8),
    ("kl", 128, 128, 5, [36.3, 55.5, 15.2, 19.7, 20.6], 50.2),
    ("kl", 173, 585, 5, [54.5, 59.0, 54.5, 46.8, 69.0], 65.5),
    ("kl", 768, 768, 2, [73.7, 75.1, 128.4, 92.3, 145.2], 82.3),
    ("kl", 799, 122, 3, [28.7, 31.3, 33.2, 29.0, 39.4], 31.0),
    ("kl", 256, 256, 11, [133.1, 203.5, 103.3, 86.8, 93.0], 185.5),
    ("kl", 1024, 1024, 5, [358.0, 329.0, 467.1, 340.5, 554.7], 450.3),
    ("kl", 2000, 40, 5, [50.5, 56.4, 57.3, 47.5, 73.2], 60.8),
    ("kl", 132, 100, 16, [247.7, 393.1, 102.7, 117.7, 95.4], 360.2),
]


@pytest.fixture(scope="module")
def lib():
    so = os.path.join(HERE, "host", "libnlm_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-o", so + ".tmp",
                           os.path.join(HERE, "host", "nlm_host.cpp")])
    os.replace(so + ".tmp", so)
    L = ctypes.CDLL(so)
    L.host_nlm_shape.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return L


@pytest.mark.parametrize("distance,height,width,radius,us,blocks", MEASURED)
def test_f64_shape(lib, distance, height, width, radius, us, blocks):
    t = dict(zip(SHAPES, us))[lib.host_nlm_shape(1, distance == "kl", height, width, radius)]
    assert t <= (1.07 if radius <= 2 else 1.01) * blocks
    assert t <= 1.2 * min(us)


@pytest.mark.parametrize("kl,height,width,shape", [(1, 1, 1, 28), (1, 2045, 60, 28), (1, 2047, 63, 24), (0, 3686, 319, 24),
                                                   (0, 18431, 5, 21), (1, 18431, 5, 31), (1, 1 << 18, 1 << 20, 31)])
def test_f32_shape(lib, kl, height, width, shape):
    for radius in (0, 1, 16):
        assert lib.host_nlm_shape(0, kl, height, width, radius) == shape


@pytest.mark.parametrize("kl", [0, 1])
@pytest.mark.parametrize("height,width", [(1, 1), (1, 1 << 20), (4 * 65535, 1), (4 * 65535, 1 << 20)])
@pytest.mark.parametrize("radius", [0, 1, 16])
def test_f64_shape_exists(lib, kl, height, width, radius):
    assert lib.host_nlm_shape(1, kl, height, width, radius) in SHAPES
