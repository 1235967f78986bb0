"""The rules that choose streaming or cached accesses, compiled for the host:
at sizes where both were timed with several inputs in turn and with one, no form
that was slower than streaming is chosen, and a pass without a gradient streams."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LOADS, STORES = 1, 2  # streaming
MB = 1 << 20


@pytest.fixture(scope="module")
def lib():
    so = os.path.join(HERE, "host", "libaccess_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-o", so + ".tmp",
                           os.path.join(HERE, "host", "access_host.cpp")])
    os.replace(so + ".tmp", so)
    L = ctypes.CDLL(so)
    L.host_inv_det_access.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    L.host_wishart_access.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4
    L.host_off_lines.argtypes = [ctypes.c_uint64, ctypes.c_int64, ctypes.c_int]
    return L


@pytest.mark.parametrize("es", [4, 8])
@pytest.mark.parametrize("mb,off_in,off_grad,mode", [
    (24, 0, 0, STORES), (80, 0, 0, STORES), (96, 0, 0, LOADS | STORES), (128, 0, 0, LOADS | STORES),
    (160, 0, 0, LOADS | STORES), (192, 0, 0, LOADS | STORES), (256, 0, 0, LOADS | STORES),
    (32, 0, 1, STORES), (64, 0, 1, STORES), (96, 0, 1, 0), (160, 0, 1, 0), (192, 0, 1, LOADS | STORES),
    (256, 0, 1, LOADS | STORES), (384, 0, 1, LOADS | STORES),
    (64, 1, 1, STORES), (96, 1, 1, 0), (160, 1, 1, 0), (224, 1, 1, STORES), (400, 1, 1, STORES), (1500, 1, 1, STORES)])
def test_wishart(lib, es, mb, off_in, off_grad, mode):
    n = mb * MB // (18 * es)
    assert lib.host_wishart_access(n, es, 1, off_in, off_grad) == mode
    assert lib.host_wishart_access(n, es, 0, off_in, 0) == LOADS | STORES


@pytest.mark.parametrize("es", [4, 8])
@pytest.mark.parametrize("mb,off,mode", [(16, 0, STORES), (40, 0, STORES), (56, 0, LOADS | STORES),
                                         (188, 0, LOADS | STORES), (16, 1, STORES), (188, 1, STORES),
                                         (224, 1, STORES), (412, 1, STORES), (768, 1, STORES)])
def test_inverse(lib, es, mb, off, mode):
    assert lib.host_inv_det_access(mb * MB // (9 * es), es, off) == mode


def test_inverse_of_large_images_streams(lib):
    assert lib.host_inv_det_access((1 << 25) - 1, 4, 1) == STORES
    assert lib.host_inv_det_access(1 << 25, 4, 1) == LOADS | STORES


@pytest.mark.parametrize("p,pitch,es,off", [(0, 32, 4, 0), (128, 16, 8, 0), (0, 33, 4, 1), (64, 32, 4, 1), (0, 40, 8, 1)])
def test_off_lines(lib, p, pitch, es, off):
    assert lib.host_off_lines(p, pitch, es) == off
