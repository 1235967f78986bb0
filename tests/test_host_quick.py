"""The quick form of the FP32 compensated inverse, compiled for the host:
what it claims about a pixel holds, and its result is within the bound it is
accepted by, on matrices over the ranges where its limits lie (condition
numbers up to 1e10, scales from 1e-38 to 1e38, graded diagonals, indefinite,
small integers, non-finite)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_1807_08084_amd import synth

HERE = os.path.dirname(os.path.abspath(__file__))
NONE, VALUE, ALL = 0, 1, 2


@pytest.fixture(scope="module")
def lib():
    so = os.path.join(HERE, "host", "libquick_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fopenmp", "-ffp-contract=off", "-o",
                           so + ".tmp", os.path.join(HERE, "host", "quick_host.cpp")])
    os.replace(so + ".tmp", so)
    L = ctypes.CDLL(so)
    L.host_quick.restype = ctypes.c_int64
    return L


def _run(lib, z):
    n = z.shape[1]
    inv, det = np.empty((9, n), np.float32), np.empty(n, np.float32)
    quick, ok, st = (np.empty(n, np.uint8) for _ in range(3))
    bad = lib.host_quick(ctypes.c_int64(n), *(a.ctypes.data_as(ctypes.c_void_p) for a in (z, inv, det, quick, ok, st)),
                         ctypes.c_int(max(1, min(8, len(os.sched_getaffinity(0))))))
    return inv, det, quick, ok, st, bad


def _matrices(name):
    rng = np.random.default_rng(17)
    m = 60000
    U = synth.haar_unitary(rng, m)

    def spectrum(eig):
        return synth.pack(np.einsum("mij,mj,mkj->mik", U, eig, np.conj(U)))

    if name == "hard":
        return spectrum(np.stack([np.ones(m), 10.0 ** -rng.uniform(0, 9, m), 10.0 ** -rng.uniform(0, 10, m)], 1))
    if name == "scaled":
        eig = np.stack([np.ones(m), 10.0 ** -rng.uniform(0, 4, m), 10.0 ** -rng.uniform(0, 8, m)], 1)
        return spectrum(eig * (10.0 ** rng.uniform(-38, 38, m))[:, None])
    if name == "range":  # around tr = 2^40 and det = 2^-88 (1 + tr)
        eig = np.stack([np.ones(m), 10.0 ** -rng.uniform(0, 3, m), 10.0 ** -rng.uniform(0, 4, m)], 1)
        return spectrum(eig * np.where(rng.random(m) < 0.5, 2.0 ** rng.uniform(36, 42, m),
                                       2.0 ** rng.uniform(-32, -24, m))[:, None])
    if name == "graded":
        d = 10.0 ** rng.uniform(-8, 8, (m, 3))
        eig = np.stack([np.ones(m), 10.0 ** -rng.uniform(0, 3, m), 10.0 ** -rng.uniform(0, 7, m)], 1)
        z = np.einsum("mij,mj,mkj->mik", U, eig, np.conj(U)) * d[:, :, None] * d[:, None, :]
        return synth.pack(z)
    if name == "indefinite":
        eig = np.stack([np.ones(m), 10.0 ** -rng.uniform(0, 8, m), 10.0 ** -rng.uniform(0, 9, m)], 1)
        return spectrum(eig * np.where(rng.random((m, 3)) < 0.3, -1, 1))
    if name == "integers":
        return rng.integers(-4, 5, (9, m)).astype(float)
    z = rng.standard_normal((9, m))
    z[:3] = np.abs(z[:3]) * 10
    z[rng.random((9, m)) < 0.05] = np.nan
    z[rng.random((9, m)) < 0.05] = np.inf
    z[rng.random((9, m)) < 0.1] = 0
    return z


@pytest.mark.parametrize("name", ["hard", "scaled", "range", "graded", "indefinite", "integers", "nonfinite"])
def test_quick_form(lib, name):
    with np.errstate(over="ignore", under="ignore"):
        z = np.ascontiguousarray(_matrices(name).astype(np.float32))
    inv, det, quick, ok, st, bad = _run(lib, z)
    assert bad == 0
    # QUICK_ALL: the FP32 evaluation carries the pixel; QUICK_VALUE: it is
    # positive definite, so that its status is OK or REROUTED
    assert np.all(ok[quick == ALL] == 1)
    assert np.all(st[quick != NONE] == 1)
    w = z.astype(np.float64)
    finite = np.isfinite(w).all(axis=0)
    assert np.all(quick[~finite] == NONE)
    if name in ("hard", "graded", "range"):
        assert (quick == ALL).mean() > 0.2 and (quick == NONE).any()
    sel = quick != NONE
    if not sel.any():
        return
    assert np.all(oracle.pd_class(w[:, sel]) == 0)
    (ih, il), (dh, dl) = oracle.ge128(w[:, sel])
    # 9e-8 of the form's bound, one FP32 rounding of the result
    tol = 9e-8 + 2.0 ** -24
    assert np.all(oracle.det_rel_err(det[sel], dh, dl) <= tol)
    normal = (np.abs(ih) > 1e-30).all(axis=0) if name == "graded" else np.ones(sel.sum(), bool)
    assert np.all(oracle.inv_rel_err(inv[:, sel], ih, il)[normal] <= tol)


# Where FP32 alone carries a well-conditioned matrix, the quick form does too
# and settles its status, but within a factor of two of the ends of FP32's range.
@pytest.mark.parametrize("scale", [3e-10, 5e-10, 1e-9, 1.5e-9, 3e-9, 1e-8, 1e-4, 1.0, 1e6, 1e11, 1e12])
def test_quick_form_carries_well_conditioned_scales(lib, scale):
    rng = np.random.default_rng(23)
    s = (rng.standard_normal((20000, 3, 8)) + 1j * rng.standard_normal((20000, 3, 8))) * np.sqrt(0.5)
    z = synth.pack(np.einsum("mik,mjk->mij", s, np.conj(s)) / 8 * scale)
    z = np.ascontiguousarray(z.astype(np.float32))
    inv, det, quick, ok, st, bad = _run(lib, z)
    assert bad == 0 and ok.mean() >= 0.99
    assert (quick[ok == 1] == ALL).mean() >= 0.99
    assert np.all(ok[quick == ALL] == 1) and np.all(st[quick != NONE] == 1)
    sel = quick != NONE
    (ih, il), (dh, dl) = oracle.ge128(z[:, sel].astype(np.float64))
    tol = 9e-8 + 2.0 ** -24
    assert np.all(oracle.det_rel_err(det[sel], dh, dl) <= tol)
    assert np.all(oracle.inv_rel_err(inv[:, sel], ih, il) <= tol)


# The ends themselves: determinants and traces across both limits, ALL only
# where the FP32 evaluation carries the pixel.
@pytest.mark.parametrize("lo,hi", [(-36, -28), (38, 46)])
def test_quick_form_at_the_ends_of_its_range(lib, lo, hi):
    rng = np.random.default_rng(31)
    m = 200000
    U = synth.haar_unitary(rng, m)
    eig = np.stack([np.ones(m), 10.0 ** -rng.uniform(0, 3, m), 10.0 ** -rng.uniform(0, 4, m)], 1)
    with np.errstate(over="ignore", under="ignore"):
        z = synth.pack(np.einsum("mij,mj,mkj->mik", U, eig, np.conj(U))) * 2.0 ** rng.uniform(lo, hi, m)
        z = np.ascontiguousarray(z.astype(np.float32))
    inv, det, quick, ok, st, bad = _run(lib, z)
    assert bad == 0
    assert (quick == ALL).any() and (quick == NONE).any() and (ok == 0).any()
    assert np.all(ok[quick == ALL] == 1) and np.all(st[quick != NONE] == 1)
