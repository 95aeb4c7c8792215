"""The library's host side on a CPU stand-in for the HIP runtime (fake_hip.cpp):
what stays allocated between contexts, and which device is waited for."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_02833_amd", "csrc")
GB = 1 << 30
N, EDGE = 3, 128                      # 16 moments of 128^3 cells
CELLS = EDGE ** 3
STATE = 16 * (CELLS + 64) * 8         # planes padded off the power of two


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libpm_host.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "flux.cpp"),
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.fake_live.restype = L.pm_device_bytes.restype = ctypes.c_longlong
    L.fake_reset.argtypes = [ctypes.c_longlong]
    L.fake_others.argtypes = [ctypes.c_int, ctypes.c_longlong]
    L.pm_init.argtypes = [ctypes.c_int] * 4 + [ctypes.c_double] * 2 + [ctypes.POINTER(ctypes.c_double)] * 3
    yield L
    L.pm_finalize()


FIELD = np.full(CELLS, 0.5)


def _init(L, edge=EDGE):
    p = FIELD.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    assert L.pm_init(N, edge, edge, edge, 1.0 / edge, 0.5 / edge, p, p, None) == 0


@pytest.mark.parametrize("free", [12 * GB, 40 * GB, 288 * GB])
def test_kept_memory_is_a_share_of_the_free_memory(host, free):
    """A dropped recording of 20 states stays for the next one, but at most an
    eighth of what the card has free and 1/32 of the card."""
    host.fake_reset(288 * GB)
    host.fake_others(0, 288 * GB - free)
    try:
        _init(host)
        context = host.fake_live(0)
        assert host.pm_set_checkpoint(1) == 0 and host.pm_step(20) == 0
        assert host.fake_live(0) >= context + 20 * STATE
        assert host.pm_set_checkpoint(0) == 0
        kept = host.fake_live(0) - host.pm_device_bytes()
        share = min((free - host.pm_device_bytes()) // 8, 9 * GB)
        assert kept <= share
        assert kept > min(20 * STATE, share) - 2 * STATE
    finally:
        host.pm_finalize()
    assert host.fake_live(0) == 0


@pytest.mark.parametrize("replace", [False, True])
def test_work_on_freed_blocks_is_waited_for_on_their_device(host, replace):
    """A recording or a context given up while another device is current: its
    blocks may be handed out again, so the work on them is waited for where it
    runs, and the caller's device stays current."""
    host.fake_reset(288 * GB)
    try:
        _init(host)
        assert host.pm_set_checkpoint(1) == 0 and host.pm_step(3) == 0
        assert host.fake_busy(0)
        host.hipSetDevice(1)
        if replace:
            _init(host, edge=16)
            assert host.fake_live(1) > 0
        else:
            assert host.pm_set_checkpoint(0) == 0
        assert not host.fake_busy(0)
        dev = ctypes.c_int(-1)
        host.hipGetDevice(ctypes.byref(dev))
        assert dev.value == 1
    finally:
        host.pm_finalize()
    assert host.fake_live(0) == host.fake_live(1) == 0


@pytest.mark.parametrize("prec,tables", [(0, 27 * 8), (1, 27 * 12)])
def test_a_context_holds_no_medium_after_its_tables(host, prec, tables):
    """State, tables and one float64 plane, and less than 1 MB beside them: the
    copies of sigma_a and sigma_s are needed for the tables only."""
    host.fake_reset(288 * GB)
    assert host.pm_set_precision(prec) == 0
    try:
        _init(host)
        assert host.pm_device_bytes() < STATE // (1 + prec) + CELLS * (tables + 8) + (1 << 20)
    finally:
        host.pm_set_precision(0)
        host.pm_finalize()


def test_the_latest_blocks_stay(host):
    """A program that differentiates over and over takes the same pool again,
    also when older blocks of other sizes had filled the library's share."""
    host.fake_reset(288 * GB)
    grad = np.zeros(CELLS).ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    try:
        _init(host)
        assert host.pm_set_checkpoint(1) == 0 and host.pm_step(32) == 0
        _init(host, edge=112)         # 32 states of 268 MB are left: the share is full
        assert host.pm_set_checkpoint(4) == 0 and host.pm_step(8) == 0
        assert host.pm_grad(grad, None, None) == 0
        before = host.fake_mallocs()
        for _ in range(3):
            assert host.pm_grad(grad, None, None) == 0
        assert host.fake_mallocs() == before
    finally:
        host.pm_finalize()


def test_kept_blocks_are_few(host):
    """Contexts of ever new sizes do not leave a growing list of small blocks."""
    host.fake_reset(288 * GB)
    try:
        for nz in range(1, 300):
            p = FIELD.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
            assert host.pm_init(N, 8, 8, 12 * nz, 0.1, 0.05, p, p, None) == 0
        assert host.fake_blocks() <= 256 + 20
    finally:
        host.pm_finalize()
