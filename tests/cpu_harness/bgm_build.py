"""Compile the host (CPU) builds of the two-sided recursion for the tests."""
import ctypes
import os
import subprocess

import numpy as np

from .build import CSRC, HERE, OUT

DEPS = [os.path.join(CSRC, h) for h in ('me_device.h', 'me_bg.h', 'me_bgh.h', 'me_bgm.h', 'me_bgm_shape.h',
                                        'me_bgm_tables.h', 'me_bg_desc.h', 'me_pair_desc.h')]


def _lib(name, opt):
    os.makedirs(OUT, exist_ok=True)
    src, lib = os.path.join(HERE, name + '.cpp'), os.path.join(OUT, name + '.so')
    if not os.path.exists(lib) or os.path.getmtime(lib) < max(os.path.getmtime(d) for d in DEPS + [src]):
        subprocess.run(['g++', opt, '-std=c++17', '-shared', '-fPIC', '-I', HERE, '-I', CSRC, src, '-o', lib + '.tmp'],
                       check=True)
        os.replace(lib + '.tmp', lib)
    return ctypes.CDLL(lib)


def jamps(n, mom, g, mt):
    """(dual amplitudes [nevt][2^(n+1)][n!], helicity index of each row) of n-gluon events."""
    import math
    mom = np.ascontiguousarray(mom, dtype=np.float64)
    rows = 2 << n
    out = np.zeros((mom.shape[0], rows, math.factorial(n), 2))
    hel = np.zeros(rows, dtype=np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    assert _lib('bgm_harness', '-O2').harness_bgm_eval(n, p(mom), mom.shape[0], ctypes.c_double(g),
                                                       ctypes.c_double(mt), p(out), p(hel)) == 0
    return out[..., 0] + 1j * out[..., 1], hel


def table_words_off(n):
    """Words of the built work-item tables beyond those the kernels index."""
    return _lib('bgm_harness', '-O2').harness_bgm_words(n)


def sectors(n, cf):
    """(orbits [norb][2^nsym], sector matrices [2^nsym][norb][norb]) of a colour matrix."""
    cf = np.ascontiguousarray(cf, dtype=np.int32)
    g = 2 << (n // 2)
    orb, sec = np.zeros(len(cf) * 2, dtype=np.int32), np.zeros(g * 64 * 64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    no = _lib('bgm_harness', '-O2').harness_bgm_sectors(n, p(cf), p(orb), p(sec))
    return orb[:no * g].reshape(no, g), sec[:g * no * no].reshape(g, no, no)


def row(n, h):
    """Row of helicity index h of n gluons."""
    return _lib('bgm_harness', '-O2').harness_bgm_row(n, h)


def mirror_pairs(good, nhel):
    """[(lower helicity index, good helicities of the pair)] of a list of good helicities."""
    good, pairs = np.ascontiguousarray(good, dtype=np.int32), np.zeros(nhel, dtype=np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    k = _lib('bgm_harness', '-O2').harness_mirror_pairs(p(good), len(good), nhel, p(pairs))
    return [(int(x) & 0xffff, int(x) >> 16) for x in pairs[:k]]


def draw(w, t):
    """(entry drawn from the weights w at running sum t, the running sum before each lane's two)."""
    w, cum = np.ascontiguousarray(w, dtype=np.float64), np.zeros(64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    return _lib('bgm_harness', '-O2').harness_bgm_draw(len(w), p(w), ctypes.c_double(t), p(cum)), cum


def count_event(n, mom):
    """Counted operations of one event: set-up, stored currents, spinors, Q.J, prefix items."""
    m = np.ascontiguousarray(mom, dtype=np.float64)
    out = (ctypes.c_longlong * 5)()
    assert _lib('count_bgm_harness', '-O1').count_bgm_event(n, m.ctypes.data_as(ctypes.c_void_p), out) == 0
    return list(out)
