"""Which contexts share copy streams (csrc/copy_pool.h, compiled for the host): those whose copies wait
for the same compute stream of the same device, and no others; no pair is lost or used after its end."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "copy_pool.h"
using namespace k3lms;
static CopyPool pool;
static long made = 0, fail = 0;
extern "C" {
void *lease(void *have, int device, long compute)
{
    return pool.lease((CopyPair *)have, device, (stream_t)compute, [](CopyPair &p) {
        if (fail) return 1;
        p.d2h = (stream_t)(++made);
        p.h2d = (stream_t)(++made);
        return 0;
    });
}
int give_back(void *have, int device)
{
    auto out = pool.give_back((CopyPair *)have, device);
    for (CopyPair *p : out) delete p;
    return (int)out.size();
}
long d2h(void *p) { return (long)((CopyPair *)p)->d2h; }
int users(void *p) { return ((CopyPair *)p)->users; }
void fail_next(int f) { fail = f; }
}
"""


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    d = tmp_path_factory.mktemp("copy_pool")
    cpp, so = str(d / "copy_pool.cpp"), str(d / "copy_pool.so")
    with open(cpp, "w") as f:
        f.write(SRC)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "paper_1811_12174_amd", "csrc"), "-o", so, cpp])
    L = ctypes.CDLL(so)
    L.lease.restype, L.lease.argtypes = ctypes.c_void_p, [ctypes.c_void_p, ctypes.c_int, ctypes.c_long]
    L.give_back.argtypes = [ctypes.c_void_p, ctypes.c_int]
    L.d2h.restype, L.d2h.argtypes = ctypes.c_long, [ctypes.c_void_p]
    L.users.argtypes = [ctypes.c_void_p]
    return L


def test_pairs_follow_the_compute_stream(L):
    a, b, c = L.lease(None, 0, 0), L.lease(None, 0, 0), L.lease(None, 0, 7)
    assert a == b != c and L.users(a) == 2           # the default stream's two share, the other stream's has its own
    d = L.lease(None, 1, 0)
    assert d not in (a, c)                           # another device
    assert L.lease(a, 0, 0) == a and L.users(a) == 2
    c = L.lease(c, 0, 8)                             # alone: its pair goes with it
    assert L.users(c) == 1 and L.lease(c, 0, 8) == c
    b2 = L.lease(b, 0, 9)                            # leaves the shared one
    assert b2 not in (a, c) and L.users(a) == 1
    b3 = L.lease(b2, 0, 0)                           # and comes back; its own is spare now
    assert b3 == a and L.users(a) == 2 and L.users(b2) == 0
    e = L.lease(None, 0, 11)                         # who takes the spare one over
    assert e == b2
    f = L.lease(c, 0, 11)                            # two streams become one: c's pair is spare
    assert f == e and L.users(e) == 2
    assert L.give_back(a, 0) == 1                    # (that one), the shared ones stay
    assert L.give_back(b3, 0) == 1 and L.give_back(e, 0) == 0 and L.give_back(f, 0) == 1
    assert L.give_back(d, 1) == 1 and L.give_back(None, 0) == 0


def test_a_failed_creation_changes_nothing(L):
    a = L.lease(None, 0, 1)
    b = L.lease(None, 0, 1)
    L.fail_next(1)
    assert L.lease(None, 0, 2) is None and L.lease(b, 0, 2) is None and L.users(a) == 2
    L.fail_next(0)
    assert L.give_back(a, 0) == 0 and L.give_back(b, 0) == 1
