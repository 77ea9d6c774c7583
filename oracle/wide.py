"""L(U) of a leaf in 80-bit arithmetic, from the wide build of the oracle
(wide.cpp).  TEST INFRASTRUCTURE."""
from __future__ import annotations

import ctypes as C
import os
import subprocess

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "wide.cpp")
LIB = os.path.join(HERE, "_build", "libwide.so")


def build() -> str:
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(
            os.path.getmtime(SRC), os.path.getmtime(os.path.join(HERE, "hydro_oracle.c"))):
        subprocess.check_call(["g++", "-O2", "-ffp-contract=off", "-std=c++17", "-fPIC", "-shared", "-w",
                               "-o", LIB + ".tmp", SRC])
        os.replace(LIB + ".tmp", LIB)
    return LIB


def rhs(P, dx, origin, gamma, omega=0.0, eta1=1e-3):
    """L(U) [n][7][8][8][8] (long double) of padded blocks P [n][7][14][14][14]."""
    L = C.CDLL(build())
    dp = C.POINTER(C.c_double)
    L.wide_leaf_rhs.argtypes = [dp, C.c_double, dp, C.c_double, C.c_double, C.c_double, C.c_void_p]
    P = np.ascontiguousarray(P, dtype=np.float64)
    out = np.empty((P.shape[0], 7, 8, 8, 8), dtype=np.longdouble)
    for i in range(P.shape[0]):
        org = np.ascontiguousarray(origin[i], dtype=np.float64)
        L.wide_leaf_rhs(P[i].ctypes.data_as(dp), float(dx[i]), org.ctypes.data_as(dp), gamma, omega, eta1,
                        out[i].ctypes.data)
    return out
