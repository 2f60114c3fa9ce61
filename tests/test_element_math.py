"""The element physics of csrc/device_math.h in FP32, compiled for the CPU, against its textbook form in
FP64: first Piola stress and conduction of warm tissue under small elastic strains.

Bound: what forming F_e - I = H / l - (l - 1) / l in FP32 brings by itself (the rest of the textbook form then
evaluated in FP64), and 8 u, u = 2^-24, for the chain from that gradient to the stress, whose roundings are
relative to the stress.  Conduction (scale, stretch, volume ratio and a product with I - N): 6 u."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_10400_amd", "csrc")
U = 2.0 ** -24

STUB = r"""
#pragma once
#include <cmath>
#include <cstdint>
#include <cstddef>
#include <cstring>
#define __device__
#define __forceinline__ inline
struct float4 { float x, y, z, w; };
static inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
static inline float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }
static inline float __builtin_amdgcn_logf(float x) { return log2f(x); }
static inline float rsqrtf(float x) { return 1.0f / sqrtf(x); }
"""

MAIN = r"""
#include <hip/hip_runtime.h>
#include "device_math.h"
using namespace tled;
extern "C" int element(int mode, int n, const KMat *m, size_t size, const float *H, const float *gT, const float *dT,
                       const float *a, float V0, float *PV, float *qV, float *Jmin) {
    if (size != sizeof(KMat)) return 1;
    for (int i = 0; i < n; ++i) {
        ElemOut o;
        float th[1];
        if (mode == kIso) element_physics<0, kIso>(*m, H + 9 * i, gT + 3 * i, dT[i], a + 3 * i, V0, th, false, o, nullptr, i);
        else element_physics<0, kTi>(*m, H + 9 * i, gT + 3 * i, dT[i], a + 3 * i, V0, th, false, o, nullptr, i);
        memcpy(PV + 9 * i, o.PV, sizeof(o.PV));
        memcpy(qV + 3 * i, o.qV, sizeof(o.qV));
        Jmin[i] = o.Jmin;
    }
    return 0;
}
"""

F, I = ctypes.c_float, ctypes.c_int


class KMat(ctypes.Structure):
    _fields_ = ([(k, F) for k in ("mu", "kappa", "eta", "alpha", "alpha_m", "alpha_n", "k", "k_m", "muT_off", "muT_inv",
                                  "muT_drop", "sh_off", "sh_inv", "sh_eps", "ck_off", "ck_inv", "c_lo", "c_hi", "kr_hi")]
                + [("pc1", F * 4), ("pc2", F * 4), ("hgk", F)]
                + [(k, I) for k in ("n_prony", "expan_mode", "cond_mode", "muT_on", "shrink_on", "ckT_on")])


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("element_math")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    so = str(d / "libelement.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fno-fast-math", "-w", "-shared", "-fPIC",
                           f"-I{d}", f"-I{CSRC}", str(d / "main.cpp"), "-o", so])
    return ctypes.CDLL(so)


def material(expan_mode=0, cond_mode=0, shrink=0.0):
    m = KMat(mu=1007.0, kappa=50000.0, eta=2500.0, alpha=1e-4, alpha_m=2.5e-4, k=0.5, k_m=0.8, expan_mode=expan_mode,
             cond_mode=cond_mode)
    if shrink:
        m.shrink_on, m.sh_off, m.sh_inv, m.sh_eps = 1, -20.0, 0.1, shrink
    return m


def stretch_m1(m, dT):
    """lambda - 1 in dT's precision, in small quantities."""
    t = m.alpha * dT
    if m.shrink_on:
        s1 = m.sh_eps * np.clip((dT + dT.dtype.type(m.sh_off)) * dT.dtype.type(m.sh_inv), 0, 1)
        t = t + s1 + s1 * t
    return t


def textbook(m, H, gT, dT, a, V0, He=None):
    """Table 5's stress on F_e = F F_th^-1 (I + He if given), pulled back; J F^-1 D F^-T grad T: all in FP64."""
    H, gT, dT, a = (np.asarray(x, np.float64) for x in (H, gT, dT, a))
    I3 = np.eye(3)
    a = a / np.linalg.norm(a, axis=1, keepdims=True)
    A0 = a[:, :, None] * a[:, None, :]
    li = 1.0 + stretch_m1(m, dT)
    lm = 1.0 + m.alpha_m * dT if m.expan_mode == 1 else li
    Fi = (1.0 / li)[:, None, None] * I3 + (1.0 / lm - 1.0 / li)[:, None, None] * A0
    Ft = H + I3
    Fe = Ft @ Fi if He is None else I3 + He
    C = Fe.transpose(0, 2, 1) @ Fe
    J, Ci = np.linalg.det(Fe), np.linalg.inv(C)
    I1, I4 = np.trace(C, axis1=1, axis2=2), (C * A0).sum((1, 2))
    j = J ** (-2.0 / 3.0)

    def e(w):
        return np.asarray(w)[:, None, None]

    S = (e(m.mu * j) * (I3 - e(I1 / 3.0) * Ci) + e(2.0 * m.eta * (j * I4 - 1.0) * j) * (A0 - e(I4 / 3.0) * Ci)
         + e(m.kappa * J * (J - 1.0)) * Ci)
    S = e(li * li * lm) * (Fi @ S @ Fi)
    Fn = np.linalg.inv(Ft)
    D = m.k * I3 + ((m.k_m - m.k) * A0 if m.cond_mode == 1 else 0.0)
    K = e(np.linalg.det(Ft)) * (Fn @ D @ Fn.transpose(0, 2, 1))
    return V0 * (Ft @ S), V0 * np.einsum("nij,nj->ni", K, gT)


def run(lib, mode, m, H, gT, dT, a, V0):
    n = len(dT)
    PV, qV, Jm = np.empty((n, 3, 3), np.float32), np.empty((n, 3), np.float32), np.empty(n, np.float32)

    def p(x):
        return x.ctypes.data_as(ctypes.c_void_p)

    assert lib.element(mode, n, ctypes.byref(m), ctypes.c_size_t(ctypes.sizeof(m)), p(H), p(gT), p(dT), p(a), F(V0), p(PV),
                       p(qV), p(Jm)) == 0
    return PV, qV, Jm


@pytest.mark.parametrize("dT,shrink,elastic", [(0.0, 0.0, 1e-4), (25.0, 0.0, 1e-4), (100.0, 0.0, 1e-4), (40.0, -0.054, 1e-3),
                                               (25.0, -0.1, 1e-3), (25.0, 0.0, 3e-2)])
@pytest.mark.parametrize("mode", [0, 1])
def test_stress_and_conduction_of_warm_tissue(lib, mode, dT, shrink, elastic):
    m, n = material(shrink=shrink), 20000
    rng = np.random.default_rng(11)
    t = (dT * rng.uniform(0.99, 1.01, n)).astype(np.float32)
    stretch = 1.0 + stretch_m1(m, t.astype(np.float64))
    Fe = np.eye(3) + elastic * rng.standard_normal((n, 3, 3))
    H = np.ascontiguousarray((stretch[:, None, None] * Fe - np.eye(3)), np.float32)
    a = rng.standard_normal((n, 3))
    a = np.ascontiguousarray(a / np.linalg.norm(a, axis=1, keepdims=True), np.float32)
    gT = (1e3 * rng.standard_normal((n, 3))).astype(np.float32)
    V0 = float(np.float32(1e-9))
    PV, qV, Jmin = run(lib, mode, m, H, gT, t, a, V0)
    P64, q64 = textbook(m, H, gT, t, a, V0)
    # the elastic gradient in FP32
    f32 = np.float32
    t1 = stretch_m1(m, t)
    inv = f32(1) / (f32(1) + t1)
    He = H * inv[:, None, None] - (t1 * inv)[:, None, None] * np.eye(3, dtype=f32)
    assert He.dtype == f32
    split, _ = textbook(m, H, gT, t, a, V0, He.astype(np.float64))

    def rms(x):
        return float(np.sqrt((np.asarray(x, np.float64) ** 2).mean()))

    err, q_err = rms(PV - P64) / rms(P64), rms(qV - q64) / rms(q64)
    bound = rms(split - P64) / rms(P64) + 8 * U
    print(f"  mode {mode} dT {dT} shrink {shrink} elastic {elastic}: stress {err:.2e} (bound {bound:.2e}) conduction {q_err:.2e}")
    assert err <= bound
    assert q_err <= 6 * U
    J = np.linalg.det(H.astype(np.float64) + np.eye(3))
    assert np.all((Jmin > 0) == (J > 0))


def test_isotropic_code_is_the_same_in_both_forms(lib):
    """An isotropic problem gives the same bits from the kernels that hold the isotropic modes only and from
    those that also hold the transversely isotropic ones (the batch's persistent kernel, the end of a chunk
    that gave up)."""
    m, n = material(shrink=-0.05), 2000
    rng = np.random.default_rng(5)
    H = np.ascontiguousarray(0.3 * rng.standard_normal((n, 3, 3)), np.float32)
    a = rng.standard_normal((n, 3))
    a = np.ascontiguousarray(a / np.linalg.norm(a, axis=1, keepdims=True), np.float32)
    gT = rng.standard_normal((n, 3)).astype(np.float32)
    t = rng.uniform(0, 60, n).astype(np.float32)
    for x, y in zip(run(lib, 0, m, H, gT, t, a, 1.0), run(lib, 1, m, H, gT, t, a, 1.0)):
        assert np.array_equal(x, y, equal_nan=True)


@pytest.mark.parametrize("expan,cond", [(1, 0), (0, 1), (1, 1)])
def test_transversely_isotropic_modes(lib, expan, cond):
    m, n = material(expan, cond), 20000
    rng = np.random.default_rng(7)
    t = rng.uniform(20.0, 30.0, n).astype(np.float32)
    a = rng.standard_normal((n, 3))
    a = np.ascontiguousarray(a / np.linalg.norm(a, axis=1, keepdims=True), np.float32)
    H = np.ascontiguousarray(m.alpha * t[:, None, None] * np.eye(3) + 1e-3 * rng.standard_normal((n, 3, 3)), np.float32)
    gT = (1e3 * rng.standard_normal((n, 3))).astype(np.float32)
    PV, qV, _ = run(lib, 1, m, H, gT, t, a, 1e-9)
    P64, q64 = textbook(m, H, gT, t, a, float(np.float32(1e-9)))
    assert np.sqrt(((PV - P64) ** 2).mean() / (P64 ** 2).mean()) <= 16 * U * (1 + m.alpha_m * 30 / 1e-3)
    assert np.sqrt(((qV - q64) ** 2).mean() / (q64 ** 2).mean()) <= 12 * U
