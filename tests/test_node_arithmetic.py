"""The device code's node arithmetic on the CPU, against extended precision.

The sections of csrc/lbm_kernels.hip that hold the arithmetic of one node, and the lines of
csrc/lbm_host.cpp that fill a domain's parameters, are compiled as they stand for the host.  The
hardware's estimates are replaced by what they promise at best: the FP64 reciprocal by one of 24
bits, the FP32 reciprocal and square roots by correctly rounded ones, which take subnormals for 0 as
the instructions do.
"""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1707_00198_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

HEAD = r"""
#include <cmath>
#include <cstdint>
#include <cstring>
#include "lbm_internal.h"
#undef __device__
#undef __forceinline__
#define __device__
#define __forceinline__ inline
using namespace lbmcg;
using std::sqrt;
#define fsqrt node_fsqrt  // the C library has an fsqrt of its own
static double est_rcp(double x) { int e; const double m = std::frexp(x, &e); return std::ldexp((double)(float)(1.0 / m), -e); }
#define __builtin_amdgcn_rcp(x) est_rcp(x)
static double flush(float x) { return std::fabs(x) < 0x1p-126f ? std::copysign(0.0, (double)x) : (double)x; }
#define __builtin_amdgcn_rcpf(x) (float)(1.0 / flush(x))
#define __builtin_amdgcn_sqrtf(x) (float)std::sqrt(flush(x))
#define __builtin_amdgcn_rsqf(x) (float)(1.0 / std::sqrt(flush(x)))
template <class AT> using ParC = const DomPar<AT>;
"""

TAIL = r"""
struct Q { double nu_r, nu_b, sigma, beta, theta_deg, s_e, s_eps, s_q, rho0, eps, outlet_u; };
static const double WH[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
static void fill(const Q &q, DomDev &D) {
    const double th = q.theta_deg * M_PI / 180.0;
    %FILL%
}
static const DomPar<double> &of(const DomDev &D, double) { return D.d; }
static const DomPar<float> &of(const DomDev &D, float) { return D.f; }
// post-collision deviations, velocity and red fraction of n nodes of one pure phase (red = 1 or blue
// = 0), no force
template <class AT> static void nodes(const Q *q, int n, const AT *d, int red, AT *o, AT *u) {
    DomDev D{};
    fill(*q, D);
    for (int i = 0; i < n; i++) {
        AT rR, rB, bx, by;
        gather_interior(of(D, AT()), d + 9 * i, AT(red), rR, rB, [&](int, bool, AT &cs, AT &ev) { cs = AT(red); ev = AT(0); });
        collide(of(D, AT()), d + 9 * i, AT(0), AT(0), colour_indicator(rR, rB), rR, rB, AT(0), AT(0),
                *reinterpret_cast<AT (*)[9]>(o + 9 * i), u[3 * i], u[3 * i + 1], u[3 * i + 2], bx, by);
    }
}
extern "C" {
void nodes_f64(const Q *q, int n, const double *d, int red, double *o, double *u) { nodes(q, n, d, red, o, u); }
void nodes_f32(const Q *q, int n, const float *d, int red, float *o, float *u) { nodes(q, n, d, red, o, u); }
// densities of n interior nodes from the deviations d, the red fractions c and e_a . v of their sources
void gather_f32(const Q *q, int n, const float *d, const float *c, const float *ev, float *rho) {
    DomDev D{};
    fill(*q, D);
    for (int i = 0; i < n; i++)
        gather_interior(of(D, 0.0f), d + 9 * i, c[9 * i], rho[2 * i], rho[2 * i + 1],
                        [&](int a, bool, float &cs, float &e) { cs = c[9 * i + a]; e = ev[9 * i + a]; });
}
void normals_f64(int n, const double *g, double eps, double *out) {
    for (int i = 0; i < n; i++) unit_normal(g[2 * i], g[2 * i + 1], eps, out[3 * i], out[3 * i + 1], out[3 * i + 2]);
}
void normals_f32(int n, const float *g, float eps, float *out) {
    for (int i = 0; i < n; i++) unit_normal(g[2 * i], g[2 * i + 1], eps, out[3 * i], out[3 * i + 1], out[3 * i + 2]);
}
void quotients(int n, const double *a, const double *b, double *out) {
    for (int i = 0; i < n; i++) out[i] = quotient(a[i], b[i], rcp(b[i]));
}
}
"""


class Q(C.Structure):
    _fields_ = [(k, C.c_double) for k in ("nu_r", "nu_b", "sigma", "beta", "theta_deg", "s_e", "s_eps", "s_q", "rho0",
                                          "eps", "outlet_u")]


def _between(text, first, last):
    i = text.index(first)
    return text[i:text.index(last, i)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    k = open(os.path.join(CSRC, "lbm_kernels.hip")).read()
    h = open(os.path.join(CSRC, "lbm_host.cpp")).read()
    code = HEAD + _between(k, "// D2Q9 velocity set", "// ------------------------------------------------------------------ storage codec")
    code += _between(k, "// e_a . v of a colour state", "// Completes the post-streaming populations")
    code += _between(k, "// MRT collision with Guo forcing", "// Work item of block b")
    code += TAIL.replace("%FILL%", _between(h, "DomPar<double> &PD = D.d;", "int n_fluid_bnd = 0;"))
    d = tmp_path_factory.mktemp("node")
    src, so = str(d / "node.cpp"), str(d / "node.so")
    with open(src, "w") as f:
        f.write(code)
    subprocess.check_call([os.path.join(ROCM, "llvm", "bin", "clang++"), "-std=c++17", "-O2", "-mfma", "-fPIC", "-shared", "-w",
                           "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", CSRC, "-o", so, src])
    return C.CDLL(so)


def _params(nu_r, nu_b):
    return Q(nu_r, nu_b, 0.01, 0.7, 90.0, 1.64, 1.54, 1.9, 1.0, 1e-10, 0.0)


def _nodes(lib, q, d, red):
    o, u = np.empty_like(d), np.empty((len(d), 3), d.dtype)
    p = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    (lib.nodes_f64 if d.dtype == np.float64 else lib.nodes_f32)(C.byref(q), len(d), p(d), red, p(o), p(u))
    return o, u


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("nu,ratio", [(0.3, 1000.0), (0.45, 1000.0), (0.137, 1000.0), (1.0 / 6.0, 50.0), (0.35, 100.0)])
def test_viscosity_of_a_pure_phase(lib, nu, ratio, dtype):
    """s_nu of either pure phase, whichever is the viscous one, from a node that holds nothing but
    the normal stress m_7.  Rounded are the stored 1/(2 nu) (half a unit), the sum with 3, the
    product and the step's own m_7 (half a unit each) and the reciprocal (one): 4 units, with u the
    spacing at 1."""
    a = dtype(2.0 ** -6)
    d = np.array([[0, a, -a, a, -a, 0, 0, 0, 0]], dtype)
    for red in (1, 0):
        o, _ = _nodes(lib, _params(*((nu, nu / ratio) if red else (nu / ratio, nu))), d, red)
        m7 = np.longdouble(o[0, 1]) - o[0, 2] + o[0, 3] - o[0, 4]
        s = 1 - m7 / (4 * np.longdouble(a))
        want = 1 / (3 * np.longdouble(nu) + np.longdouble(0.5))
        assert abs(s / want - 1) <= 4 * np.finfo(dtype).eps, (red, float(s / want - 1))


def test_velocity_takes_the_density_from_the_deviations(lib):
    """Deviations that are multiples of 2^-20 below 1/8: their sums, and 1 plus their sum, are exact
    in FP32, so the velocity of a force-free node carries the roundings of the reciprocal and of
    the product alone, half a unit each.  The sum of nine populations w_a + d_a, each rounded, would
    bring its own.  The red fraction, by the same reciprocal, is exactly 1."""
    rng = np.random.default_rng(11)
    d = (rng.integers(-2 ** 17, 2 ** 17, (20000, 9)) * 2.0 ** -20).astype(np.float32)
    e = np.array([[0, 0], [1, 0], [0, 1], [-1, 0], [0, -1], [1, 1], [-1, 1], [-1, -1], [1, -1]], np.float64)
    _, u = _nodes(lib, _params(0.5, 0.25), d, 1)
    want = (d.astype(np.float64) @ e) / (1.0 + d.astype(np.float64).sum(axis=1))[:, None]
    assert (u[:, 2] == 1).all()
    some = np.abs(want) > 0
    err = np.abs(u[:, :2][some] / want[some] - 1.0)
    assert err.max() <= np.finfo(np.float32).eps * (1 + 2.0 ** -20), err.max()


def test_fp64_divisions_round_as_the_ieee_division(lib):
    """Quotients by Newton steps and a residual correction: two steps from an estimate of 24 bits
    leave 2^-90 before the last rounding, so a quotient differs from the correctly rounded one only
    where that lies within about 2^-38 units of a tie (none in 1e5 to expect).  The unit normal is
    the gradient over the modulus that comes with it, 0 up to the threshold."""
    rng = np.random.default_rng(5)
    n = 100000
    p = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    a, b, out = rng.uniform(-1.0, 1.0, n), rng.uniform(0.5, 2.0, n), np.empty(n)
    lib.quotients(n, p(a), p(b), p(out))
    assert np.array_equal(out, a / b)
    g, r = rng.uniform(-1.0, 1.0, (n, 2)) * 10.0 ** rng.uniform(-9.0, 0.0, (n, 1)), np.empty((n, 3))
    lib.normals_f64(n, p(g), C.c_double(1e-10), p(r))
    assert np.array_equal(r[:, 1:], np.where(r[:, :1] > 1e-10, g / r[:, :1], 0.0))
    # below the threshold, and where there is no gradient at all
    g, r = np.array([[0.0, 0.0], [6e-11, -7e-11], [0.0, -1e-10]]), np.empty((3, 3))
    lib.normals_f64(3, p(g), C.c_double(1e-10), p(r))
    assert np.array_equal(r[:, 1:], np.zeros((3, 2)))


def test_fp32_normals(lib):
    """The FP32 modulus and normal against FP64: half a unit from the square's sum and its two products
    each (the root halves them), one from the reciprocal root and half from the product.  Gradients
    whose square is subnormal or 0 are below any threshold that single precision can tell from 0."""
    rng = np.random.default_rng(6)
    n = 100000
    p = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    g, r = (rng.uniform(-1.0, 1.0, (n, 2)) * 10.0 ** rng.uniform(-9.0, 0.0, (n, 1))).astype(np.float32), np.empty((n, 3), np.float32)
    lib.normals_f32(n, p(g), C.c_float(1e-10), p(r))
    m = np.hypot(*g.astype(np.float64).T)
    on = m > 1.1e-10
    want = np.column_stack([m, g / m[:, None]])[on]
    assert np.abs(r[on] - want).max(axis=0)[1:].max() <= 3 * 2.0 ** -23 and (np.abs(r[on, 0] / m[on] - 1) <= 3 * 2.0 ** -23).all()
    g = (rng.uniform(-1.0, 1.0, (n, 2)) * 10.0 ** rng.uniform(-25.0, -19.3, (n, 1))).astype(np.float32)
    g[:3] = [[0, 0], [0, 1e-20], [1e-22, 0]]
    lib.normals_f32(n, p(g), C.c_float(1e-10), p(r))
    assert not r.any()
    lib.normals_f32(n, p(g), C.c_float(1e-30), p(r))
    assert np.isfinite(r).all() and np.abs(r[:, 1:]).max() <= 1.0 + 2.0 ** -22


def test_fp32_densities_of_the_minority_colour(lib):
    """The blue density of nearly red nodes carries the rounding of each red part alone: half a unit
    of populations near 4/9 (2^-26), 1/9 (2^-28) and 1/36 (2^-30), 1.125 x 2^-25 over the nine (the
    parts' own sums are a thousand times smaller), where the total minus the red density would add
    the roundings of two sums of order one.  Pure nodes are exactly pure."""
    rng = np.random.default_rng(7)
    n = 20000
    p = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, np.float32)
    d = (rng.uniform(-0.02, 0.02, (n, 9)) * w).astype(np.float32)
    c = (1.0 - 10.0 ** rng.uniform(-7.0, -3.0, (n, 9))).astype(np.float32)
    ev = ((1 - c) * rng.uniform(-0.5, 0.5, (n, 9))).astype(np.float32)
    ev[:, 0] = 0
    rho = np.empty((n, 2), np.float32)
    lib.gather_f32(C.byref(_params(0.5, 0.25)), n, p(d), p(c), p(ev), p(rho))
    f, ld = (w + d).astype(np.longdouble), np.longdouble
    want = ((1 - c.astype(ld)) * f - w.astype(ld) * ev).sum(axis=1)
    assert np.abs(rho[:, 1] - want).max() <= 1.125 * 2.0 ** -25 + 9 * 2.0 ** -34
    for pure in (0, 1):
        c[:], ev[:] = pure, 0
        lib.gather_f32(C.byref(_params(0.5, 0.25)), n, p(d), p(c), p(ev), p(rho))
        assert (rho[:, 1 - pure] > 0).all() and not rho[:, pure].any()
