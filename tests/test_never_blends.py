"""The projection's proof that a tet cannot blend (never_blends) against the
evaluation of its pairs (pixel_eval), both taken from the device header and
compiled for the CPU: random tets, round to slivers, at every steepness, with f
rising along the rays (where the proof says yes) from flat to steep and from a
large offset, the pixel near an edge of the projection, where rounding decides
who is in front.  No tet that is left out may have a pixel that would blend."""
import os
import re
import shutil
import subprocess

import pytest

HEADER = os.path.join(os.path.dirname(__file__), "..", "paper_2406_01579_amd", "csrc", "ts_device.h")

MAIN = r"""
int main(int argc, char** argv) {
  std::mt19937_64 rng(atoi(argv[1]));
  const long n = atol(argv[2]);
  const double slo = atof(argv[3]), shi = atof(argv[4]), off = atof(argv[6]);
  const int shape = atoi(argv[5]);
  const float amin = (float)atof(argv[7]);
  auto U = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
  auto N = [&]() { return std::normal_distribution<double>()(rng); };
  auto LU = [&](double a, double b) { return exp(U(log(a), log(b))); };
  long idle = 0, pairs = 0, bad = 0;
  for (long it = 0; it < n; ++it) {
    const double Z0 = LU(0.3, 8), h = LU(0.0006, 0.2) * Z0, f0 = LU(60, 2000);
    const double c[3] = {U(-0.5, 0.5) * Z0, U(-0.5, 0.5) * Z0, Z0};
    double q[4], l = 0, P[4][3] = {{0, 0, 0}, {1, 0, 0}, {1, 1, 0}, {1, 1, 1}}, x[4][3];
    for (auto& v : q) l += (v = N()) * v;
    for (auto& v : q) v /= sqrt(l);
    const double R[3][3] = {
        {1 - 2 * (q[2] * q[2] + q[3] * q[3]), 2 * (q[1] * q[2] - q[3] * q[0]), 2 * (q[1] * q[3] + q[2] * q[0])},
        {2 * (q[1] * q[2] + q[3] * q[0]), 1 - 2 * (q[1] * q[1] + q[3] * q[3]), 2 * (q[2] * q[3] - q[1] * q[0])},
        {2 * (q[1] * q[3] - q[2] * q[0]), 2 * (q[2] * q[3] + q[1] * q[0]), 1 - 2 * (q[1] * q[1] + q[2] * q[2])}};
    const double flat = shape == 2 ? LU(1e-3, 1) : 1;
    if (shape) for (auto& p : P) for (int m = 0; m < 3; ++m) p[m] = N() * (m == 2 ? flat : 1);
    float X[4], Y[4], Z[4], px[4], py[4], f[4], D[4];
    bool near = false;
    for (int a = 0; a < 4; ++a) {
      for (int m = 0; m < 3; ++m) x[a][m] = c[m] + h * (R[m][0] * P[a][0] + R[m][1] * P[a][1] + R[m][2] * P[a][2]);
      X[a] = x[a][0], Y[a] = x[a][1], Z[a] = x[a][2];
      near = near || Z[a] < 0.05f;
    }
    if (near) continue;
    double g[3], len = 0;
    for (int m = 0; m < 3; ++m) len += (g[m] = c[m] / Z0 * LU(1e-3, 1) + N() * LU(1e-3, 1)) * g[m];
    const double steep = LU(0.3, 1) / sqrt(len) * (off > 0 ? LU(1e-7, 1) : 1), base = off > 0 ? -LU(1e-3, off) : U(-0.02, 0);
    for (int a = 0; a < 4; ++a) {
      double v = base;
      for (int m = 0; m < 3; ++m) v += steep * g[m] * (x[a][m] - c[m]);
      f[a] = v;
    }
    const float s = LU(slo, shi), fx = f0;
    // the image's centre such that pixel (i, j) lies near a point of an edge
    const int ea = rng() % 4, eb = (ea + 1 + rng() % 3) % 4, i = rng() % 1024, j = rng() % 1024;
    const double t = U(0, 1), e = h / Z0 * f0;
    const double ex = f0 * ((1 - t) * x[ea][0] / x[ea][2] + t * x[eb][0] / x[eb][2]);
    const double ey = f0 * ((1 - t) * x[ea][1] / x[ea][2] + t * x[eb][1] / x[eb][2]);
    const float cx = i + 0.5 - ex + e * LU(1e-7, 1) * (rng() & 1 ? 1 : -1), cy = j + 0.5 - ey + e * LU(1e-7, 1) * (rng() & 1 ? 1 : -1);
    float x0 = INFINITY, x1 = -INFINITY, y0 = INFINITY, y1 = -INFINITY;
    ViewRec r;
    for (int a = 0; a < 4; ++a) {
      r.px[a] = px[a] = fmaf(fx, X[a] / Z[a], cx), r.py[a] = py[a] = fmaf(fx, Y[a] / Z[a], cy);
      r.iz[a] = 1.0f / Z[a], r.f[a] = f[a];
      x0 = fminf(x0, px[a]), x1 = fmaxf(x1, px[a]), y0 = fminf(y0, py[a]), y1 = fmaxf(y1, py[a]);
    }
    for (int F = 0; F < 4; ++F) {
      const int A = face_vertex(F, 0), B = face_vertex(F, 1), C = face_vertex(F, 2);
      D[F] = (px[B] - px[A]) * (py[C] - py[A]) - (py[B] - py[A]) * (px[C] - px[A]);
      rcp_ulp = (int)(rng() % 3) - 1;
      r.rD[F] = D[F] != 0.0f ? rcp(D[F]) : 0.0f;
    }
    rcp_ulp = (int)(rng() % 3) - 1;
    const float reach = fmaxf(1.0f, fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fmaxf(fabsf(y0), fabsf(y1))) / fx);
    if (!never_blends(X, Y, Z, f, D, fmaxf(x1 - x0, y1 - y0), reach, s, amin)) continue;
    ++idle;
    for (rcp_ulp = -1; rcp_ulp <= 1; ++rcp_ulp) {
      PixEval p;
      if (!pixel_eval(r, i + 0.5f, j + 0.5f, s, p)) continue;
      ++pairs;
      bad += p.alpha >= amin ? 1 : 0;
    }
  }
  printf("%ld %ld %ld\n", idle, pairs, bad);
}
"""

PRELUDE = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
int rcp_ulp;   // the hardware reciprocal's error, in units of the last place
static float hw_rcp(float x) {
  const float r = 1.0f / x;
  return rcp_ulp == 0 ? r : std::nextafterf(r, rcp_ulp > 0 ? INFINITY : -INFINITY);
}
#define __host__
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcpf hw_rcp
#define __builtin_amdgcn_exp2f exp2f
struct ViewRec { float px[4], py[4], iz[4], f[4], rD[4]; };
"""


def _block(src, start):
    """The definition that starts with the line matching `start`, to its closing brace in column 0."""
    m = re.search(r"^" + start, src, re.M)
    assert m, start
    return src[m.start():src.index("\n}", m.start()) + 2]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = open(HEADER).read()
    fn = r"__device__ __forceinline__ \w+ "
    parts = [re.search(r"^.*float rcp\(float x\).*$", src, re.M).group(0),
             _block(src, r"__host__ __device__ constexpr int face_vertex"), _block(src, fn + "face_inside"),
             _block(src, "struct PixEval") + ";", re.search(r"^.*float fast_exp\(float x\).*$", src, re.M).group(0),
             _block(src, fn + "fast_expm1_neg"), _block(src, fn + "pixel_eval"), _block(src, fn + "never_blends")]
    d = tmp_path_factory.mktemp("never_blends")
    (d / "t.cpp").write_text(PRELUDE + "\n".join(parts) + MAIN)
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", "-w", "-o", str(d / "t"), str(d / "t.cpp")],
                   check=True)
    return str(d / "t")


@pytest.mark.parametrize("shape", [0, 1, 2])            # cell tets, random tets, flattened ones
@pytest.mark.parametrize("slo,shi,off,amin", [
    (1.0, 100.0, 0.0, 1 / 255), (300.0, 330.0, 0.0, 1 / 255), (500.0, 2000.0, 0.0, 1 / 255),
    (5e3, 1e5, 0.0, 1 / 255), (300.0, 330.0, 100.0, 1 / 255), (1e4, 1e5, 0.1, 1 / 255), (1e5, 1e7, 1.0, 1 / 255),
    (100.0, 1e4, 1.0, 1e-6), (100.0, 1e4, 1.0, 0.3)])
def test_no_pixel_of_a_left_out_tet_blends(program, shape, slo, shi, off, amin):
    out = subprocess.run([program, "1", "300000", str(slo), str(shi), str(shape), str(off), str(amin)],
                         check=True, capture_output=True, text=True).stdout
    idle, pairs, bad = map(int, out.split())
    assert idle > 0 and pairs > 0   # (the proof does leave tets out here)
    assert bad == 0
