// Device-side helpers of the gfx950 tetrahedron rasterizer.
//
// The library is compiled with -ffp-contract=off: every fused multiply-add
// is written out with fmaf(), so the binning quantities (projected
// vertices, pixel rectangles, depth keys, face determinants, coverage
// signs) come from a fixed IEEE operation sequence.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ts_internal.h"

namespace ts {

__device__ __forceinline__ int find_view_by_tile(const DevView* views, int nv, int tile) {
  int lo = 0, hi = nv - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_base <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Eq. 1 in the stable form alpha = -expm1(-s d) / (1 + exp(s f_next)),
// d = f_prev - f_next; zero unless d > 0 (the max(., 0) of Eq. 1).
__device__ __forceinline__ float alpha_eq1(float fprev, float fnext, float s) {
  float d = fprev - fnext;
  if (!(d > 0.0f)) return 0.0f;
  return -expm1f(-(s * d)) / (1.0f + expf(s * fnext));
}

// face vertex table: (0,1,2) (0,1,3) (0,2,3) (1,2,3)
__host__ __device__ constexpr int face_vertex(int F, int k) {
  return F == 0 ? (k == 0 ? 0 : k == 1 ? 1 : 2)
       : F == 1 ? (k == 0 ? 0 : k == 1 ? 1 : 3)
       : F == 2 ? (k == 0 ? 0 : k == 1 ? 2 : 3)
                : (k == 0 ? 1 : k == 1 ? 2 : 3);
}

// rD: 1 / D, or 0 where D == 0 (it has D's sign).  Written without branches
// (bitwise on the comparisons), so the four faces' tests are plain compares
// rather than divergent blocks that each wait for their own LDS operands.
__device__ __forceinline__ bool face_inside(float N0, float N1, float N2, float rD) {
  const bool up = (N0 >= 0.0f) & (N1 >= 0.0f) & (N2 >= 0.0f);
  const bool down = (N0 <= 0.0f) & (N1 <= 0.0f) & (N2 <= 0.0f);
  return ((rD > 0.0f) & up) | ((rD < 0.0f) & down);
}

// One pixel centre against one record.  For a projected face (A,B,C) the
// rows of the inverse barycentric system times [p;1] (App. A.1) are
// N = (cross(B',C'), cross(C',A'), cross(A',B')) over D, with X' = X - p;
// the pixel is inside iff the three N have the sign of D (D == 0: never).
// The six edge cross products e_ij = cross(P_i - p, P_j - p) give every N
// exactly (a swapped pair is an exact negation).  Along the ray, with
// w_k = 1/Z_k (App. A.2):  f = sum N_k w_k f_k / sum N_k w_k,
// 1/z = sum N_k w_k / D.  Entry = nearest hit face, exit = farthest; the
// interpolated f is divided out for those two faces only.
struct PixEval {
  float ax[4], ay[4];
  float N[4][3];
  float S[4];
  float fin, fout; // f at the entry / exit face
  int fe, fx;      // entry / exit face
  float zin_inv;   // 1 / depth where the ray enters (entry face); larger is nearer
  float alpha;     // Eq. 1 (unclamped)
  float e1, e2;    // expm1(-s d), exp(s f_next) (for the derivative)
};

// Image planes and scene arrays are reached through pointers read from a
// descriptor, which the compiler treats as generic (flat) addresses.  A flat load also
// counts against the LDS wait counter, so every LDS wait after it waits for
// the load too; through a global-space pointer it does not.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gmem(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

// What a kernel only reads and one workgroup reads alike (its slot, its view),
// through the constant space: by scalar loads into scalar registers, beside
// the vector loads' counter instead of in it.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* cmem(const T* p) {
  return (const __attribute__((address_space(4))) T*)p;
}

// A tet's four vertex ids through a global-space pointer.
__device__ __forceinline__ int4 load_tet(const int32_t* tets, size_t k) {
  const auto* t = gmem(tets) + 4 * k;
  return make_int4(t[0], t[1], t[2], t[3]);
}

// Float atomic add to device memory through a global-space pointer (for a
// pointer read from a descriptor; see gmem).
__device__ __forceinline__ void gatomic_add(float* p, float v) {
  __hip_atomic_fetch_add(gmem(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wave-uniform float moved into a scalar register: its load is waited for
// here, once, and not at its first use inside a loop, where the wait would
// also cover every load the loop's prefetch has in flight.
__device__ __forceinline__ float uniform_f(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// exp(x) from the hardware base-2 exponential
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

// expm1(x) for x <= 0: Taylor series through x^7/5040 on [-0.25, 0] (truncation
// below 1e-9 relative), exp(x) - 1 below (no cancellation there).
__device__ __forceinline__ float fast_expm1_neg(float x) {
  float p = fmaf(x, 1.0f / 5040.0f, 1.0f / 720.0f);
  p = fmaf(x, p, 1.0f / 120.0f);
  p = fmaf(x, p, 1.0f / 24.0f);
  p = fmaf(x, p, 1.0f / 6.0f);
  p = fmaf(x, p, 0.5f);
  p = fmaf(x, p, 1.0f);
  const float small = x * p;
  const float big = fast_exp(x) - 1.0f;
  return x > -0.25f ? small : big;
}

__device__ __forceinline__ bool pixel_eval(const ViewRec& r, float qx, float qy, float s, PixEval& h) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    h.ax[k] = r.px[k] - qx;
    h.ay[k] = r.py[k] - qy;
  }
  const float e01 = h.ax[0] * h.ay[1] - h.ay[0] * h.ax[1];
  const float e02 = h.ax[0] * h.ay[2] - h.ay[0] * h.ax[2];
  const float e03 = h.ax[0] * h.ay[3] - h.ay[0] * h.ax[3];
  const float e12 = h.ax[1] * h.ay[2] - h.ay[1] * h.ax[2];
  const float e13 = h.ax[1] * h.ay[3] - h.ay[1] * h.ax[3];
  const float e23 = h.ax[2] * h.ay[3] - h.ay[2] * h.ax[3];
  h.N[0][0] = e12; h.N[0][1] = -e02; h.N[0][2] = e01;
  h.N[1][0] = e13; h.N[1][1] = -e03; h.N[1][2] = e01;
  h.N[2][0] = e23; h.N[2][1] = -e03; h.N[2][2] = e02;
  h.N[3][0] = e23; h.N[3][1] = -e13; h.N[3][2] = e12;
  // every face is evaluated (no branches); only inside faces are selected
  int nh = 0;
  float best_in = -INFINITY, best_out = INFINITY;
  float num_in = 0.0f, S_in = 1.0f, num_out = 0.0f, S_out = 1.0f;
  h.fe = 0;
  h.fx = 0;
#pragma unroll
  for (int F = 0; F < 4; ++F) {
    const bool in = face_inside(h.N[F][0], h.N[F][1], h.N[F][2], r.rD[F]);
    const int A = face_vertex(F, 0), B = face_vertex(F, 1), C = face_vertex(F, 2);
    const float qa = h.N[F][0] * r.iz[A], qb = h.N[F][1] * r.iz[B], qc = h.N[F][2] * r.iz[C];
    const float S = (qa + qb) + qc;
    const float num = fmaf(qa, r.f[A], fmaf(qb, r.f[B], qc * r.f[C]));
    const float invz = S * r.rD[F];  // 1 / depth at the hit: larger is nearer
    h.S[F] = S;
    nh += in ? 1 : 0;
    const bool bi = in && invz > best_in, bo = in && invz < best_out;
    best_in = bi ? invz : best_in;
    num_in = bi ? num : num_in;
    S_in = bi ? S : S_in;
    h.fe = bi ? F : h.fe;
    best_out = bo ? invz : best_out;
    num_out = bo ? num : num_out;
    S_out = bo ? S : S_out;
    h.fx = bo ? F : h.fx;
  }
  const float fin = num_in * rcp(S_in), fout = num_out * rcp(S_out);
  h.fin = fin;
  h.fout = fout;
  h.zin_inv = best_in;
  // Eq. 1, stable form, with the hardware exponential
  const float d = fin - fout;
  const bool pos = d > 0.0f;
  const float x = pos ? -(s * d) : 0.0f;
  h.e1 = fast_expm1_neg(x);
  h.e2 = pos ? fast_exp(s * fout) : 0.0f;
  h.alpha = pos ? -h.e1 * rcp(1.0f + h.e2) : 0.0f;
  return nh >= 2;
}

// The same pixel against the same record for the kernels that share a tile
// between waves: the same results, bit for bit, from fewer instructions.  A
// ray meets two faces of a tet, so instead of evaluating four and selecting
// among their sums (seven selects a face), the operands of the first and the
// last inside face are selected (most are shared: faces 0 and 1 contain edge
// 01, faces 2 and 3 edge 23) and only those two evaluated: 91 instructions
// against 114.  A pixel on a projected edge can be inside three or four faces;
// it goes through them one by one (a loop, which needs no registers of its own).
// With the pixel's lookup (for_each_pair) 222 to 160 instructions a pair:
// forward 83 to 79 us at 4 x 512^2, 772 to 728 us at 8 x 1024^2.
struct PixHit {
  float alpha;     // Eq. 1 (unclamped)
  float e2;        // exp(s f_next)
  float zin_inv;   // 1 / depth where the ray enters
  int faces;       // entry face | exit face << 2
};

template <class Rec>
__device__ __forceinline__ bool pixel_hit(const Rec& r, float qx, float qy, float s, PixHit& h) {
  float ax[4], ay[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ax[k] = r.px[k] - qx;
    ay[k] = r.py[k] - qy;
  }
  const float e01 = ax[0] * ay[1] - ay[0] * ax[1];
  const float e02 = ax[0] * ay[2] - ay[0] * ax[2];
  const float e03 = ax[0] * ay[3] - ay[0] * ax[3];
  const float e12 = ax[1] * ay[2] - ay[1] * ax[2];
  const float e13 = ax[1] * ay[3] - ay[1] * ax[3];
  const float e23 = ax[2] * ay[3] - ay[2] * ax[3];
  // copies, so that the selections below are made among registers
  const float iz0 = r.iz[0], iz1 = r.iz[1], iz2 = r.iz[2], iz3 = r.iz[3];
  const float f0 = r.f[0], f1 = r.f[1], f2 = r.f[2], f3 = r.f[3];
  const float4 rD = *reinterpret_cast<const float4*>(r.rD);
  // face_inside of the four faces as masks over the wave: every compare leaves
  // a mask in scalar registers, and they are combined there
  const uint64_t p01 = __ballot(e01 >= 0.0f), n01 = __ballot(e01 <= 0.0f), p02 = __ballot(e02 >= 0.0f);
  const uint64_t n02 = __ballot(e02 <= 0.0f), p03 = __ballot(e03 >= 0.0f), n03 = __ballot(e03 <= 0.0f);
  const uint64_t p12 = __ballot(e12 >= 0.0f), n12 = __ballot(e12 <= 0.0f), p13 = __ballot(e13 >= 0.0f);
  const uint64_t n13 = __ballot(e13 <= 0.0f), p23 = __ballot(e23 >= 0.0f), n23 = __ballot(e23 <= 0.0f);
  const uint64_t m0 = (__ballot(rD.x > 0.0f) & p12 & n02 & p01) | (__ballot(rD.x < 0.0f) & n12 & p02 & n01);
  const uint64_t m1 = (__ballot(rD.y > 0.0f) & p13 & n03 & p01) | (__ballot(rD.y < 0.0f) & n13 & p03 & n01);
  const uint64_t m2 = (__ballot(rD.z > 0.0f) & p23 & n03 & p02) | (__ballot(rD.z < 0.0f) & n23 & p03 & n02);
  const uint64_t m3 = (__ballot(rD.w > 0.0f) & p23 & n13 & p12) | (__ballot(rD.w < 0.0f) & n23 & p13 & n12);
  const auto lane_bit = [](uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); };
  const bool i0 = lane_bit(m0), i1 = lane_bit(m1), i2 = lane_bit(m2), i3 = lane_bit(m3);
  const bool i01 = lane_bit(m0 | m1), i23 = lane_bit(m2 | m3);
  const uint64_t two = (m0 & m1) | (m2 & m3) | ((m0 | m1) & (m2 | m3));
  const uint64_t three = (m0 & m1 & (m2 | m3)) | (m2 & m3 & (m0 | m1));
  // a: the first inside face (0, 1 or 2), b: the last (1, 2 or 3)
  const float qa0 = (i0 ? e12 : i1 ? e13 : e23) * iz0;
  const float qa1 = -(i0 ? e02 : e03) * (i01 ? iz1 : iz2);
  const float qa2 = (i01 ? e01 : e02) * (i0 ? iz2 : iz3);
  const float qb0 = (i23 ? e23 : e13) * (i3 ? iz1 : iz0);
  const float qb1 = -(i3 ? e13 : e03) * (i23 ? iz2 : iz1);
  const float qb2 = (i3 ? e12 : i2 ? e02 : e01) * iz3;
  const float Sa = (qa0 + qa1) + qa2, Sb = (qb0 + qb1) + qb2;
  const float na = fmaf(qa0, f0, fmaf(qa1, i01 ? f1 : f2, qa2 * (i0 ? f2 : f3)));
  const float nb = fmaf(qb0, i3 ? f1 : f0, fmaf(qb1, i23 ? f2 : f1, qb2 * f3));
  const float za = Sa * (i0 ? rD.x : i1 ? rD.y : rD.z), zb = Sb * (i3 ? rD.w : i2 ? rD.z : rD.y);
  // (equal depths: face a is entry and exit, and alpha zero, as in pixel_eval)
  const bool b_in = zb > za, b_out = zb < za;
  float num_in = b_in ? nb : na, S_in = b_in ? Sb : Sa, num_out = b_out ? nb : na, S_out = b_out ? Sb : Sa;
  const int fa = i0 ? 0 : i1 ? 1 : 2, fb = i3 ? 3 : i2 ? 2 : 1;
  h.faces = (b_in ? fb : fa) | (b_out ? fb : fa) << 2;
  h.zin_inv = b_in ? zb : za;
  const uint64_t several = three | (two & __ballot(!(fabsf(za) + fabsf(zb) < INFINITY)));
  if (several && lane_bit(several)) {
    float best_in = -INFINITY, best_out = INFINITY;
    num_in = num_out = 0.0f;
    S_in = S_out = 1.0f;
    h.faces = 0;
#pragma unroll 1
    for (int F = 0; F < 4; ++F) {
      const int A = F == 3 ? 1 : 0, B = F < 2 ? 1 : 2, C = F == 0 ? 2 : 3;
      const float xa = r.px[A] - qx, ya = r.py[A] - qy, xb = r.px[B] - qx, yb = r.py[B] - qy;
      const float xc = r.px[C] - qx, yc = r.py[C] - qy;
      const float N0 = xb * yc - yb * xc, N1 = -(xa * yc - ya * xc), N2 = xa * yb - ya * xb;
      if (!face_inside(N0, N1, N2, r.rD[F])) continue;
      const float q0 = N0 * r.iz[A], q1 = N1 * r.iz[B], q2 = N2 * r.iz[C];
      const float S = (q0 + q1) + q2, num = fmaf(q0, r.f[A], fmaf(q1, r.f[B], q2 * r.f[C]));
      const float z = S * r.rD[F];
      if (z > best_in) {
        best_in = z;
        num_in = num;
        S_in = S;
        h.faces = (h.faces & 12) | F;
      }
      if (z < best_out) {
        best_out = z;
        num_out = num;
        S_out = S;
        h.faces = (h.faces & 3) | F << 2;
      }
    }
    h.zin_inv = best_in;
  }
  const float fin = num_in * rcp(S_in), fout = num_out * rcp(S_out);
  const float d = fin - fout;
  const bool pos = d > 0.0f;
  const float x = pos ? -(s * d) : 0.0f;
  h.e2 = pos ? fast_exp(s * fout) : 0.0f;
  h.alpha = pos ? -fast_expm1_neg(x) * rcp(1.0f + h.e2) : 0.0f;
  return lane_bit(two);
}

template <class Rec>
__device__ __forceinline__ void unpack_rect(const Rec& r, int& i0, int& i1, int& j0, int& j1) {
  i0 = (int)(r.rx & 0xffffu);
  i1 = (int)(r.rx >> 16);
  j0 = (int)(r.ry & 0xffffu);
  j1 = (int)(r.ry >> 16);
}

// Columns and rows per unit of a record's spans: the rectangle's width and
// height fit 16 columns and 8 strips of these (a power of two, as a shift).
__device__ __forceinline__ int span_shift(int n, int units_log2) {
  const int x = (n - 1) >> units_log2;
  return x > 0 ? 32 - __clz(x) : 0;
}

// The pixels that a record's hull may cover, as one byte per strip of rows of
// its pixel rectangle: first and last column unit (4 bits each, relative to
// i0; first = last + 1 for none).  Half of a projected tet's rectangle lies
// outside its hull, and a pixel there costs a full evaluation that can only
// find no hit.  The spans are conservative: a pixel they leave out is at
// least SPAN_MARGIN of a pixel off the hull in both directions, where the
// float cross products of the coverage test (rounding error up to 2^-20 e^2
// for a hull of extent e) cannot put it inside a face of doubled area D,
// since its distance to one of the face's edges is at least the margin times
// the face's smallest sine, which is D / e^2 or more.  A record with a thin
// face (margin |D| < 2^-18 e^3), or with coordinates too large for the
// crossings below, keeps its whole rectangle.  The evaluated pairs per 64
// entries fall from 1159 to 668 (hull alone 0.48 to 0.58 of a rectangle, spans
// 0.52 to 0.61): forward 96 to 82 us at 4 x 512^2 and 870 to 757 us at
// 8 x 1024^2, for 7 and 19 us more in the projection, which computes them.
constexpr float SPAN_MARGIN = 0.05f;

// (false if no pixel is left)
__device__ __forceinline__ bool hull_spans(const float (&px)[4], const float (&py)[4], const float (&D)[4], float ext,
                                           int i0, int i1, int j0, int j1, uint32_t (&span)[2]) {
  bool tight = ext < 65536.0f;
  const float thin = ext * ext * ext * (1.0f / (262144.0f * SPAN_MARGIN));
#pragma unroll
  for (int F = 0; F < 4; ++F) tight = tight && (D[F] == 0.0f || fabsf(D[F]) >= thin);
  span[0] = span[1] = 0xf0f0f0f0u;   // every column
  if (!tight) return true;
  constexpr int EA[6] = {0, 0, 0, 1, 1, 2}, EB[6] = {1, 2, 3, 2, 3, 3};
  float dx[6], inv[6];
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    dx[e] = px[EB[e]] - px[EA[e]];
    inv[e] = rcp(py[EB[e]] - py[EA[e]]);   // infinite for a level edge, whose parameters are then 0 and 1 or equal
  }
  const int sx = span_shift(i1 - i0 + 1, 4), sy = span_shift(j1 - j0 + 1, 3);
  const float fi0 = (float)i0, fi1 = (float)i1;
  uint32_t w[2] = {0u, 0u};
  bool any = false;
  for (int k = 0; k < 8; ++k) {
    const int ja = j0 + (k << sy), jb = min(ja + (1 << sy) - 1, j1);
    if (ja > j1) break;
    const float ya = (float)ja + (0.5f - SPAN_MARGIN), yb = (float)jb + (0.5f + SPAN_MARGIN);
    // the hull between the lines ya and yb: the part of every edge there, from
    // parameter ta to tb (both at one end of an edge that does not reach it)
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const float ta = __builtin_amdgcn_fmed3f((ya - py[EA[e]]) * inv[e], 0.0f, 1.0f);
      const float tb = __builtin_amdgcn_fmed3f((yb - py[EA[e]]) * inv[e], 0.0f, 1.0f);
      const float xa = fmaf(ta, dx[e], px[EA[e]]), xb = fmaf(tb, dx[e], px[EA[e]]);
      const bool in = ta != tb;
      lo = fminf(lo, in ? fminf(xa, xb) : INFINITY);
      hi = fmaxf(hi, in ? fmaxf(xa, xb) : -INFINITY);
    }
    const float ca = fmaxf(ceilf(lo - (0.5f + SPAN_MARGIN)), fi0), cb = fminf(floorf(hi - (0.5f - SPAN_MARGIN)), fi1);
    uint32_t b = 1u;   // none
    if (ca <= cb) b = (uint32_t)(((int)ca - i0) >> sx) | (uint32_t)(((int)cb - i0) >> sx) << 4;
    any = any || ca <= cb;
    w[k >> 2] |= b << (8 * (k & 3));
  }
  span[0] = w[0];
  span[1] = w[1];
  return any;
}

// Whether no ray of the view can blend the tet: f does not fall along any ray
// that crosses it, so d = f_prev - f_next <= 0 (or so little above that Eq. 1
// stays below alpha_min).  With g the gradient of f in camera space, f changes
// by g . (X / Z) per unit of depth at X, and over the tet g . X is f minus f's
// continuation to the camera: smallest at a vertex.  d is then at most
// max(0, -min_k g . X_k) (Zmax / Zmin - 1), plus what g, computed in floats,
// misses of the vertices' values (its residual r, once per face).
//   The evaluation of a pair rounds, and what that can add to d stands beside it:
// the two interpolated values (8 rounding units of the largest |f| each, however
// flat f is); the order and the place of the two faces, whose weights and
// depths are off by the cross products' rounding over a face's area (thin:
// hull extent^2 / least area; a ray through less than that of relative thickness
// may see the faces exchanged and d with the other sign); the projected vertices
// (reach: |pixel| / focal length), which move a tet's faces by more of its
// height the flatter it is (e^3 / det).  The units of the last two are twice and
// five times what random tets down to slivers were seen to need (none of 280 M
// pairs near a projected edge would blend in a tet left out).  Where s makes
// that matter, or thin is past 64, the tet is kept: 53.5 in 100 records of a
// 64^3 grid at s = 320 are left out, 53.9 without these terms.  NaNs compare
// false: kept.
//   Half the kept tets around a surface face away.  Most are behind it, but
// they are 19 to 22 in 100 of the pairs that were evaluated (64^3 grids with
// noise, s = 320, from 2.5 away): forward 73 to 69 us at 4 x 512^2, 684 to 635
// us at 8 x 1024^2, for 1 and 4 us of the projection; and half the entries of
// the lists (see k_tile_depth_sort).
__device__ __forceinline__ bool never_blends(const float (&X)[4], const float (&Y)[4], const float (&Z)[4],
                                             const float (&f)[4], const float (&D)[4], float ext, float reach, float s,
                                             float alpha_min) {
  float ex[3], ey[3], ez[3], df[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ex[a] = X[a + 1] - X[0];
    ey[a] = Y[a + 1] - Y[0];
    ez[a] = Z[a + 1] - Z[0];
    df[a] = f[a + 1] - f[0];
  }
  float g[3] = {0.0f, 0.0f, 0.0f}, det = 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int b = (a + 1) % 3, c = (a + 2) % 3;
    const float cx = fmaf(ey[b], ez[c], -(ez[b] * ey[c])), cy = fmaf(ez[b], ex[c], -(ex[b] * ez[c]));
    const float cz = fmaf(ex[b], ey[c], -(ey[b] * ex[c]));
    if (a == 0) det = fmaf(ex[0], cx, fmaf(ey[0], cy, ez[0] * cz));
    g[0] = fmaf(cx, df[a], g[0]);
    g[1] = fmaf(cy, df[a], g[1]);
    g[2] = fmaf(cz, df[a], g[2]);
  }
  const float id = rcp(det);
#pragma unroll
  for (int m = 0; m < 3; ++m) g[m] *= id;
  float r = 0.0f, e = 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    r = fmaxf(r, fabsf(fmaf(g[0], ex[a], fmaf(g[1], ey[a], fmaf(g[2], ez[a], -df[a])))));
    e = fmaxf(e, fmaxf(fabsf(ex[a]), fmaxf(fabsf(ey[a]), fabsf(ez[a]))));
  }
  r = fmaf((fabsf(g[0]) + fabsf(g[1]) + fabsf(g[2])) * e, 0x1p-21f, r);
  const float G0 = fmaf(g[0], X[0], fmaf(g[1], Y[0], g[2] * Z[0]));
  const float Gabs = fabsf(g[0] * X[0]) + fabsf(g[1] * Y[0]) + fabsf(g[2] * Z[0]);
  const float lo = fminf(0.0f, fminf(df[0], fminf(df[1], df[2]))), hi = fmaxf(0.0f, fmaxf(df[0], fmaxf(df[1], df[2])));
  const float zmin = fminf(fminf(Z[0], Z[1]), fminf(Z[2], Z[3])), zmax = fmaxf(fmaxf(Z[0], Z[1]), fmaxf(Z[2], Z[3]));
  const float zr = zmax * rcp(zmin);
  const float fall = fmaxf(0.0f, fmaf(Gabs, 0x1p-20f, r - (G0 + lo)));   // of f, per relative depth, at most
  float area = INFINITY, top = 0.0f;
#pragma unroll
  for (int F = 0; F < 4; ++F) {
    area = fminf(area, D[F] != 0.0f ? fabsf(D[F]) : INFINITY);   // (a face without area is never hit)
    top = fmaxf(top, fabsf(f[F]));
  }
  const float thin = ext * ext * rcp(area);
  const float order = (fabsf(G0) + fmaxf(hi, -lo)) * zr * fmaf(thin, 0x1p-23f, 0x1p-20f);
  const float moved = (fabsf(g[0]) + fabsf(g[1]) + fabsf(g[2])) * zmax * reach * (e * e * e) * fabsf(id) * 0x1p-25f;
  const float bound = fmaf(fall, zr - 1.0f + 0x1p-20f, 2.0f * r + fmaf(top, 0x1p-20f, order + moved));
  bool ok = alpha_min > 0.0f && zmin > 0.0f && s >= 0.0f && s * bound <= 0.95f * alpha_min;
#pragma unroll
  for (int F = 0; F < 4; ++F) ok = ok && (D[F] == 0.0f || fabsf(D[F]) * 64.0f >= ext * ext);
  return ok;
}

// Dispatch-order bucket of a list length: 0 for an empty list, then four
// buckets per power of two.
__device__ __forceinline__ int len_bucket(uint32_t len) {
  if (len == 0) return 0;
  const int b = 31 - __clz(len);  // floor(log2 len)
  const int sub = b >= 2 ? (int)((len >> (b - 2)) & 3u) : (b == 1 ? (int)((len & 1u) << 1) : 0);
  return 1 + 4 * b + sub;
}

// ---------------------------------------------------------------------------
// Reverse mode of one (pixel, record) pair: the pixel's blend weight w and
// dL/dalpha are chained to the record's 23 screen-space parameters.
// ---------------------------------------------------------------------------
// dL/dalpha of a pair chained through Eq. 1 (stable form) to its entry and
// exit SDF values: alpha = A / B, A = -expm1(-s d), B = 1 + exp(s f_next),
// d = f_prev - f_next; e2 = exp(s f_next).  Zero when alpha is zero (the
// max(., 0) of Eq. 1).
__device__ __forceinline__ void eq1_chain(float da, float alpha, float e2, float s, float& dd, float& dfn) {
  const bool on = da != 0.0f && alpha > 0.0f;
  const float B = 1.0f + e2;
  const float invB = rcp(B);
  const float e1p1 = 1.0f - alpha * B;                   // exp(-s d) = 1 + expm1(-s d)
  const float dA = da * invB;
  const float dB = -da * alpha * invB;
  const float ddv = dA * s * e1p1;                       // d/df_prev
  dd = on ? ddv : 0.0f;
  dfn = on ? dB * s * e2 - ddv : 0.0f;                   // d/df_next
}

// g <- the pair's gradient with respect to the record's 23 screen-space
// parameters, given the blend weight w = T alpha (colour, depth and normal
// enter linearly), dL/df_prev = dd and dL/df_next = dfn, and the entry/exit
// faces fs = fe | fx << 2.  Without branches: all four faces are chained, a
// face whose weight is zero contributes exactly zero (its 1/S is taken as 0),
// so a lane with w = dd = dfn = 0 returns zeros.
//   Face F: f = sum N_k w_k f_k / S, S = sum N_k w_k, N_k = +- e_ij of its
// other two vertices.  With U_F = dL/df / S and d_kF = (f_k - f) U_F:
//   dL/df_k = w_k sum_F N_kF U_F, dL/dw_k = sum_F N_kF d_kF,
//   dL/de_ij = sum over the two faces with edge ij of +- w_k d_kF,
// and the six edge cross products e_ij = cross(P_i - p, P_j - p) carry on to
// the vertices together (24 products for the four faces, not 24 for each).
__device__ __forceinline__ void pair_grad_all(const ViewRec& R, float qx, float qy, const float (&gr)[8], float dd,
                                              float dfn, float w, int fs, float (&g)[TGRAD_STRIDE - 1]) {
  g[G_C + 0] = w * gr[0];
  g[G_C + 1] = w * gr[1];
  g[G_C + 2] = w * gr[2];
  g[G_ZT] = w * gr[4];
  g[G_N + 0] = w * gr[5];
  g[G_N + 1] = w * gr[6];
  g[G_N + 2] = w * gr[7];
  const int fe = fs & 3, fx = fs >> 2;
  float ax[4], ay[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ax[k] = R.px[k] - qx;
    ay[k] = R.py[k] - qy;
  }
  constexpr int EI[6] = {0, 0, 0, 1, 1, 2}, EJ[6] = {1, 2, 3, 2, 3, 3};
  float e[6], de[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    e[q] = ax[EI[q]] * ay[EJ[q]] - ay[EI[q]] * ax[EJ[q]];
    de[q] = 0.0f;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) g[G_F + k] = g[G_IZ + k] = 0.0f;
#pragma unroll
  for (int F = 0; F < 4; ++F) {
    const int v[3] = {face_vertex(F, 0), face_vertex(F, 1), face_vertex(F, 2)};
    // N_0 = e_12, N_1 = -e_02, N_2 = e_01 of the face's vertices in order
    // (their indices ascend, so each is one of the six e)
    const int q12 = v[1] == 1 ? (v[2] == 2 ? 3 : 4) : 5, q02 = v[0] == 0 ? (v[2] == 2 ? 1 : 2) : 4,
              q01 = v[0] == 0 ? (v[1] == 1 ? 0 : 1) : 3;
    const int q[3] = {q12, q02, q01};
    const float N[3] = {e[q12], -e[q02], e[q01]};
    const float wF = (fe == F ? dd : 0.0f) + (fx == F ? dfn : 0.0f);
    const float qa = N[0] * R.iz[v[0]], qb = N[1] * R.iz[v[1]], qc = N[2] * R.iz[v[2]];
    const float S = (qa + qb) + qc;
    const float invS = wF != 0.0f ? rcp(S) : 0.0f;
    const float f = fmaf(qa, R.f[v[0]], fmaf(qb, R.f[v[1]], qc * R.f[v[2]])) * invS;
    const float U = wF * invS;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float dk = (R.f[v[k]] - f) * U;
      g[G_F + v[k]] = fmaf(N[k], U, g[G_F + v[k]]);
      g[G_IZ + v[k]] = fmaf(N[k], dk, g[G_IZ + v[k]]);
      de[q[k]] = fmaf(k == 1 ? -R.iz[v[k]] : R.iz[v[k]], dk, de[q[k]]);
    }
  }
  float gx[4] = {0.0f, 0.0f, 0.0f, 0.0f}, gy[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const int i = EI[q], j = EJ[q];
    gx[i] = fmaf(de[q], ay[j], gx[i]);
    gy[i] = fmaf(-de[q], ax[j], gy[i]);
    gx[j] = fmaf(-de[q], ay[i], gx[j]);
    gy[j] = fmaf(de[q], ax[i], gy[j]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    g[G_F + k] *= R.iz[k];
    g[G_PX + k] = gx[k];
    g[G_PY + k] = gy[k];
  }
}

// ---------------------------------------------------------------------------
// Wave-wide scans and exchanges on the data-parallel primitives (DPP) and the
// lane swaps, not on LDS permutes: a step of a scan is one instruction of some
// eight cycles against more than a hundred for a permute and its wait, and
// the one-wave phases of the compositing kernels are chains of such steps.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}

// inclusive sum over the lanes at or before this one (every lane active)
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t x) {
  x += dpp_u32<0x111>(x);   // row_shr 1, 2, 4, 8 (0 past the row's start)
  x += dpp_u32<0x112>(x);
  x += dpp_u32<0x114>(x);
  x += dpp_u32<0x118>(x);
  // a row's last lane to the next row (rows 1 and 3), then lane 31 to rows 2 and 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);
  return x;
}

// The same steps with max: lane 63 holds the wave's largest value.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, dpp_u32<0x111>(x));
  x = max(x, dpp_u32<0x112>(x));
  x = max(x, dpp_u32<0x114>(x));
  x = max(x, dpp_u32<0x118>(x));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));
  return x;
}

// ---------------------------------------------------------------------------
// Transpose of the 64 x 64 bit matrix whose row r is lane r's word: bit c of
// lane r becomes bit r of lane c.  Six butterfly steps; at step j, lanes r
// and r ^ j exchange the j-wide column blocks that the transpose swaps.
// ---------------------------------------------------------------------------
// a step below a byte: w's partner word y, K the columns that stay in the
// lane whose bit j is clear
template <int J, uint32_t K>
__device__ __forceinline__ uint32_t transpose_step(uint32_t w, uint32_t y, bool upper) {
  return upper ? (w & ~K) | ((y & ~K) >> J) : (w & K) | ((y & K) << J);
}
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x) {
  const unsigned lane = __lane_id();
  // 32: the lower lanes' high words against the upper lanes' low words
  const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)(x >> 32), false, false);
  uint32_t w[2] = {h[0], h[1]};
  const bool b4 = lane & 16u, b3 = lane & 8u, b2 = lane & 4u, b1 = lane & 2u, b0 = lane & 1u;
  // byte selectors of (partner, own): own bytes are 0-3, the partner's 4-7
  const uint32_t s16 = b4 ? 0x03020706u : 0x05040100u, s8 = b3 ? 0x03070105u : 0x06020400u;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const auto p = __builtin_amdgcn_permlane16_swap(w[i], w[i], false, false);
    w[i] = __builtin_amdgcn_perm(b4 ? p[0] : p[1], w[i], s16);
    w[i] = __builtin_amdgcn_perm(dpp_u32<0x128>(w[i]), w[i], s8);                                   // lane ^ 8
    w[i] = transpose_step<4, 0x0f0f0f0fu>(w[i], dpp_u32<0x1B>(dpp_u32<0x141>(w[i])), b2);           // lane ^ 4
    w[i] = transpose_step<2, 0x33333333u>(w[i], dpp_u32<0x4E>(w[i]), b1);                           // lane ^ 2
    w[i] = transpose_step<1, 0x55555555u>(w[i], dpp_u32<0xB1>(w[i]), b0);                           // lane ^ 1
  }
  return ((uint64_t)w[1] << 32) | w[0];
}

// ---------------------------------------------------------------------------
// wave-wide transposed sum of 32 per-lane values (gfx950 permlane swaps and
// DPP): afterwards lane L holds the sum over all 64 lanes of v[L >> 1].
// Each step halves the values per lane while pairing lanes across a 32-,
// 16-, 8-, 4-, 2- and 1-lane distance: 16+8 swaps, 4+2+1 DPP-fused adds.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}

__device__ __forceinline__ float wave_transpose_sum32(const float (&v)[32]) {
  float u[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[k]), __float_as_uint(v[k + 16]), false, false);
    u[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  float w[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u[k]), __float_as_uint(u[k + 8]), false, false);
    w[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const unsigned lane = __lane_id();
  const bool b3 = lane & 8u, b2 = lane & 4u, b1 = lane & 2u;
  float x[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float send = b3 ? w[k] : w[k + 4];
    const float keep = b3 ? w[k + 4] : w[k];
    x[k] = keep + dpp<0x128>(send);   // row_ror:8  (lane j <-> j ^ 8)
  }
  float y[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float send = b2 ? x[k] : x[k + 2];
    const float keep = b2 ? x[k + 2] : x[k];
    y[k] = keep + dpp<0x141>(send);   // row_half_mirror (j <-> 7 - j)
  }
  const float send = b1 ? y[0] : y[1];
  const float keep = b1 ? y[1] : y[0];
  float z = keep + dpp<0x4E>(send);   // quad_perm [2,3,0,1]
  z = z + dpp<0xB1>(z);               // quad_perm [1,0,3,2]
  return z;
}

}  // namespace ts
