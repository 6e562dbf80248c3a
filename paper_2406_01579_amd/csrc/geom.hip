// Geometry regularisers of Sec. 4.2 on the deformable tet grid, for gfx950.
//
//  * eikonal term  L_eik = sum_k (|g_k| - 1)^2 over the tets, g_k the SDF
//    gradient inside tet k (App. A.3, as the 3x3 edge system g = E^-1 df);
//  * normal-consistency term  L_nc = sum_e (1 - cos(m_a, m_b)) over the
//    unique edges (a, b), m_v = sum of the unit normals g_k/|g_k| of the tets
//    around vertex v.
//
// Three grid-stride passes: per tet (g, the eikonal partial sums, scatter of
// n_k into m), per edge (the consistency term and dL/dm), per tet again
// (g recomputed; dL/dg from both terms chained to the four SDF values and
// vertex positions).  1 - cos is evaluated as |u_a - u_b|^2 / 2 on the unit
// vectors, which has no cancellation for nearly parallel normals.  Loss
// partial sums are per block in a fixed order and summed in double by one
// block, so the losses do not depend on scheduling except through the float
// atomics that build m.
//
// The unique-edge list is built once per topology: the (a < b) pairs of every
// tet, freed of most repeats in LDS, are binned by a, and each vertex's bucket
// is sorted and freed of the rest.
//
// Marching Tetrahedra (the mesh extraction of Sec. 4.1): a mark/scan/write
// sequence over the edges places one surface vertex on every edge whose ends
// differ in the inside test (f < 0), numbered in edge order; one over the tets
// writes one triangle (one or three inside vertices) or two (two inside) in
// tet order, looking the crossed edges up in the sorted edge list.  The
// winding is fixed by a 16-entry case table built at compile time (outward
// normals, flipped for negatively oriented tets).
#include <algorithm>

#include "ts_device.h"

namespace ts {
namespace {

constexpr int RT = 256;
constexpr int RBLOCKS = 1024;
constexpr int EDGE_ITEMS = 8;
constexpr int EDGE_TILE = RT * EDGE_ITEMS;

__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* lds /*[RT/64]*/, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds[wave] = x;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < RT / 64; ++w) {
    const uint32_t t = lds[w];
    if (w < wave) base += t;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + x - v;
}

__device__ __forceinline__ float block_sum(float v, float* lds /*[RT/64]*/) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.0f;
#pragma unroll
  for (int w = 0; w < RT / 64; ++w) s += lds[w];
  __syncthreads();
  return s;
}

__device__ __forceinline__ bool load_tet(const int32_t* tets, uint32_t k, int32_t V, int32_t (&v)[4]) {
  const int4 t = reinterpret_cast<const int4*>(tets)[k];
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  return (uint32_t)t.x < (uint32_t)V && (uint32_t)t.y < (uint32_t)V && (uint32_t)t.z < (uint32_t)V &&
         (uint32_t)t.w < (uint32_t)V;
}

// the (a < b) vertex pair of local edge e of tet k; (V, V) for a tet with an
// index outside [0, V)
__device__ __forceinline__ void pair_of(const int32_t* tets, uint32_t i, int32_t V, uint32_t& a, uint32_t& b) {
  const uint32_t k = i / 6, e = i - 6 * k;
  int32_t v[4];
  if (!load_tet(tets, k, V, v)) {
    a = b = (uint32_t)V;
    return;
  }
  // local pairs (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
  const int32_t p = e < 3 ? v[0] : (e < 5 ? v[1] : v[2]);
  const int32_t q = e == 0 ? v[1] : (e == 1 || e == 3) ? v[2] : v[3];
  a = (uint32_t)min(p, q);
  b = (uint32_t)max(p, q);
}

// SDF gradient of the linear interpolant over the tet: E g = df with rows
// e_a = x_{a+1} - x_0, df_a = f_{a+1} - f_0; cr[a] is column a of det * E^-1
struct TetGrad {
  float x[4][3], f[4];
  float cr[3][3];
  float det;
  float g[3];
};

__device__ __forceinline__ void tet_grad(const float* verts, const float* sdf, const int32_t (&v)[4], TetGrad& T) {
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int m = 0; m < 3; ++m) T.x[a][m] = verts[3 * (size_t)v[a] + m];
    T.f[a] = sdf[v[a]];
  }
  float e[3][3], df[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int m = 0; m < 3; ++m) e[a][m] = T.x[a + 1][m] - T.x[0][m];
    df[a] = T.f[a + 1] - T.f[0];
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int b = (a + 1) % 3, c = (a + 2) % 3;
    T.cr[a][0] = e[b][1] * e[c][2] - e[b][2] * e[c][1];
    T.cr[a][1] = e[b][2] * e[c][0] - e[b][0] * e[c][2];
    T.cr[a][2] = e[b][0] * e[c][1] - e[b][1] * e[c][0];
  }
  T.det = e[0][0] * T.cr[0][0] + e[0][1] * T.cr[0][1] + e[0][2] * T.cr[0][2];
#pragma unroll
  for (int m = 0; m < 3; ++m)
    T.g[m] = T.det != 0.0f ? (T.cr[0][m] * df[0] + T.cr[1][m] * df[1] + T.cr[2][m] * df[2]) / T.det : 0.0f;
}

// ---------------------------------------------------------------------------
// unique edges
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(RT) void k_edge_keys_b(const int32_t* tets, uint32_t n, int32_t V, uint32_t* keyb,
                                                    uint32_t* n_dev) {
  if (blockIdx.x == 0 && threadIdx.x == 0) n_dev[0] = n;
  for (uint32_t i = blockIdx.x * RT + threadIdx.x; i < n; i += gridDim.x * RT) {
    uint32_t a, b;
    pair_of(tets, i, V, a, b);
    keyb[i] = b;
  }
}

__global__ __launch_bounds__(RT) void k_edge_keys_a(const int32_t* tets, uint32_t n, int32_t V, const uint32_t* idx,
                                                    uint32_t* keya) {
  for (uint32_t j = blockIdx.x * RT + threadIdx.x; j < n; j += gridDim.x * RT) {
    uint32_t a, b;
    pair_of(tets, idx[j], V, a, b);
    keya[j] = a;
  }
}

// flag = first of its run of equal pairs, and a real edge
__device__ __forceinline__ uint32_t edge_flags(const int32_t* tets, uint32_t n, int32_t V, const uint32_t* idx,
                                               uint32_t j0, uint32_t (&ab)[EDGE_ITEMS][2]) {
  uint32_t bits = 0;
  uint32_t pa = 0xffffffffu, pb = 0xffffffffu;
  if (j0 > 0 && j0 - 1 < n) pair_of(tets, idx[j0 - 1], V, pa, pb);
#pragma unroll
  for (int t = 0; t < EDGE_ITEMS; ++t) {
    const uint32_t j = j0 + t;
    uint32_t a = (uint32_t)V, b = (uint32_t)V;
    if (j < n) pair_of(tets, idx[j], V, a, b);
    ab[t][0] = a;
    ab[t][1] = b;
    if (j < n && a < (uint32_t)V && (a != pa || b != pb)) bits |= 1u << t;
    pa = a;
    pb = b;
  }
  return bits;
}

__global__ __launch_bounds__(RT) void k_edge_count(const int32_t* tets, uint32_t n, int32_t V, const uint32_t* idx,
                                                   uint32_t* bsum) {
  __shared__ uint32_t lds[RT / 64];
  uint32_t ab[EDGE_ITEMS][2];
  const uint32_t j0 = blockIdx.x * EDGE_TILE + threadIdx.x * EDGE_ITEMS;
  const uint32_t c = __popc(edge_flags(tets, n, V, idx, j0, ab));
  uint32_t tot;
  block_scan_excl(c, lds, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// one block of 1024: exclusive scan of nb block sums in place, and their total
__device__ __forceinline__ void spine_1024(uint32_t* bsum, uint32_t nb, int32_t* n_edges) {
  __shared__ uint32_t part[16];
  const uint32_t t = threadIdx.x;
  const uint32_t per = (nb + 1023) / 1024;
  const uint32_t lo = min(nb, t * per), hi = min(nb, (t + 1) * per);
  uint32_t s = 0;
  for (uint32_t i = lo; i < hi; ++i) s += bsum[i];
  const int lane = t & 63, wave = t >> 6;
  uint32_t x = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) part[wave] = x;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) base += part[w];
    tot += part[w];
  }
  uint32_t run = base + x - s;
  for (uint32_t i = lo; i < hi; ++i) {
    const uint32_t c = bsum[i];
    bsum[i] = run;
    run += c;
  }
  if (t == 0) n_edges[0] = (int32_t)tot;
}

__global__ __launch_bounds__(1024) void k_edge_spine(uint32_t* bsum, uint32_t nb, int32_t* n_edges) {
  spine_1024(bsum, nb, n_edges);
}

__global__ __launch_bounds__(RT) void k_edge_write(const int32_t* tets, uint32_t n, int32_t V, const uint32_t* idx,
                                                   const uint32_t* bsum, int32_t* edges) {
  __shared__ uint32_t lds[RT / 64];
  uint32_t ab[EDGE_ITEMS][2];
  const uint32_t j0 = blockIdx.x * EDGE_TILE + threadIdx.x * EDGE_ITEMS;
  const uint32_t bits = edge_flags(tets, n, V, idx, j0, ab);
  uint32_t tot;
  uint32_t o = bsum[blockIdx.x] + block_scan_excl(__popc(bits), lds, &tot);
#pragma unroll
  for (int t = 0; t < EDGE_ITEMS; ++t) {
    if (bits & (1u << t)) {
      reinterpret_cast<int2*>(edges)[o] = make_int2((int32_t)ab[t][0], (int32_t)ab[t][1]);
      ++o;
    }
  }
}

// Per-block sums over vertices.  Every vertex of a grid belongs to some two
// dozen tets and a dozen edges, and neighbouring tets and edges are
// neighbours in memory: a block takes a contiguous chunk of them and adds
// into LDS first.  The LDS sums are kept in groups of 16 consecutive
// vertices, found by hashing the group number (open addressing, bounded
// probe), so that a group's sums go out as one contiguous run: float atomics
// to scattered addresses are what bounds these passes (measured: 21 G/s, one
// address per lane and request; a chunk of 2048 tets of a cube grid has 8192
// corners but some 780 vertices, in runs of 16).  A vertex whose group finds
// no place is added to device memory directly.  The sums are doubles: an LDS
// add of a double takes 9 cycles per wave and CU on this chip, one of a float
// 194 (64 distinct addresses, measured), and the sum is rounded only once.
// 64^3 grid, 1.57 M tets: the tet pass 888 us with scattered atomics, 123 us
// with float sums in LDS, 27 us so; its backward 1095, 161 and 32 us; the edge
// pass with gradients 204, 83 and 22 us.
constexpr int VS_RUN = 16;
constexpr int VS_GROUPS = 128;
constexpr int VS_PROBES = 8;
constexpr int VS_T = 512;       // threads of a block that sums over vertices
static_assert(VS_GROUPS == 1 << 7, "the group hash keeps 7 bits");

template <int C>
struct VertexSums {
  double val[C][VS_GROUPS * VS_RUN];
  uint32_t key[VS_GROUPS];               // group number + 1; 0: free
};

template <int C>
__device__ __forceinline__ void vs_clear(VertexSums<C>& S) {
  for (int i = threadIdx.x; i < VS_GROUPS; i += VS_T) S.key[i] = 0u;
  for (int i = threadIdx.x; i < C * VS_GROUPS * VS_RUN; i += VS_T) (&S.val[0][0])[i] = 0.0;
}

// the place of vertex v's sums under the group keys, -1 if its group finds none
__device__ __forceinline__ int group_place(uint32_t* key, uint32_t v) {
  const uint32_t g = v / VS_RUN + 1u;
  uint32_t h = (g * 2654435761u) >> 25;
#pragma unroll 1
  for (int p = 0; p < VS_PROBES; ++p) {
    uint32_t k = key[h];
    if (k == 0u) {
      k = atomicCAS(&key[h], 0u, g);
      if (k == 0u) k = g;
    }
    if (k == g) return (int)(h * VS_RUN + v % VS_RUN);
    h = (h + 1u) & (VS_GROUPS - 1u);
  }
  return -1;
}

template <int C>
__device__ __forceinline__ int vs_place(VertexSums<C>& S, uint32_t v) {
  return group_place(S.key, v);
}

// component c of vertex v's sum, N components per vertex in out
template <int C, int N>
__device__ __forceinline__ void vs_add(VertexSums<C>& S, int place, int c, float x, float* out, int32_t v, int oc) {
  if (place >= 0) unsafeAtomicAdd(&S.val[c][place], (double)x);
  else unsafeAtomicAdd(&out[N * (size_t)v + oc], x);
}

// components [c0, c0 + N) of the sums into out[N v + c], the threads of a run
// at consecutive addresses
template <int C, int N>
__device__ __forceinline__ void vs_flush(const VertexSums<C>& S, int c0, float* __restrict__ out) {
  for (int q = threadIdx.x; q < VS_GROUPS * VS_RUN * N; q += VS_T) {
    const int h = q / (VS_RUN * N), r = q - h * (VS_RUN * N);
    const uint32_t g = S.key[h];
    if (g == 0u) continue;
    const float x = (float)S.val[c0 + r % N][h * VS_RUN + r / N];
    if (x != 0.0f) unsafeAtomicAdd(&out[(size_t)(g - 1u) * (VS_RUN * N) + r], x);
  }
}

// A block's next chunk of `chunk` consecutive items out of n: chunks are dealt
// to blocks so that the blocks of one XCD (every eighth block) take
// neighbouring chunks, whose vertices then stay in that XCD's L2.
__device__ __forceinline__ uint32_t xcd_chunk(uint32_t j, uint32_t nchunks) {
  const uint32_t per = (nchunks + 7u) / 8u;
  return (j & 7u) * per + (j >> 3);   // j < 8 per; may be >= nchunks
}

// A thread's item of a round of VS_T consecutive ones: the lanes of a wave
// are VS_T / 64 items apart, so that they rarely share a vertex (the tets of
// one cell all share two; LDS adds to one address wait for each other).
__device__ __forceinline__ uint32_t vs_item() {
  return (threadIdx.x & 63u) * (VS_T / 64) + (threadIdx.x >> 6);
}

// ---------------------------------------------------------------------------
// unique edges, binned by their lower vertex.  A chunk of tets puts its pairs
// into an LDS set first (neighbouring tets share most of their edges: the
// 3072 pairs of 512 tets of a cube grid are some 1,400 different ones), and
// each different pair takes a rank among its lower vertex's pairs, from LDS
// counters whose totals go to the vertices' counters in runs of 16.  The
// counts' scan gives every vertex a bucket, the pairs' upper vertices are
// placed there, and each bucket is sorted and freed of the repeats that other
// chunks brought.  The sort of all 6 K pairs by both vertices, which this
// replaces where mesh_edges_binned_fits says so, read and wrote them six times.
//   A bucket of up to EU_SMALL entries (some 13 on a cube grid) is sorted by
// comparison counts, several buckets at a time; one of up to EU_CAP by a bitonic
// network in LDS; a longer one (a vertex that thousands of tets share) goes to
// k_edge_long.  A pair that finds no slot in the set, or whose vertex finds no
// place, goes out on its own; in tets of no order most pairs do.
// 64^3 grid, 1.57 M tets: 787 us with the sort, 221 us so; its tets and vertices
// in random order 1161 and 950 us; a 96^3 grid with every boundary face joined
// to one point (a bucket of thousands) 3434 and 786 us.  Bound by k_edge_bin's
// LDS set (101 us) and, without order, by an atomic per pair.  (Buckets past LDS
// sorted by one block's merges instead: 13.5 ms for that point.)  What the sort
// would still do faster is random tets that all share one vertex: 100,000 on
// 80,000 vertices 132 and 213 us, 500,000 on 400,000 392 and 759 us, a block's pass
// over a bucket.
// ---------------------------------------------------------------------------
constexpr int EB_T = 512;             // threads
constexpr uint32_t EB_CHUNK = 512;    // tets per chunk
constexpr uint32_t EB_SET = 2048;     // slots of the pair set
constexpr int EB_PROBES = 32;
constexpr uint64_t EB_FREE = ~0ull;
constexpr uint32_t EB_GONE = ~0u;     // a slot whose pair went out on its own

struct PairSet {
  unsigned long long pair[EB_SET];                   // a << 32 | b
  uint32_t where[EB_SET];                            // vertex place << 16 | rank among the chunk's pairs of a
  uint32_t vkey[VS_GROUPS];                          // groups of 16 lower vertices, as in VertexSums
  uint32_t vcnt[VS_GROUPS * VS_RUN];                 // pairs per vertex, then the first one's rank
  uint32_t nitem, base;
};

// pair e of a tet, its vertices in order: (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
__device__ __forceinline__ uint32_t pair_low(const int32_t (&v)[4], int e) {
  return (uint32_t)min(v[e < 3 ? 0 : (e < 5 ? 1 : 2)], v[e == 0 ? 1 : (e == 1 || e == 3) ? 2 : 3]);
}
__device__ __forceinline__ uint32_t pair_high(const int32_t (&v)[4], int e) {
  return (uint32_t)max(v[e < 3 ? 0 : (e < 5 ? 1 : 2)], v[e == 0 ? 1 : (e == 1 || e == 3) ? 2 : 3]);
}

// n_item: the list's pairs, and behind them the count of long buckets
__global__ __launch_bounds__(RT) void k_edge_clear(uint32_t* cnt, uint32_t n, uint32_t* n_item) {
  if (blockIdx.x == 0 && threadIdx.x < 2) n_item[threadIdx.x] = 0u;
  for (uint32_t i = blockIdx.x * RT + threadIdx.x; i < n; i += gridDim.x * RT) cnt[i] = 0u;
}

// cnt[V + 1]: pairs per lower vertex (cleared); n_item: pairs listed (cleared)
__global__ __launch_bounds__(EB_T) void k_edge_bin(const int32_t* tets, uint32_t K, int32_t V, uint32_t* cnt,
                                                   uint32_t* n_item, uint32_t* la, uint32_t* lb, uint32_t* lr) {
  static_assert(EB_CHUNK == EB_T && EB_T == VS_T, "a tet per thread");
  __shared__ PairSet S;
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t nchunks = (K + EB_CHUNK - 1u) / EB_CHUNK, nj = (nchunks + 7u) / 8u * 8u;
  for (uint32_t j = blockIdx.x; j < nj; j += gridDim.x) {
    const uint32_t ch = xcd_chunk(j, nchunks);
    if (ch >= nchunks) continue;
    for (uint32_t i = t; i < EB_SET; i += EB_T) S.pair[i] = EB_FREE;
    for (uint32_t i = t; i < VS_GROUPS; i += EB_T) S.vkey[i] = 0u;
    for (uint32_t i = t; i < VS_GROUPS * VS_RUN; i += EB_T) S.vcnt[i] = 0u;
    if (t == 0u) S.nitem = 0u;
    __syncthreads();
    const uint32_t k = ch * EB_CHUNK + vs_item();
    int32_t v[4] = {0, 0, 0, 0};
    const bool tet_ok = k < min(K, (ch + 1u) * EB_CHUNK) && load_tet(tets, k, V, v);
    uint32_t own = 0u;   // bit e: pair e goes out on its own, with ow[e] its where (EB_GONE: no vertex place)
    uint32_t ow[6] = {EB_GONE, EB_GONE, EB_GONE, EB_GONE, EB_GONE, EB_GONE};
    if (tet_ok) {
#pragma unroll
      for (int e = 0; e < 6; ++e) {
        const uint32_t a = pair_low(v, e), b = pair_high(v, e);
        const uint64_t key = (uint64_t)a << 32 | b;
        uint32_t h = (a * 2654435761u ^ b * 2246822519u) >> 21;   // 11 bits: EB_SET
        bool mine = true;
        uint32_t slot = EB_SET;
#pragma unroll 1
        for (int pr = 0; pr < EB_PROBES; ++pr) {
          unsigned long long old = S.pair[h];
          if (old == EB_FREE) {
            old = atomicCAS(&S.pair[h], EB_FREE, key);
            if (old == EB_FREE) {
              slot = h;
              break;
            }
          }
          if (old == key) {
            mine = false;
            break;
          }
          h = (h + 1u) & (EB_SET - 1u);
        }
        if (!mine) continue;
        const int place = group_place(S.vkey, a);
        const uint32_t where = place >= 0 ? (uint32_t)place << 16 | atomicAdd(&S.vcnt[place], 1u) : EB_GONE;
        if (slot < EB_SET) S.where[slot] = where;
        if (slot == EB_SET || place < 0) {
          own |= 1u << e;
          ow[e] = where;
        }
      }
    }
    __syncthreads();
    // the vertices' counters, a group's 16 at consecutive addresses
    {
      constexpr int NV = VS_GROUPS * VS_RUN / EB_T;   // a thread's atomics in flight together
      uint32_t c[NV];
#pragma unroll
      for (int i = 0; i < NV; ++i) c[i] = S.vcnt[t + EB_T * i];
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const uint32_t q = t + EB_T * i;
        if (c[i] != 0u) c[i] = atomicAdd(&cnt[(S.vkey[q / VS_RUN] - 1u) * VS_RUN + q % VS_RUN], c[i]);
      }
#pragma unroll
      for (int i = 0; i < NV; ++i) S.vcnt[t + EB_T * i] = c[i];
    }
    // and those of the vertices without a place, a pair each, but the lanes that
    // share the first one's vertex together (a vertex of very many tets)
    uint32_t orank[6];
    uint64_t same[6];
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const bool gone = ((own >> e) & 1u) && ow[e] == EB_GONE;
      const uint64_t m = __ballot(gone);
      same[e] = 0ull;
      if (m == 0ull) continue;
      const int lead = __ffsll((unsigned long long)m) - 1;
      const uint32_t a = pair_low(v, e), a0 = (uint32_t)__builtin_amdgcn_readlane((int)a, lead);
      same[e] = __ballot(gone && a == a0);
      if (gone && (a != a0 || (int)lane == lead)) orank[e] = atomicAdd(&cnt[a], a == a0 ? (uint32_t)__popcll(same[e]) : 1u);
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      if (same[e] == 0ull) continue;
      const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)orank[e], __ffsll((unsigned long long)same[e]) - 1);
      if ((same[e] >> lane) & 1ull) orank[e] = r0 + (uint32_t)__popcll(same[e] & ((1ull << lane) - 1ull));
    }
    // the chunk's pairs into consecutive places of the list
    uint32_t at_[EB_SET / EB_T];
#pragma unroll
    for (uint32_t i = 0; i < EB_SET / EB_T; ++i) {
      const uint32_t s = t + i * EB_T;
      const bool out = S.pair[s] != EB_FREE && S.where[s] != EB_GONE;
      const uint64_t m = __ballot(out);
      uint32_t w = 0u;
      if (lane == 0u && m) w = atomicAdd(&S.nitem, (uint32_t)__popcll(m));
      w = (uint32_t)__builtin_amdgcn_readfirstlane((int)w);
      at_[i] = out ? w + (uint32_t)__popcll(m & ((1ull << lane) - 1ull)) : EB_GONE;
    }
    uint32_t oat = 0u;
    if (__ballot(own != 0u)) {
      const uint32_t c = (uint32_t)__popc(own), x = wave_scan_add(c);
      uint32_t w = 0u;
      if (lane == 63u) w = atomicAdd(&S.nitem, x);
      oat = (uint32_t)__builtin_amdgcn_readlane((int)w, 63) + x - c;
    }
    __syncthreads();
    if (t == 0u) S.base = atomicAdd(n_item, S.nitem);
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < EB_SET / EB_T; ++i) {
      if (at_[i] == EB_GONE) continue;
      const uint32_t s = t + i * EB_T, o = S.base + at_[i], w = S.where[s];
      la[o] = (uint32_t)(S.pair[s] >> 32);
      lb[o] = (uint32_t)S.pair[s];
      lr[o] = S.vcnt[w >> 16] + (w & 0xffffu);
    }
    if (own != 0u) {
      uint32_t o = S.base + oat;
#pragma unroll
      for (int e = 0; e < 6; ++e) {
        if (!((own >> e) & 1u)) continue;
        la[o] = pair_low(v, e);
        lb[o] = pair_high(v, e);
        lr[o] = ow[e] != EB_GONE ? S.vcnt[ow[e] >> 16] + (ow[e] & 0xffffu) : orank[e];
        ++o;
      }
    }
    __syncthreads();
  }
}

// sums of 2048 counts each, for the spine
constexpr uint32_t EB_SCAN = 2048;
__global__ __launch_bounds__(RT) void k_cnt_sum(const uint32_t* cnt, uint32_t n, uint32_t* bsum) {
  __shared__ uint32_t lds[RT / 64];
  const uint32_t i0 = blockIdx.x * EB_SCAN + threadIdx.x;
  uint32_t s = 0;
#pragma unroll
  for (uint32_t i = 0; i < EB_SCAN; i += RT) s += i0 + i < n ? cnt[i0 + i] : 0u;
  uint32_t tot;
  block_scan_excl(s, lds, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// in place: counts to bucket starts (the blocks' first from the spine)
__global__ __launch_bounds__(RT) void k_cnt_starts(uint32_t* cnt, uint32_t n, const uint32_t* bsum) {
  __shared__ uint32_t lds[RT / 64];
  constexpr uint32_t PER = EB_SCAN / RT;
  const uint32_t i0 = blockIdx.x * EB_SCAN + threadIdx.x * PER;
  uint32_t c[PER], s = 0;
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) {
    c[i] = i0 + i < n ? cnt[i0 + i] : 0u;
    s += c[i];
  }
  uint32_t tot;
  uint32_t run = bsum[blockIdx.x] + block_scan_excl(s, lds, &tot);
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) {
    if (i0 + i < n) cnt[i0 + i] = run;
    run += c[i];
  }
}

__global__ __launch_bounds__(RT) void k_edge_place(const uint32_t* start, const uint32_t* n_item, const uint32_t* la,
                                                   const uint32_t* lb, const uint32_t* lr, uint32_t* bucket) {
  const uint32_t n = *n_item;
  for (uint32_t i = blockIdx.x * RT + threadIdx.x; i < n; i += gridDim.x * RT) bucket[start[la[i]] + lr[i]] = lb[i];
}

constexpr uint32_t EU_CAP = 2048;     // entries of a block's buckets in LDS
constexpr uint32_t EU_VERTS = 64;     // buckets per block
constexpr uint32_t EU_SMALL = 64;     // entries of a bucket sorted by comparison counts
constexpr int EU_PER = EU_CAP / RT;   // entries per thread
static_assert(EU_SMALL <= 64, "a small bucket's bits lie in two words");

// b[0, n), n <= EU_CAP, ascending (every thread; b is padded up to a power of two)
__device__ __forceinline__ void bitonic_sort(uint32_t* b, uint32_t n) {
  uint32_t p = 1u;
  while (p < n) p <<= 1;
  for (uint32_t i = n + threadIdx.x; i < p; i += RT) b[i] = ~0u;
  __syncthreads();
  for (uint32_t k = 2u; k <= p; k <<= 1)
    for (uint32_t j = k >> 1; j > 0u; j >>= 1) {
      for (uint32_t q = threadIdx.x; q < p / 2u; q += RT) {
        const uint32_t i = ((q & ~(j - 1u)) << 1) | (q & (j - 1u));
        const uint32_t x = b[i], y = b[i + j];
        if ((x > y) == ((i & k) == 0u)) {
          b[i] = y;
          b[i + j] = x;
        }
      }
      __syncthreads();
    }
}

// Each bucket sorted and freed of repeats in place; ucnt: what is left of it,
// bsum: of the block's buckets.  start[V] is the end of the last bucket.  The
// long ones are listed for k_edge_long.
__global__ __launch_bounds__(RT) void k_edge_unique(const uint32_t* start, uint32_t V, uint32_t* bucket,
                                                    uint32_t* n_long, uint32_t* long_v, uint32_t* ucnt,
                                                    uint32_t* bsum) {
  __shared__ uint32_t b[EU_CAP];
  __shared__ uint8_t owner[EU_CAP];
  __shared__ uint64_t keep[EU_CAP / 64];
  __shared__ uint32_t s0[EU_VERTS + 1], u[EU_VERTS];
  __shared__ uint32_t lds[RT / 64];
  const uint32_t v0 = blockIdx.x * EU_VERTS, nv = min(EU_VERTS, V - v0), t = threadIdx.x;
  if (t <= nv) s0[t] = start[v0 + t];
  if (t < EU_VERTS) u[t] = 0u;
  __syncthreads();
  for (uint32_t g0 = 0; g0 < nv;) {
    uint32_t g1 = g0 + 1u;
    const uint32_t e0 = s0[g0], n0 = s0[g1] - e0;
    if (n0 > EU_CAP) {
      if (t == 0u) long_v[atomicAdd(n_long, 1u)] = v0 + g0;
      g0 = g1;
      continue;
    }
    if (n0 > EU_SMALL) {
      for (uint32_t i = t; i < n0; i += RT) b[i] = bucket[e0 + i];
      bitonic_sort(b, n0);
      uint32_t run = 0;
      for (uint32_t i0 = 0; i0 < n0; i0 += RT) {
        const uint32_t i = i0 + t;
        const bool keep = i < n0 && (i == 0u || b[i - 1u] != b[i]);
        uint32_t tot;
        const uint32_t p = run + block_scan_excl(keep ? 1u : 0u, lds, &tot);
        if (keep) bucket[e0 + p] = b[i];
        run += tot;
      }
      if (t == 0u) u[g0] = run;
      __syncthreads();
      g0 = g1;
      continue;
    }
    // as many small buckets at a time as fit in LDS: an entry's place is the
    // number of entries before it in the bucket's order
    while (g1 < nv && s0[g1 + 1u] - e0 <= EU_CAP && s0[g1 + 1u] - s0[g1] <= EU_SMALL) ++g1;
    const uint32_t n = s0[g1] - e0;
    for (uint32_t i = t; i < n; i += RT) b[i] = bucket[e0 + i];
    for (uint32_t g = g0 + t; g < g1; g += RT)
      for (uint32_t i = s0[g] - e0; i < s0[g + 1u] - e0; ++i) owner[i] = (uint8_t)g;
    __syncthreads();
    uint32_t x[EU_PER], p[EU_PER];
#pragma unroll
    for (int q = 0; q < EU_PER; ++q) {
      const uint32_t i = t + RT * q;
      if (i >= n) continue;
      x[q] = b[i];
      const uint32_t g = owner[i], i0 = s0[g] - e0, i1 = s0[g + 1u] - e0;
      p[q] = i0;
      for (uint32_t j = i0; j < i1; ++j) p[q] += (b[j] < x[q] || (b[j] == x[q] && j < i)) ? 1u : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EU_PER; ++q)
      if (t + RT * q < n) b[p[q]] = x[q];
    __syncthreads();
    // the first of every run of equal ones, as a bit per entry
#pragma unroll
    for (int q = 0; q < EU_PER; ++q) {
      const uint32_t i = t + RT * q;
      const bool first = i < n && (i == s0[owner[i]] - e0 || b[i - 1u] != b[i]);
      const uint64_t m = __ballot(first);
      if ((t & 63u) == 0u) keep[i >> 6] = m;
    }
    __syncthreads();
    // set bits of keep in [i0, i1), at most EU_SMALL apart
    const auto kept = [&](uint32_t i0, uint32_t i1) {
      const uint32_t w = i0 >> 6;
      const uint64_t lo = keep[w] & (~0ull << (i0 & 63u)), hi = w + 1u < EU_CAP / 64u ? keep[w + 1u] : 0ull;
      if (i1 <= 64u * w + 64u) return (uint32_t)__popcll(i1 > i0 ? lo & (~0ull >> (63u - ((i1 - 1u) & 63u))) : 0ull);
      return (uint32_t)__popcll(lo) + (uint32_t)__popcll(hi & (~0ull >> (63u - ((i1 - 1u) & 63u))));
    };
#pragma unroll
    for (int q = 0; q < EU_PER; ++q) {
      const uint32_t i = t + RT * q;
      if (i >= n || !((keep[i >> 6] >> (i & 63u)) & 1ull)) continue;
      const uint32_t i0 = s0[owner[i]] - e0;
      bucket[e0 + i0 + kept(i0, i)] = b[i];
    }
    for (uint32_t g = g0 + t; g < g1; g += RT) u[g] = kept(s0[g] - e0, s0[g + 1u] - e0);
    __syncthreads();
    g0 = g1;
  }
  if (t < nv) ucnt[v0 + t] = u[t];
  if (t < 64u) {
    uint32_t x = t < nv ? u[t] : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (t == 0u) bsum[blockIdx.x] = x;
  }
}

// The buckets past EU_CAP: a bitmap of the upper vertices in LDS, EL_BITS of
// them at a time, gives a bucket in order and without repeats in one pass over
// its entries per window.  A block per bucket; the result goes to long_out, at
// the bucket's own place, and ucnt and bsum as above.
constexpr uint32_t EL_T = 1024;
constexpr uint32_t EL_BITS = 1u << 20;   // 128 KB of LDS
constexpr uint32_t EL_PER = 16;          // loads of a thread in flight together
__global__ __launch_bounds__(EL_T) void k_edge_long(const uint32_t* start, uint32_t V, const uint32_t* bucket,
                                                    uint32_t* long_out, const uint32_t* n_long,
                                                    const uint32_t* long_v, uint32_t* ucnt, uint32_t* bsum) {
  __shared__ uint32_t bits[EL_BITS / 32];
  __shared__ uint32_t wsum[EL_T / 64];
  const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, nl = *n_long;
  for (uint32_t l = blockIdx.x; l < nl; l += gridDim.x) {
    const uint32_t a = long_v[l], e0 = start[a], n = start[a + 1u] - e0;
    uint32_t run = 0;
    for (uint32_t w0 = a; w0 < V; w0 += EL_BITS) {   // (a tet with a repeated vertex has the pair (a, a))
      const uint32_t nw = min(EL_BITS, V - w0), words = (nw + 31u) / 32u;
      for (uint32_t i = t; i < words; i += EL_T) bits[i] = 0u;
      __syncthreads();
      for (uint32_t r0 = 0; r0 < n; r0 += EL_T * EL_PER) {
        uint32_t x[EL_PER];   // (past the bucket: its last entry again; below the window: wraps past it)
#pragma unroll
        for (uint32_t q = 0; q < EL_PER; ++q) x[q] = bucket[e0 + min(r0 + q * EL_T + t, n - 1u)] - w0;
#pragma unroll
        for (uint32_t q = 0; q < EL_PER; ++q)
          if (x[q] < nw) atomicOr(&bits[x[q] >> 5], 1u << (x[q] & 31u));
      }
      __syncthreads();
      // a wave's words are consecutive, 64 of them a round
      const uint32_t per = (words + EL_T - 1u) / EL_T * 64u, i0 = wave * per, i1 = min(i0 + per, words);
      uint32_t c = 0u;
      for (uint32_t i = i0 + lane; i < i1; i += 64u) c += (uint32_t)__popc(bits[i]);
      c = wave_scan_add(c);
      if (lane == 63u) wsum[wave] = c;
      __syncthreads();
      uint32_t o = run;
#pragma unroll
      for (uint32_t w = 0; w < EL_T / 64; ++w) {
        o += w < wave ? wsum[w] : 0u;
        run += wsum[w];
      }
      for (uint32_t i = i0; i < i1; i += 64u) {
        uint32_t m = i + lane < i1 ? bits[i + lane] : 0u;
        const uint32_t m1 = (uint32_t)__popc(m), x = wave_scan_add(m1);
        uint32_t p = e0 + o + x - m1;
        for (; m != 0u; m &= m - 1u) long_out[p++] = w0 + 32u * (i + lane) + (uint32_t)__ffs(m) - 1u;
        o += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
      }
      __syncthreads();
    }
    if (t == 0u) {
      ucnt[a] = run;
      atomicAdd(&bsum[a / EU_VERTS], run);
    }
    __syncthreads();
  }
}

// The edges out, 64 vertices a block; a long bucket by EO_PARTS of the blocks
// past those (256 threads would take 1.4 ms for a million edges).
constexpr uint32_t EO_PARTS = 16, EO_LONG = 512;   // EO_LONG: blocks for the long buckets
__global__ __launch_bounds__(RT) void k_edge_out(const uint32_t* start, uint32_t V, uint32_t nu, const uint32_t* bucket,
                                                 const uint32_t* long_out, const uint32_t* n_long,
                                                 const uint32_t* long_v, const uint32_t* ucnt, const uint32_t* bsum,
                                                 int2* edges) {
  __shared__ uint32_t off[EU_VERTS + 1], s0[EU_VERTS + 1];
  const uint32_t t = threadIdx.x;
  // a block's vertices: the bounds of their buckets and their edges' offsets
  const auto load = [&](uint32_t blk) {
    const uint32_t v0 = blk * EU_VERTS, nv = min(EU_VERTS, V - v0);
    if (t < 64u) {
      const uint32_t c = t < nv ? ucnt[v0 + t] : 0u, x = wave_scan_add(c);
      off[t + 1u] = x;
      if (t == 0u) off[0] = 0u;
    }
    if (t <= nv) s0[t] = start[v0 + t];
    __syncthreads();
  };
  if (blockIdx.x >= nu) {
    const uint32_t nw = *n_long * EO_PARTS;
    for (uint32_t w = blockIdx.x - nu; w < nw; w += gridDim.x - nu) {
      const uint32_t a = long_v[w / EO_PARTS], g = a % EU_VERTS;
      load(a / EU_VERTS);
      const uint32_t n = off[g + 1u] - off[g], o = bsum[a / EU_VERTS] + off[g], e0 = s0[g];
      for (uint32_t i = w % EO_PARTS * RT + t; i < n; i += EO_PARTS * RT)
        edges[o + i] = make_int2((int32_t)a, (int32_t)long_out[e0 + i]);
      __syncthreads();
    }
    return;
  }
  load(blockIdx.x);
  const uint32_t v0 = blockIdx.x * EU_VERTS, n = off[EU_VERTS], o0 = bsum[blockIdx.x];
  for (uint32_t i = t; i < n; i += RT) {
    uint32_t g = 0;   // the last vertex whose first edge is at or before i
#pragma unroll
    for (uint32_t step = EU_VERTS / 2; step > 0u; step >>= 1) g = off[g + step] <= i ? g + step : g;
    if (s0[g + 1u] - s0[g] > EU_CAP) {   // on to the end of the long bucket
      i += (off[g + 1u] - 1u - i) / RT * RT;
      continue;
    }
    edges[o0 + i] = make_int2((int32_t)(v0 + g), (int32_t)bucket[s0[g] + (i - off[g])]);
  }
}

// ---------------------------------------------------------------------------
// regularisers
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(RT) void k_fill_f32(float* p, size_t n, float v) {
  for (size_t i = blockIdx.x * (size_t)RT + threadIdx.x; i < n; i += (size_t)gridDim.x * RT) p[i] = v;
}

// the three accumulators of the gradient pass, cleared in one launch
__global__ __launch_bounds__(RT) void k_reg_clear(float* dm, float* dverts, float* dsdf, size_t V) {
  for (size_t i = blockIdx.x * (size_t)RT + threadIdx.x; i < 3 * V; i += (size_t)gridDim.x * RT) {
    dm[i] = 0.0f;
    dverts[i] = 0.0f;
    if (i < V) dsdf[i] = 0.0f;
  }
}

__device__ __forceinline__ float block_sum_vs(float v, float* lds /*[VS_T/64]*/) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.0f;
#pragma unroll
  for (int w = 0; w < VS_T / 64; ++w) s += lds[w];
  return s;
}

__global__ __launch_bounds__(VS_T) void k_reg_tet_fwd(const float* verts, const int32_t* tets, const float* sdf,
                                                    int32_t V, uint32_t K, uint32_t chunk, float* m, float* part) {
  __shared__ VertexSums<3> S;
  __shared__ float lds[VS_T / 64];
  float eik = 0.0f;
  const uint32_t nchunks = (K + chunk - 1) / chunk, nj = (nchunks + 7u) / 8u * 8u;
  for (uint32_t j = blockIdx.x; j < nj; j += gridDim.x) {
    const uint32_t ch = xcd_chunk(j, nchunks);
    if (ch >= nchunks) continue;
    vs_clear(S);
    __syncthreads();
    const uint32_t k1 = min(K, (ch + 1u) * chunk);
    for (uint32_t k = ch * chunk + vs_item(); k < k1; k += VS_T) {
      int32_t v[4];
      if (!load_tet(tets, k, V, v)) continue;
      TetGrad T;
      tet_grad(verts, sdf, v, T);
      if (T.det == 0.0f) continue;
      const float gn = sqrtf(T.g[0] * T.g[0] + T.g[1] * T.g[1] + T.g[2] * T.g[2]);
      eik += (gn - 1.0f) * (gn - 1.0f);
      if (gn > 0.0f) {
        const float ig = 1.0f / gn;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const int p = vs_place(S, (uint32_t)v[a]);
#pragma unroll
          for (int c = 0; c < 3; ++c) vs_add<3, 3>(S, p, c, T.g[c] * ig, m, v[a], c);
        }
      }
    }
    __syncthreads();
    vs_flush<3, 3>(S, 0, m);
    __syncthreads();
  }
  const float s = block_sum_vs(eik, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// one edge: its term of L_nc (0 if left out) and, per end, the unit normal
// and inverse length that its gradient needs
struct EdgeTerm {
  float t;                 // 1 - cos = |u_b - u_a|^2 / 2
  float ua[3], ub[3], d[3], ia, ib;
};
__device__ __forceinline__ bool edge_term(const float* m, int2 ab, int32_t V, EdgeTerm& E) {
  if ((uint32_t)ab.x >= (uint32_t)V || (uint32_t)ab.y >= (uint32_t)V) return false;
  float ma[3], mb[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    ma[c] = m[3 * (size_t)ab.x + c];
    mb[c] = m[3 * (size_t)ab.y + c];
  }
  const float la = sqrtf(ma[0] * ma[0] + ma[1] * ma[1] + ma[2] * ma[2]);
  const float lb = sqrtf(mb[0] * mb[0] + mb[1] * mb[1] + mb[2] * mb[2]);
  if (!(la > 0.0f && lb > 0.0f)) return false;
  E.ia = 1.0f / la;
  E.ib = 1.0f / lb;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    E.ua[c] = ma[c] * E.ia;
    E.ub[c] = mb[c] * E.ib;
    E.d[c] = E.ub[c] - E.ua[c];
  }
  E.t = 0.5f * (E.d[0] * E.d[0] + E.d[1] * E.d[1] + E.d[2] * E.d[2]);
  return true;
}

__global__ __launch_bounds__(RT) void k_reg_edge(const int32_t* edges, const int32_t* n_edges, uint32_t cap,
                                                 int32_t V, const float* m, float* part) {
  __shared__ float lds[RT / 64];
  const uint32_t ne = min((uint32_t)max(n_edges[0], 0), cap);
  float nc = 0.0f;
  for (uint32_t e = blockIdx.x * RT + threadIdx.x; e < ne; e += gridDim.x * RT) {
    EdgeTerm E;
    if (edge_term(m, reinterpret_cast<const int2*>(edges)[e], V, E)) nc += E.t;
  }
  const float s = block_sum(nc, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// dL/dm of the consistency term; the loss partial sums again where part is given
__global__ __launch_bounds__(VS_T) void k_reg_edge_bwd(const int32_t* edges, const int32_t* n_edges, uint32_t cap,
                                                     int32_t V, uint32_t chunk, const float* m, float* dm,
                                                     const float* w, float* part) {
  __shared__ VertexSums<3> S;
  __shared__ float lds[VS_T / 64];
  const uint32_t ne = min((uint32_t)max(n_edges[0], 0), cap);
  const float wnc = w[1];
  float nc = 0.0f;
  const uint32_t nchunks = (ne + chunk - 1) / chunk, nj = (nchunks + 7u) / 8u * 8u;
  for (uint32_t j = blockIdx.x; j < nj; j += gridDim.x) {
    const uint32_t ch = xcd_chunk(j, nchunks);
    if (ch >= nchunks) continue;
    vs_clear(S);
    __syncthreads();
    const uint32_t e1 = min(ne, (ch + 1u) * chunk);
    for (uint32_t e = ch * chunk + vs_item(); e < e1; e += VS_T) {
      const int2 ab = reinterpret_cast<const int2*>(edges)[e];
      EdgeTerm E;
      if (!edge_term(m, ab, V, E)) continue;
      nc += E.t;
      // d(1 - ua.ub)/dm_a = -(ub - cos ua)/|m_a| = -(d + t ua)/|m_a|, and symmetrically for b
      const int pa = vs_place(S, (uint32_t)ab.x), pb = vs_place(S, (uint32_t)ab.y);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float xa = -wnc * (E.d[c] + E.t * E.ua[c]) * E.ia, xb = -wnc * (-E.d[c] + E.t * E.ub[c]) * E.ib;
        vs_add<3, 3>(S, pa, c, xa, dm, ab.x, c);
        vs_add<3, 3>(S, pb, c, xb, dm, ab.y, c);
      }
    }
    __syncthreads();
    vs_flush<3, 3>(S, 0, dm);
    __syncthreads();
  }
  if (!part) return;
  const float s = block_sum_vs(nc, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ __launch_bounds__(VS_T) void k_reg_tet_bwd(const float* verts, const int32_t* tets, const float* sdf,
                                                    int32_t V, uint32_t K, uint32_t chunk, const float* dm,
                                                    const float* w, float* dverts, float* dsdf) {
  __shared__ VertexSums<4> S;   // dverts xyz, dsdf
  const float weik = w[0];
  const uint32_t nchunks = (K + chunk - 1) / chunk, nj = (nchunks + 7u) / 8u * 8u;
  for (uint32_t j = blockIdx.x; j < nj; j += gridDim.x) {
    const uint32_t ch = xcd_chunk(j, nchunks);
    if (ch >= nchunks) continue;
    vs_clear(S);
    __syncthreads();
    const uint32_t k1 = min(K, (ch + 1u) * chunk);
    for (uint32_t k = ch * chunk + vs_item(); k < k1; k += VS_T) {
      int32_t v[4];
      if (!load_tet(tets, k, V, v)) continue;
      TetGrad T;
      tet_grad(verts, sdf, v, T);
      if (T.det == 0.0f) continue;
      const float gn = sqrtf(T.g[0] * T.g[0] + T.g[1] * T.g[1] + T.g[2] * T.g[2]);
      if (!(gn > 0.0f)) continue;
      const float ig = 1.0f / gn;
      float n[3], dn[3] = {0.0f, 0.0f, 0.0f}, dg[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) n[c] = T.g[c] * ig;
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) dn[c] += dm[3 * (size_t)v[a] + c];
      const float nd = n[0] * dn[0] + n[1] * dn[1] + n[2] * dn[2];
      const float ke = weik * 2.0f * (gn - 1.0f);
#pragma unroll
      for (int c = 0; c < 3; ++c) dg[c] = ke * n[c] + (dn[c] - n[c] * nd) * ig;
      // g = E^-1 df: dL/ddf = E^-T dg = mu; dL/dE = -mu g^T
      float mu[4], msum = 0.0f;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        mu[a + 1] = (T.cr[a][0] * dg[0] + T.cr[a][1] * dg[1] + T.cr[a][2] * dg[2]) / T.det;
        msum += mu[a + 1];
      }
      mu[0] = -msum;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int p = vs_place(S, (uint32_t)v[a]);
#pragma unroll
        for (int c = 0; c < 3; ++c) vs_add<4, 3>(S, p, c, -mu[a] * T.g[c], dverts, v[a], c);
        vs_add<4, 1>(S, p, 3, mu[a], dsdf, v[a], 0);
      }
    }
    __syncthreads();
    vs_flush<4, 3>(S, 0, dverts);
    vs_flush<4, 1>(S, 3, dsdf);
    __syncthreads();
  }
}


// ---------------------------------------------------------------------------
// Marching Tetrahedra
// ---------------------------------------------------------------------------
struct MTCase {
  uint8_t ntri;   // 0, 1 or 2
  uint8_t o[4];   // local vertex order (i, j, k, l), an even permutation
  uint8_t rev;    // reverse the winding (lone outside vertex)
};
struct MTTable {
  MTCase c[16];
};

constexpr MTTable make_mt_table() {
  MTTable T{};
  for (int m = 0; m < 16; ++m) {
    const int cnt = (m & 1) + ((m >> 1) & 1) + ((m >> 2) & 1) + ((m >> 3) & 1);
    MTCase c{};
    int o[4] = {0, 1, 2, 3};
    int n = 0;
    if (cnt == 1 || cnt == 3) {
      const int want = cnt == 1 ? 1 : 0;
      for (int q = 0; q < 4; ++q)
        if (((m >> q) & 1) == want) o[n++] = q;
      for (int q = 0; q < 4; ++q)
        if (((m >> q) & 1) != want) o[n++] = q;
      c.ntri = 1;
      c.rev = cnt == 3;
    } else if (cnt == 2) {
      for (int q = 0; q < 4; ++q)
        if ((m >> q) & 1) o[n++] = q;
      for (int q = 0; q < 4; ++q)
        if (!((m >> q) & 1)) o[n++] = q;
      c.ntri = 2;
    }
    int inv = 0;
    for (int a = 0; a < 4; ++a)
      for (int b = a + 1; b < 4; ++b) inv += o[a] > o[b];
    if (inv & 1) {
      const int t = o[2];
      o[2] = o[3];
      o[3] = t;
    }
    for (int q = 0; q < 4; ++q) c.o[q] = (uint8_t)o[q];
    T.c[m] = c;
  }
  return T;
}
__constant__ MTTable c_mt = make_mt_table();

// Marching Tetrahedra runs in three passes with a scan between.  The first
// marks: per edge whether its ends differ in the inside test, per tet its four
// inside bits, as ballots of 64 consecutive edges or tets (a wave takes eight
// rows of 64, so that every load is contiguous), and counts per block.  The
// writing passes read the marks, not the SDF, and only the marked few do any
// work: the tets that give triangles are first listed per block in LDS, in tet
// order.  A crossed edge's number is found through the first edge of its lower
// vertex where the table of those fits the workspace (a binary search over all
// edges otherwise: some 21 dependent loads against 3).
constexpr int MT_ROWS = EDGE_ITEMS;   // rows of 64 per wave: EDGE_TILE per block

__global__ __launch_bounds__(RT) void k_mt_edge_mark(const float* sdf, int32_t V, const int32_t* edges,
                                                     const int32_t* n_edges, uint32_t cap, uint64_t* mark,
                                                     uint32_t* first_edge, uint32_t* bsum) {
  __shared__ uint32_t wsum[RT / 64];
  const uint32_t ne = min((uint32_t)max(n_edges[0], 0), cap);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t j0 = blockIdx.x * EDGE_TILE + wave * (64u * MT_ROWS);
  uint32_t cnt = 0;
  int2 e[MT_ROWS];
#pragma unroll
  for (int i = 0; i < MT_ROWS; ++i) {
    const uint32_t j = j0 + 64u * i + lane;
    e[i] = j < ne ? reinterpret_cast<const int2*>(edges)[j] : make_int2(-1, -1);
  }
#pragma unroll
  for (int i = 0; i < MT_ROWS; ++i) {
    const uint32_t j = j0 + 64u * i + lane;
    const bool ok = (uint32_t)e[i].x < (uint32_t)V && (uint32_t)e[i].y < (uint32_t)V;
    const bool cut = ok && (sdf[e[i].x] < 0.0f) != (sdf[e[i].y] < 0.0f);
    const uint64_t m = __ballot(cut);
    if (lane == 0u && j0 + 64u * i < ne) mark[(j0 + 64u * i) / 64u] = m;
    cnt += (uint32_t)__popcll(m);
    if (first_edge) {
      // edges ascend by (a, b): the first of its lower vertex differs from the
      // one before (an unused vertex's entry is never read; every lane takes part
      // in the exchange, also one whose own edge is foreign or past the list)
      int before = __shfl_up(e[i].x, 1, 64);
      if (lane == 0u) before = j > 0u && j < ne ? reinterpret_cast<const int2*>(edges)[j - 1u].x : -1;
      if (ok && before != e[i].x) first_edge[e[i].x] = j;
    }
  }
  if (lane == 0u) wsum[wave] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// the edge blocks' and the tet blocks' sums, a block each
__global__ __launch_bounds__(1024) void k_mt_spines(uint32_t* be, uint32_t ne, uint32_t* bt, uint32_t nt,
                                                    int32_t* counts) {
  if (blockIdx.x == 0) spine_1024(be, ne, counts);
  else spine_1024(bt, nt, counts + 1);
}

__global__ __launch_bounds__(RT) void k_fill_u32(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = blockIdx.x * (size_t)RT + threadIdx.x; i < n; i += (size_t)gridDim.x * RT) p[i] = v;
}

__global__ __launch_bounds__(RT) void k_mt_edge_write(const float* verts, const float* sdf, const int32_t* edges,
                                                      const int32_t* n_edges, uint32_t cap, const uint64_t* mark,
                                                      const uint32_t* bsum, int32_t* vid, float* out,
                                                      uint32_t vcap) {
  __shared__ uint32_t wsum[RT / 64];
  const uint32_t ne = min((uint32_t)max(n_edges[0], 0), cap);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t j0 = blockIdx.x * EDGE_TILE + wave * (64u * MT_ROWS);
  uint64_t m[MT_ROWS];
  uint32_t cnt = 0;
#pragma unroll
  for (int i = 0; i < MT_ROWS; ++i) {
    m[i] = j0 + 64u * i < ne ? mark[(j0 + 64u * i) / 64u] : 0ull;
    cnt += (uint32_t)__popcll(m[i]);
  }
  if (lane == 0u) wsum[wave] = cnt;
  __syncthreads();
  uint32_t o0 = bsum[blockIdx.x];
  for (uint32_t w = 0; w < wave; ++w) o0 += wsum[w];
#pragma unroll 1
  for (int i = 0; i < MT_ROWS; ++i) {
    const uint32_t j = j0 + 64u * i + lane, o = o0 + (uint32_t)__popcll(m[i] & ((1ull << lane) - 1ull));
    o0 += (uint32_t)__popcll(m[i]);
    const bool cut = (m[i] >> lane) & 1ull;
    if (j < ne) vid[j] = cut ? (int32_t)o : -1;
    if (!cut || o >= vcap) continue;
    const int2 ab = reinterpret_cast<const int2*>(edges)[j];
    const float fa = sdf[ab.x], fb = sdf[ab.y];
    const float tt = fa / (fa - fb);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float xa = verts[3 * (size_t)ab.x + c], xb = verts[3 * (size_t)ab.y + c];
      out[3 * (size_t)o + c] = xa + tt * (xb - xa);
    }
  }
}

__global__ __launch_bounds__(RT) void k_mt_tet_mark(const int32_t* tets, const float* sdf, int32_t V, uint32_t K,
                                                    uint64_t* mark, uint32_t* bsum) {
  __shared__ uint32_t wsum[RT / 64];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t k0 = blockIdx.x * EDGE_TILE + wave * (64u * MT_ROWS);
  uint32_t cnt = 0;
#pragma unroll
  for (int i = 0; i < MT_ROWS; ++i) {
    const uint32_t k = k0 + 64u * i + lane;
    int32_t v[4];
    bool in[4] = {false, false, false, false};
    if (k < K && load_tet(tets, k, V, v)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) in[q] = sdf[v[q]] < 0.0f;
    }
    uint64_t m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) m[q] = __ballot(in[q]);
    if (lane < 4u && k0 + 64u * i < K)
      mark[4 * (size_t)((k0 + 64u * i) / 64u) + lane] = lane == 0u ? m[0] : lane == 1u ? m[1] : lane == 2u ? m[2] : m[3];
    // one triangle where one or three are inside, two where two are
    const uint64_t odd = m[0] ^ m[1] ^ m[2] ^ m[3];
    const uint64_t some = m[0] | m[1] | m[2] | m[3], all = m[0] & m[1] & m[2] & m[3];
    cnt += (uint32_t)__popcll(odd) + 2u * (uint32_t)__popcll(some & ~all & ~odd);
  }
  if (lane == 0u) wsum[wave] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// the numbers of four edges' surface vertices (u_q, w_q), -1 if absent, their
// dependent loads in flight together
__device__ __forceinline__ void surf_vertices(const int32_t* edges, uint32_t ne, const uint32_t* first_edge,
                                              const int32_t* vid, const int32_t (&u)[4], const int32_t (&w)[4],
                                              int32_t (&out)[4]) {
  const int2* E = reinterpret_cast<const int2*>(edges);
  int32_t a[4], b[4];
  uint32_t lo[4];
  bool open[4];   // E[lo] may still be below (a, b)
  if (ne == 0u) {   // (an empty list has no last edge to read instead)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = -1;
    return;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a[q] = min(u[q], w[q]);
    b[q] = max(u[q], w[q]);
    lo[q] = first_edge ? first_edge[a[q]] : 0u;   // (past the list for a vertex without edges)
    open[q] = lo[q] < ne;
  }
  if (first_edge) {
    // a's edges follow its first one, most often within a cache line
    for (int step = 0; step < 8; ++step) {
      int2 e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = E[min(lo[q], ne - 1u)];
      bool any = false;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        open[q] = open[q] && (e[q].x < a[q] || (e[q].x == a[q] && e[q].y < b[q]));
        lo[q] += open[q] ? 1u : 0u;
        open[q] = open[q] && lo[q] < ne;
        any = any || open[q];
      }
      if (!any) break;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (open[q]) {   // no table, or a vertex of many edges
      uint32_t hi = ne;
      while (lo[q] < hi) {
        const uint32_t mid = (lo[q] + hi) >> 1;
        const int2 e = E[mid];
        if (e.x < a[q] || (e.x == a[q] && e.y < b[q])) lo[q] = mid + 1u;
        else hi = mid;
      }
    }
    out[q] = -1;
    if (lo[q] < ne) {
      const int2 e = E[lo[q]];
      if (e.x == a[q] && e.y == b[q]) out[q] = vid[lo[q]];
    }
  }
}

// four blocks per EDGE_TILE tets, each with the rows of one wave: a block of
// the surface has some 800 crossed tets, whose chains of dependent loads would
// follow one another
__global__ __launch_bounds__(RT) void k_mt_tet_write(const float* verts, const int32_t* tets, uint32_t K,
                                                     const int32_t* edges, const int32_t* n_edges, uint32_t cap,
                                                     const uint32_t* first_edge, const int32_t* vid,
                                                     const uint64_t* mark, const uint32_t* bsum, int32_t* tris,
                                                     uint32_t tcap) {
  __shared__ uint32_t wsum[RT / 64][2];
  static_assert(MT_ROWS == 8, "a row per lane 0 to 7");
  constexpr uint32_t ROWS = 64u * MT_ROWS;
  __shared__ uint32_t list[ROWS];   // the block's crossed tets: place << 4 | inside bits
  __shared__ uint32_t tri0[ROWS];   // and their first triangles
  const uint32_t tile = blockIdx.x / (RT / 64), sub = blockIdx.x % (RT / 64);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  // the crossed tets and triangles of every wave's rows (the earlier ones' are
  // this block's offset)
  uint32_t nx = 0, ntri = 0;
  uint64_t x8 = 0ull, odd8 = 0ull, in8[4] = {0ull, 0ull, 0ull, 0ull};   // this lane's row (lanes 0 to 7)
  const uint32_t krow = tile * EDGE_TILE + wave * ROWS + 64u * (lane & (MT_ROWS - 1u));
  if (lane < (uint32_t)MT_ROWS && krow < K) {
#pragma unroll
    for (int q = 0; q < 4; ++q) in8[q] = mark[4 * (size_t)(krow / 64u) + q];
    odd8 = in8[0] ^ in8[1] ^ in8[2] ^ in8[3];
    x8 = (in8[0] | in8[1] | in8[2] | in8[3]) & ~(in8[0] & in8[1] & in8[2] & in8[3]);
    nx = (uint32_t)__popcll(x8);
    ntri = nx + (uint32_t)__popcll(x8 & ~odd8);
  }
  const uint32_t sx = wave_scan_add(nx), st = wave_scan_add(ntri);
  if (lane == 63u) {
    wsum[wave][0] = sx;
    wsum[wave][1] = st;
  }
  __syncthreads();
  const uint32_t nlist = wsum[sub][0];
  if (nlist == 0u) return;
  if (wave == sub) {
    uint32_t o0 = bsum[tile];
    for (uint32_t w = 0; w < sub; ++w) o0 += wsum[w][1];
    // a lane lists its row's crossed tets
    uint32_t p = sx - nx, o = o0 + st - ntri;
    for (uint64_t r = x8; r != 0ull; r &= r - 1ull) {
      const uint32_t bit = (uint32_t)__ffsll((unsigned long long)r) - 1u;
      uint32_t bits = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) bits |= (uint32_t)((in8[q] >> bit) & 1ull) << q;
      list[p] = (64u * lane + bit) << 4 | bits;
      tri0[p] = o;
      o += ((odd8 >> bit) & 1ull) ? 1u : 2u;
      ++p;
    }
  }
  __syncthreads();
  const uint32_t ne = min((uint32_t)max(n_edges[0], 0), cap);
  for (uint32_t p = threadIdx.x; p < nlist; p += RT) {
    const MTCase c = c_mt.c[list[p] & 15u];
    const int4 row = reinterpret_cast<const int4*>(tets)[tile * EDGE_TILE + sub * ROWS + (list[p] >> 4)];
    const int32_t v[4] = {row.x, row.y, row.z, row.w};
    // orientation of the tet: sign of det[x1 - x0, x2 - x0, x3 - x0]
    float e[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int q = 0; q < 3; ++q) e[a][q] = verts[3 * (size_t)v[a + 1] + q] - verts[3 * (size_t)v[0] + q];
    const float det = e[0][0] * (e[1][1] * e[2][2] - e[1][2] * e[2][1]) +
                      e[0][1] * (e[1][2] * e[2][0] - e[1][0] * e[2][2]) +
                      e[0][2] * (e[1][0] * e[2][1] - e[1][1] * e[2][0]);
    const bool flip = det < 0.0f;
    const auto pick = [&](int q) { return q == 0 ? v[0] : q == 1 ? v[1] : q == 2 ? v[2] : v[3]; };
    const int32_t i = pick(c.o[0]), j = pick(c.o[1]), kk = pick(c.o[2]), l4 = pick(c.o[3]);
    // one triangle: edges ij, ik, il; two: ik, il, jl, jk
    const bool two = c.ntri == 2;
    const int32_t eu[4] = {i, i, two ? j : i, two ? j : i}, ew[4] = {two ? kk : j, two ? l4 : kk, l4, two ? kk : l4};
    int32_t sv[4];
    surf_vertices(edges, ne, first_edge, vid, eu, ew, sv);
    const int32_t tri[2][3] = {{sv[0], sv[1], sv[2]}, {sv[0], sv[2], sv[3]}};
    const bool rev = flip != (c.rev != 0);
    uint32_t to = tri0[p];
#pragma unroll
    for (int q = 0; q < 2; ++q, ++to) {
      if (q >= c.ntri || to >= tcap) continue;
      tris[3 * (size_t)to + 0] = tri[q][0];
      tris[3 * (size_t)to + 1] = rev ? tri[q][2] : tri[q][1];
      tris[3 * (size_t)to + 2] = rev ? tri[q][1] : tri[q][2];
    }
  }
}

__global__ __launch_bounds__(RT) void k_reg_losses(const float* part, int nb, double* losses) {
  __shared__ double lds[2][RT / 64];
  double s0 = 0.0, s1 = 0.0;
  for (int i = threadIdx.x; i < nb; i += RT) {
    s0 += (double)part[i];
    s1 += (double)part[nb + i];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    s0 += __shfl_xor(s0, o, 64);
    s1 += __shfl_xor(s1, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    lds[0][threadIdx.x >> 6] = s0;
    lds[1][threadIdx.x >> 6] = s1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int w = 0; w < RT / 64; ++w) {
      a += lds[0][w];
      b += lds[1][w];
    }
    losses[0] = a;
    losses[1] = b;
  }
}

// Vertices that per-vertex workspaces sized by the tets make room for: a mesh has
// some six tets per vertex.  With more, most belong to no tet or the tets share
// few, and the calls take the ways that need no such array, as slow as they are.
inline uint64_t mesh_vertices(int32_t K) { return (uint64_t)K + 1024; }

inline size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
inline int bit_length(uint32_t x) { return x ? 32 - __builtin_clz(x) : 0; }

}  // namespace

// --- host side ------------------------------------------------------------------
EdgeLayout edge_layout(int32_t K) {
  EdgeLayout E{};
  const uint64_t n = 6ull * (uint64_t)K;
  E.n = n;
  E.sort_blocks = (n + SORT_TILE - 1) / SORT_TILE;
  E.edge_blocks = (n + EDGE_TILE - 1) / EDGE_TILE;
  // binned: the vertices the per-vertex arrays have room for
  E.verts = mesh_vertices(K);
  size_t o = 0;
  E.o_n = o; o += al(16);
  E.o_ka = o; o += al(4 * n);
  E.o_va = o; o += al(4 * n);
  E.o_kb = o; o += al(4 * n);
  E.o_vb = o; o += al(4 * n);
  E.o_hist = o; o += al(4 * (256 * (size_t)E.sort_blocks + 256));
  E.o_bsum = o; o += al(4 * (std::max<size_t>((size_t)E.edge_blocks, (size_t)E.verts / EU_VERTS + 1) + 1));
  E.o_start = o; o += al(4 * ((size_t)E.verts + VS_RUN + 1));
  E.o_ucnt = o; o += al(4 * (size_t)E.verts);
  E.bytes = o;
  return E;
}

// The binned build where the vertex arrays fit the workspace and the buckets are
// short on average: up to eight tets per vertex.  Random tets, a million of them:
// at 6 per vertex 777 us against 778 us with the sort, at 11 846 and 777, at 50
// 1590 and 608, where what counts is the buckets' own sort.
static bool mesh_edges_binned_fits(uint64_t K, uint64_t V, const EdgeLayout& E) {
  return V + 1 <= E.verts && K <= 8 * V;
}

static hipError_t mesh_edges_binned(const int32_t* tets, uint32_t K, uint32_t V, int32_t* edges, int32_t* n_edges,
                                    char* w, const EdgeLayout& E, hipStream_t st) {
  uint32_t* n_item = reinterpret_cast<uint32_t*>(w + E.o_n);
  uint32_t* la = reinterpret_cast<uint32_t*>(w + E.o_ka);
  uint32_t* lb = reinterpret_cast<uint32_t*>(w + E.o_va);
  uint32_t* lr = reinterpret_cast<uint32_t*>(w + E.o_kb);
  uint32_t* bucket = reinterpret_cast<uint32_t*>(w + E.o_vb);
  uint32_t* bsum = reinterpret_cast<uint32_t*>(w + E.o_bsum);
  uint32_t* start = reinterpret_cast<uint32_t*>(w + E.o_start);
  uint32_t* ucnt = reinterpret_cast<uint32_t*>(w + E.o_ucnt);
  const uint32_t nc = V + 1u;   // the counts and, behind them, the total
  k_edge_clear<<<std::max(1u, std::min((nc + RT - 1) / RT, 2048u)), RT, 0, st>>>(start, nc + VS_RUN, n_item);
  const uint32_t chunks = (K + EB_CHUNK - 1u) / EB_CHUNK;
  if (K > 0) k_edge_bin<<<std::min(chunks + 7u, 2048u), EB_T, 0, st>>>(tets, K, (int32_t)V, start, n_item, la, lb, lr);
  const uint32_t nb = (nc + EB_SCAN - 1u) / EB_SCAN;
  k_cnt_sum<<<nb, RT, 0, st>>>(start, nc, bsum);
  k_edge_spine<<<1, 1024, 0, st>>>(bsum, nb, n_edges);   // (n_edges is rewritten below)
  k_cnt_starts<<<nb, RT, 0, st>>>(start, nc, bsum);
  const uint32_t nu = (V + EU_VERTS - 1u) / EU_VERTS;
  if (K > 0)
    k_edge_place<<<(unsigned)std::min<uint64_t>((E.n + RT - 1) / RT, 4096), RT, 0, st>>>(start, n_item, la, lb, lr,
                                                                                         bucket);
  // (the list's arrays have been read: la takes the long buckets' edges, lr their vertices)
  const uint32_t nlong = (uint32_t)std::min<uint64_t>(E.n / EU_CAP, 256);   // 0: no bucket can be long
  if (nu > 0) k_edge_unique<<<nu, RT, 0, st>>>(start, V, bucket, n_item + 1, lr, ucnt, bsum);
  if (nu > 0 && nlong > 0)
    k_edge_long<<<nlong, EL_T, 0, st>>>(start, V, bucket, la, n_item + 1, lr, ucnt, bsum);
  k_edge_spine<<<1, 1024, 0, st>>>(bsum, nu, n_edges);
  if (nu > 0)
    k_edge_out<<<nu + (nlong > 0 ? EO_LONG : 0u), RT, 0, st>>>(start, V, nu, bucket, la, n_item + 1, lr, ucnt, bsum,
                                                               reinterpret_cast<int2*>(edges));
  return hipGetLastError();
}

hipError_t launch_mesh_edges(const int32_t* tets, int32_t K, int32_t V, int32_t* edges, int32_t* n_edges, void* ws,
                             const EdgeLayout& E, hipStream_t st) {
  char* w = static_cast<char*>(ws);
  if (mesh_edges_binned_fits((uint64_t)K, (uint64_t)V, E))
    return mesh_edges_binned(tets, (uint32_t)K, (uint32_t)V, edges, n_edges, w, E, st);
  // the 6 K pairs sorted by b, then stably by a
  uint32_t* n_dev = reinterpret_cast<uint32_t*>(w + E.o_n);
  uint32_t* ka = reinterpret_cast<uint32_t*>(w + E.o_ka);
  uint32_t* va = reinterpret_cast<uint32_t*>(w + E.o_va);
  uint32_t* kb = reinterpret_cast<uint32_t*>(w + E.o_kb);
  uint32_t* vb = reinterpret_cast<uint32_t*>(w + E.o_vb);
  uint32_t* hist = reinterpret_cast<uint32_t*>(w + E.o_hist);
  uint32_t* bsum = reinterpret_cast<uint32_t*>(w + E.o_bsum);
  const uint32_t n = (uint32_t)E.n;
  const unsigned g = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + RT - 1) / RT, 4096));
  k_edge_keys_b<<<g, RT, 0, st>>>(tets, n, V, ka, n_dev);
  const int bits = std::max(1, bit_length((uint32_t)V));
  uint32_t *ko = nullptr, *vo = nullptr;
  hipError_t e = radix_sort_pairs(ka, va, kb, vb, true, n_dev, (int64_t)n, bits, hist, (int64_t)E.sort_blocks, st,
                                  &ko, &vo);
  if (e != hipSuccess) return e;
  // second pass keyed by a, carrying the pair indices sorted by b
  k_edge_keys_a<<<g, RT, 0, st>>>(tets, n, V, vo, ko);
  uint32_t* k2 = (ko == ka) ? kb : ka;
  uint32_t* v2 = (vo == va) ? vb : va;
  e = radix_sort_pairs(ko, vo, k2, v2, false, n_dev, (int64_t)n, bits, hist, (int64_t)E.sort_blocks, st, &ko, &vo);
  if (e != hipSuccess) return e;
  const unsigned nb = (unsigned)E.edge_blocks;
  if (nb > 0) k_edge_count<<<nb, RT, 0, st>>>(tets, n, V, vo, bsum);
  k_edge_spine<<<1, 1024, 0, st>>>(bsum, nb, n_edges);
  if (nb > 0) k_edge_write<<<nb, RT, 0, st>>>(tets, n, V, vo, bsum, edges);
  return hipGetLastError();
}

RegLayout reg_layout(int32_t V) {
  RegLayout R{};
  size_t o = 0;
  R.o_m = o; o += al(4 * 3 * (size_t)V);
  R.o_dm = o; o += al(4 * 3 * (size_t)V);
  R.o_part = o; o += al(4 * 2 * (size_t)RBLOCKS);
  R.bytes = o;
  R.blocks = RBLOCKS;
  return R;
}

// Consecutive tets or edges that a block adds up in LDS: 2048, less where n
// would leave workgroups without work.
static uint32_t reg_chunk(uint64_t n) {
  const uint64_t c = (n / RBLOCKS + VS_T - 1) / VS_T * VS_T;
  return (uint32_t)std::max<uint64_t>(VS_T, std::min<uint64_t>(c, 2048));
}

hipError_t launch_regularizers(const float* verts, const int32_t* tets, const float* sdf, int32_t V, int32_t K,
                               const int32_t* edges, const int32_t* n_edges, int64_t edge_cap, const float* weights,
                               double* losses, float* dverts, float* dsdf, void* ws, const RegLayout& R,
                               hipStream_t st) {
  char* w = static_cast<char*>(ws);
  float* m = reinterpret_cast<float*>(w + R.o_m);
  float* dm = reinterpret_cast<float*>(w + R.o_dm);
  float* part = reinterpret_cast<float*>(w + R.o_part);
  const bool bwd = dverts != nullptr;
  const size_t nv3 = 3 * (size_t)V;
  const uint32_t ct = reg_chunk((uint64_t)K), ce = reg_chunk((uint64_t)edge_cap);
  // (m and dm are neighbours in the workspace: one fill)
  const size_t nz = bwd ? R.o_dm / 4 + nv3 : nv3;
  const unsigned gf = (unsigned)std::max<size_t>(1, std::min<size_t>((nz + RT - 1) / RT, 2048));
  k_fill_f32<<<gf, RT, 0, st>>>(m, nz, 0.0f);
  k_reg_tet_fwd<<<R.blocks, VS_T, 0, st>>>(verts, tets, sdf, V, (uint32_t)K, ct, m, part);
  if (bwd) {
    k_reg_edge_bwd<<<R.blocks, VS_T, 0, st>>>(edges, n_edges, (uint32_t)edge_cap, V, ce, m, dm, weights,
                                            losses ? part + R.blocks : nullptr);
    k_reg_tet_bwd<<<R.blocks, VS_T, 0, st>>>(verts, tets, sdf, V, (uint32_t)K, ct, dm, weights, dverts, dsdf);
  } else {
    k_reg_edge<<<R.blocks, RT, 0, st>>>(edges, n_edges, (uint32_t)edge_cap, V, m, part + R.blocks);
  }
  if (losses) k_reg_losses<<<1, RT, 0, st>>>(part, R.blocks, losses);
  return hipGetLastError();
}

// The gradient pass after launch_regularizers on the same inputs and
// workspace, whose vertex normals m it reads (the tet pass and the loss sums
// of a second full call cost 37 us of 145 at 1.57 M tets).
hipError_t launch_regularizers_backward(const float* verts, const int32_t* tets, const float* sdf, int32_t V,
                                        int32_t K, const int32_t* edges, const int32_t* n_edges, int64_t edge_cap,
                                        const float* weights, float* dverts, float* dsdf, void* ws,
                                        const RegLayout& R, hipStream_t st) {
  char* w = static_cast<char*>(ws);
  const float* m = reinterpret_cast<const float*>(w + R.o_m);
  float* dm = reinterpret_cast<float*>(w + R.o_dm);
  const size_t nv3 = 3 * (size_t)V;
  const unsigned gf = (unsigned)std::max<size_t>(1, std::min<size_t>((nv3 + RT - 1) / RT, 2048));
  k_reg_clear<<<gf, RT, 0, st>>>(dm, dverts, dsdf, (size_t)V);
  k_reg_edge_bwd<<<R.blocks, VS_T, 0, st>>>(edges, n_edges, (uint32_t)edge_cap, V, reg_chunk((uint64_t)edge_cap), m,
                                            dm, weights, nullptr);
  k_reg_tet_bwd<<<R.blocks, VS_T, 0, st>>>(verts, tets, sdf, V, (uint32_t)K, reg_chunk((uint64_t)K), dm, weights,
                                           dverts, dsdf);
  return hipGetLastError();
}

MTLayout mt_layout(int32_t K, int64_t edge_cap) {
  MTLayout M{};
  M.edge_blocks = ((uint64_t)edge_cap + EDGE_TILE - 1) / EDGE_TILE;
  M.tet_blocks = ((uint64_t)K + EDGE_TILE - 1) / EDGE_TILE;
  M.verts = std::min<uint64_t>((uint64_t)edge_cap, mesh_vertices(K));   // vertices whose first edges the table holds
  size_t o = 0;
  M.o_vid = o; o += al(4 * (size_t)edge_cap);
  M.o_first = o; o += al(4 * (size_t)M.verts);
  M.o_emark = o; o += al(8 * ((size_t)edge_cap / 64 + 1));
  M.o_tmark = o; o += al(32 * ((size_t)K / 64 + 1));
  M.o_bsum_e = o; o += al(4 * ((size_t)M.edge_blocks + 1));
  M.o_bsum_t = o; o += al(4 * ((size_t)M.tet_blocks + 1));
  M.bytes = o;
  return M;
}

hipError_t launch_marching_tets(const float* verts, const int32_t* tets, const float* sdf, int32_t V, int32_t K,
                                const int32_t* edges, const int32_t* n_edges, int64_t edge_cap, float* out_verts,
                                int64_t vert_cap, int32_t* out_tris, int64_t tri_cap, int32_t* counts, void* ws,
                                const MTLayout& M, hipStream_t st) {
  char* w = static_cast<char*>(ws);
  int32_t* vid = reinterpret_cast<int32_t*>(w + M.o_vid);
  uint32_t* first = (uint64_t)V <= M.verts && V > 0 ? reinterpret_cast<uint32_t*>(w + M.o_first) : nullptr;
  uint64_t* emark = reinterpret_cast<uint64_t*>(w + M.o_emark);
  uint64_t* tmark = reinterpret_cast<uint64_t*>(w + M.o_tmark);
  uint32_t* be = reinterpret_cast<uint32_t*>(w + M.o_bsum_e);
  uint32_t* bt = reinterpret_cast<uint32_t*>(w + M.o_bsum_t);
  const unsigned ne = (unsigned)M.edge_blocks, nt = (unsigned)M.tet_blocks;
  const uint32_t ec = (uint32_t)edge_cap;
  const uint32_t vc = (uint32_t)std::min<int64_t>(vert_cap, 0xffffffffll);
  const uint32_t tc = (uint32_t)std::min<int64_t>(tri_cap, 0xffffffffll);
  if (ne > 0) {
    // (a vertex without edges of its own keeps 0xffffffff, past every list)
    if (first) k_fill_u32<<<std::min(((unsigned)V + RT - 1) / RT, 2048u), RT, 0, st>>>(first, (size_t)V, ~0u);
    k_mt_edge_mark<<<ne, RT, 0, st>>>(sdf, V, edges, n_edges, ec, emark, first, be);
  }
  if (nt > 0) k_mt_tet_mark<<<nt, RT, 0, st>>>(tets, sdf, V, (uint32_t)K, tmark, bt);
  k_mt_spines<<<2, 1024, 0, st>>>(be, ne, bt, nt, counts);
  if (ne > 0) k_mt_edge_write<<<ne, RT, 0, st>>>(verts, sdf, edges, n_edges, ec, emark, be, vid, out_verts, vc);
  if (nt > 0)
    k_mt_tet_write<<<nt * (RT / 64), RT, 0, st>>>(verts, tets, (uint32_t)K, edges, n_edges, ec, ne > 0 ? first : nullptr, vid,
                                      tmark, bt, out_tris, tc);
  return hipGetLastError();
}

}  // namespace ts
