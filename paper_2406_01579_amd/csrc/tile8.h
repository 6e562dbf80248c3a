// Helpers shared by the compositing kernels that run one 8x8 pixel tile per
// workgroup (one pixel per lane of each 64-lane wave): the tile's pixel
// coordinates, the lists of the (entry, pixel) pairs to evaluate, and the
// coalesced LDS staging of a chunk of sorted records (8 lanes per 128-byte
// record).
#pragma once

#include "ts_device.h"

namespace ts {
namespace {

// What the forward's evaluation needs of a record: all but the features,
// which go to a table of their own.
struct alignas(16) EvalRec {
  float px[4], py[4], iz[4], f[4], rD[4];
  uint32_t rx, ry, span[2];
};
static_assert(sizeof(EvalRec) == 96 && offsetof(EvalRec, rx) == 80, "six 16-byte parts");

struct Tile8 {
  int view, tile;
  int tx, ty;            // tile coordinates inside the view
  int i, j;              // this lane's pixel
  bool inside;
  uint32_t start, end;   // the tile's entry range
};

// The slot of a workgroup.
__device__ __forceinline__ TileSlot tile_slot(const TileSlot* slots) {
  const auto* p = cmem(slots) + blockIdx.x;
  return TileSlot{p->tile, p->view, p->start, p->end};
}

// sl: the workgroup's slot.  (The caller loads it first of all and starts its
// records' index loads from it before the view's fields are waited for here.)
__device__ __forceinline__ Tile8 tile8(const DevView* vw, const TileSlot& sl) {
  Tile8 c;
  c.tile = (int)sl.tile;
  c.view = (int)sl.view;
  c.start = sl.start;
  c.end = sl.end;
  const auto& V = cmem(vw)[c.view];
  const int lt = c.tile - V.tile_base;
  const int lane = threadIdx.x & 63;
  c.tx = lt % V.tiles_x;
  c.ty = lt / V.tiles_x;
  c.i = c.tx * 8 + (lane & 7);
  c.j = c.ty * 8 + (lane >> 3);
  c.inside = c.i < V.W && c.j < V.H;
  return c;
}

// ---------------------------------------------------------------------------
// Pair packing.  Of the 64 pixels of a tile, a record's pixel rectangle
// usually holds a handful; evaluating one record per wave would leave most
// lanes idle.  Instead each chunk lists the (entry, pixel) pairs whose pixel
// lies in the entry's rectangle and is still live, entry-major, and the
// workgroup's lanes take consecutive pairs.
// ---------------------------------------------------------------------------
// Pixels of the tile (bit = row-major local index) inside R's rectangle.
template <class Rec>
__device__ __forceinline__ uint64_t rect_mask(const Rec& R, const Tile8& c) {
  int i0, i1, j0, j1;
  unpack_rect(R, i0, i1, j0, j1);
  const int x0 = max(i0 - c.tx * 8, 0), x1 = min(i1 - c.tx * 8, 7);
  const int y0 = max(j0 - c.ty * 8, 0), y1 = min(j1 - c.ty * 8, 7);
  if (x0 > x1 || y0 > y1) return 0ull;
  const uint64_t row = (uint64_t)(((2u << x1) - (1u << x0)) & 0xffu);
  const uint64_t rows = (~0ull >> (8 * (7 - y1))) & (~0ull << (8 * y0));
  return (row * 0x0101010101010101ull) & rows;
}

// Of those, the pixels that R's hull may cover (its spans).
template <class Rec>
__device__ __forceinline__ uint64_t hull_mask(const Rec& R, const Tile8& c) {
  int i0, i1, j0, j1;
  unpack_rect(R, i0, i1, j0, j1);
  const int sx = span_shift(i1 - i0 + 1, 4), sy = span_shift(j1 - j0 + 1, 3);
  const int dx = i0 - c.tx * 8, dy = c.ty * 8 - j0;
  uint32_t m[2] = {0u, 0u};
#pragma unroll
  for (int y = 0; y < 8; ++y) {
    const int k = max(dy + y, 0) >> sy;   // (rows outside the rectangle are masked below)
    const uint32_t b = (k < 4 ? R.span[0] : R.span[1]) >> (8 * (k & 3));
    const int xa = max(dx + (int)((b & 15u) << sx), 0), xb = min(dx + (int)((((b >> 4) & 15u) + 1u) << sx), 8);
    const uint32_t row = xa < xb ? (1u << xb) - (1u << xa) : 0u;
    m[y >> 2] |= row << (8 * (y & 3));
  }
  return rect_mask(R, c) & (((uint64_t)m[1] << 32) | m[0]);
}

// Positions of a byte's set bits: the k-th (from 0) in bits [4k, 4k + 3).
struct ByteSelect {
  uint32_t v[256];
};
constexpr ByteSelect make_byte_select() {
  ByteSelect T{};
  for (uint32_t b = 0; b < 256; ++b) {
    uint32_t k = 0;
    for (uint32_t j = 0; j < 8; ++j)
      if ((b >> j) & 1u) T.v[b] |= j << (4 * k++);
  }
  return T;
}
__constant__ ByteSelect c_byte_select = make_byte_select();

// The byte number (sel - 0x0c0c0c00) of the eight bytes hi:lo, and zeros above.
__device__ __forceinline__ uint32_t byte_of(uint64_t x, uint32_t sel) {
  return __builtin_amdgcn_perm((uint32_t)(x >> 32), (uint32_t)x, sel);
}

// Set bits of m in the bytes below each byte (byte 0: none), as eight bytes.
__device__ __forceinline__ uint64_t bits_below(uint64_t m) {
  uint32_t x[2] = {(uint32_t)m, (uint32_t)(m >> 32)};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    x[i] -= (x[i] >> 1) & 0x55555555u;
    x[i] = (x[i] & 0x33333333u) + ((x[i] >> 2) & 0x33333333u);
    x[i] = ((x[i] + (x[i] >> 4)) & 0x0f0f0f0fu) * 0x01010101u;   // up to and with each byte
  }
  x[1] += (x[0] >> 24) * 0x01010101u;
  return ((uint64_t)x[1] << 32 | x[0]) << 8;
}

// Wave 0, lane e < n: m_e is entry e's pair mask.  Writes pmask[0..CH) and
// the exclusive offsets poff[0..CH] of the entries' pairs counted in groups
// of GROUP (poff[n] = number of groups).
template <int CH, int GROUP = 1>
__device__ __forceinline__ void pair_offsets(int n, uint64_t m_e, uint64_t* pmask, uint32_t* poff) {
  const int lane = threadIdx.x & 63;
  const uint64_t m = lane < n ? m_e : 0ull;
  const uint32_t x = wave_scan_add(((uint32_t)__popcll(m) + (GROUP - 1)) / GROUP);
  if (lane < CH) {
    pmask[lane] = m;
    poff[lane + 1] = x;
  }
  if (lane == 0) poff[0] = 0u;
}

// A chunk's pair list, laid out so that a lane finds the entry of its pair
// with a popcount and one LDS read (a binary search over the entries'
// offsets was six dependent LDS reads per pair).  The entries with at least
// one pair are listed in order; per block of 64 consecutive pairs, bstart
// marks the pairs that begin a listed entry and bfirst counts the listed
// entries that begin before the block.  Pair p (block b = p / 64) then
// belongs to listed entry bfirst[b] + (starts in block b at or before p) - 1.
// Its pixel is the mask's bit number p - first: the row is the last one whose
// pixels below number at most that (eight compares in two subtractions, on
// the bytes that pair_map leaves beside the mask), the column a table's.
// (Six halvings of the mask instead: 45 instructions of a pair's 205.)
template <int CH>
struct PairMap {
  uint64_t bstart[CH];   // per block of 64 pairs: bit q set where a listed entry's pairs begin
  ulonglong2 lmask[CH];  // listed entry k: its pixel mask, and its pixels below each row (bytes)
  uint32_t bfirst[CH];   // per block: listed entries beginning before it
  uint32_t lent[CH];     // listed entry k: its chunk index | its first pair << 8
  uint32_t total;        // pairs in the chunk
  uint32_t bsel[256];    // c_byte_select (PairSelect)
};

// The map's table, loaded at the start of a kernel and stored before the
// first barrier.
template <int CH, int NT>
struct PairSelect {
  static constexpr int N = (256 + NT - 1) / NT;
  uint32_t v[N];
  __device__ __forceinline__ void load() {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = c_byte_select.v[(threadIdx.x + NT * i) & 255u];
  }
  __device__ __forceinline__ void store(PairMap<CH>& M) const {
#pragma unroll
    for (int i = 0; i < N; ++i) M.bsel[(threadIdx.x + NT * i) & 255u] = v[i];
  }
};

// Wave 0, lane e < n: m_e is entry e's pixel mask.  Every lane of the wave
// must call it; the map is complete after the next barrier.
template <int CH>
__device__ __forceinline__ void pair_map(int n, uint64_t m_e, PairMap<CH>& M) {
  static_assert(CH <= 64, "one lane per entry");
  const int lane = threadIdx.x & 63;
  const uint64_t m = lane < n ? m_e : 0ull;
  const uint32_t cnt = (uint32_t)__popcll(m);
  const uint32_t x = wave_scan_add(cnt);
  const uint32_t first = x - cnt;
  const uint32_t k = (uint32_t)__popcll(__ballot(m != 0ull) & ((1ull << lane) - 1ull));
  // the pairs fill at most CH blocks; this wave's own LDS operations take
  // effect in program order, so the clear lands before the marks
  if (lane < CH) M.bstart[lane] = 0ull;
  __builtin_amdgcn_wave_barrier();
  if (m != 0ull) {
    M.lmask[k] = make_ulonglong2(m, bits_below(m));
    M.lent[k] = (uint32_t)lane | (first << 8);
    atomicOr(&M.bstart[first >> 6], 1ull << (first & 63u));
  }
  __builtin_amdgcn_wave_barrier();
  const uint64_t bs = lane < CH ? M.bstart[lane] : 0ull;
  const uint32_t bc = (uint32_t)__popcll(bs);
  const uint32_t y = wave_scan_add(bc);
  if (lane < CH) M.bfirst[lane] = y - bc;
  if (lane == 63) M.total = x;
}

// Wave 0, lane e < n: entry e's pairs are the pixels its hull may cover, in
// live_e (the pixels that still take part for that entry).
template <int CH, class Rec>
__device__ __forceinline__ void chunk_pairs(const Rec* recs, int n, const Tile8& c, uint64_t live_e,
                                            PairMap<CH>& M) {
  const int lane = threadIdx.x & 63;
  pair_map<CH>(n, lane < n ? hull_mask(recs[lane], c) & live_e : 0ull, M);
}

// All threads: f(e, x, y) for every listed pair (entry e, the tile's pixel
// (x, y)), entry-major, pixels in ascending order inside an entry.
template <int CH, class F>
__device__ __forceinline__ void for_each_pair(const PairMap<CH>& M, int nthreads, F&& f) {
  const uint32_t total = M.total;
  for (uint32_t p = threadIdx.x; p < total; p += (uint32_t)nthreads) {
    const uint32_t b = p >> 6;
    // pair 0 begins the first listed entry, so at least one start lies at or before p
    const uint32_t k = M.bfirst[b] + (uint32_t)__popcll(M.bstart[b] & (~0ull >> (63u - (p & 63u)))) - 1u;
    const uint32_t le = M.lent[k], j = p - (le >> 8);
    const ulonglong2 m = M.lmask[k];
    // per byte, the top bit: at most j pixels below the row (j, its pixels < 128)
    const uint32_t jj = __builtin_amdgcn_perm(0u, j, 0u) | 0x80808080u;
    const uint32_t rows = (uint32_t)__popc((jj - (uint32_t)m.y) & 0x80808080u) +
                          (uint32_t)__popc((jj - (uint32_t)(m.y >> 32)) & 0x80808080u);
    const uint32_t sel = rows + (0x0c0c0c00u - 1u);
    const uint32_t x = M.bsel[byte_of(m.x, sel)] >> (4u * (j - byte_of(m.y, sel)));
    f((int)(le & 0xffu), (int)(x & 7u), (int)(rows - 1u));
  }
}

// Software pipeline of the chunk loads: while a chunk is processed, the next
// chunk's records are in flight into registers and the record indices of the
// one after it are in flight too, so a chunk's two dependent global loads
// overlap the previous chunk's work.  Each thread owns PQ of the chunk's
// 16-byte record parts.  With E0, the copy's first-entry field comes from
// the records' first entries (loaded beside the last part).
template <int CH, int NT, bool E0 = false>
struct RecPipe {
  static constexpr int PQ = (CH * 8 + NT - 1) / NT;
  uint32_t idx[PQ];
  uint32_t cur[PQ];                      // the record indices of the parts in flight
  float vx[PQ], vy[PQ], vz[PQ], vw[PQ];  // scalars, so the parts stay in registers
  // The chunk of entries from b, cut at hi (a valid entry): a part past hi
  // loads entry hi's index again.  Callers issue every load of the pipeline
  // unconditionally (past the list: its last entry, cached and never
  // stored), so no register is given a default while an older load into it
  // may be in flight, a wait that would also cover the loads just issued.
  __device__ __forceinline__ void fetch_idx(const uint32_t* __restrict__ srec, uint32_t b, uint32_t hi) {
#pragma unroll
    for (int j = 0; j < PQ; ++j) {
      const int q = (int)threadIdx.x + j * NT;
      idx[j] = srec[min(b + (uint32_t)(q >> 3), hi)];
    }
  }
  // every part (one past the chunk reads a record of the list, never stored)
  __device__ __forceinline__ void fetch_rec(const ViewRec* __restrict__ vrec,
                                            const uint32_t* __restrict__ rfirst = nullptr) {
#pragma unroll
    for (int j = 0; j < PQ; ++j) {
      const int q = (int)threadIdx.x + j * NT;
      cur[j] = idx[j];
      const float4 t = reinterpret_cast<const float4*>(vrec)[(size_t)idx[j] * 8 + (size_t)(q & 7)];
      vx[j] = t.x;
      vy[j] = t.y;
      vz[j] = t.z;
      vw[j] = t.w;
      if (E0 && (q & 7) == 7) vw[j] = __uint_as_float(rfirst[idx[j]]);   // entry0: the record's last word
    }
  }
  // The blended features (c, zt, n: parts 5 and 6) also go to a table of
  // their own, whose per-lane gathers have no bank conflicts.  With ridx, so
  // does each record's index (what a chunk needs of srec later comes from LDS
  // then, not from a global load on its critical path).
  __device__ __forceinline__ void store(EvalRec* recs, int n, float (*feat)[CH]) const {
#pragma unroll
    for (int j = 0; j < PQ; ++j) {
      const int q = (int)threadIdx.x + j * NT;
      if (q < n * 8) {
        const int e = q >> 3, part = q & 7;
        float4* d = reinterpret_cast<float4*>(&recs[e]);
        if (part < 5) {
          d[part] = make_float4(vx[j], vy[j], vz[j], vw[j]);
        } else if (part == 5) {
          feat[0][e] = vx[j];
          feat[1][e] = vy[j];
          feat[2][e] = vz[j];
          feat[3][e] = vw[j];
        } else if (part == 6) {
          feat[4][e] = vx[j];
          feat[5][e] = vy[j];
          feat[6][e] = vz[j];
          recs[e].rx = __float_as_uint(vw[j]);
        } else {
          recs[e].ry = __float_as_uint(vx[j]);
          recs[e].span[0] = __float_as_uint(vy[j]);
          recs[e].span[1] = __float_as_uint(vz[j]);
        }
      }
    }
  }
  __device__ __forceinline__ void store(ViewRec* recs, int n, float (*feat)[CH], uint32_t* ridx = nullptr) const {
#pragma unroll
    for (int j = 0; j < PQ; ++j) {
      const int q = (int)threadIdx.x + j * NT;
      if (q < n * 8) {
        reinterpret_cast<float4*>(&recs[q >> 3])[q & 7] = make_float4(vx[j], vy[j], vz[j], vw[j]);
        const int e = q >> 3, part = q & 7;
        if (part == 5) {
          feat[0][e] = vx[j];
          feat[1][e] = vy[j];
          feat[2][e] = vz[j];
          feat[3][e] = vw[j];
        } else if (part == 6) {
          feat[4][e] = vx[j];
          feat[5][e] = vy[j];
          feat[6][e] = vz[j];
        } else if (ridx && part == 0) {
          ridx[e] = cur[j];
        }
      }
    }
  }
};

}  // namespace
}  // namespace ts
