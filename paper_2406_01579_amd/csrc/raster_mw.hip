// Multi-wave compositing kernels for 8x8 tiles.
//
// A tile's entry list is walked front to back (forward) or back to front
// (backward) by one pixel per lane, and the per-pixel state along the list
// (transmittance, the colour behind) is a short sequential recurrence.  The
// expensive part of every (pixel, entry) pair -- coverage of the projected
// hull, entry/exit SDF values and Eq. 1 -- does not depend on that state.
// So NWV waves share one 8x8 tile: for each LDS chunk of entries they
// evaluate the (entry, pixel) pairs that can hit in parallel into LDS, and one
// wave runs the recurrence over the chunk.  The backward's recurrence leaves,
// per blended pair, dL/df_prev, dL/df_next and the blend weight in a pair
// buffer, grouped per (tile, entry) segment; a second, flat kernel chains
// every pair to its record's 23 screen-space parameters and sums each
// segment, with no per-tile sequence and no atomics.  The forward counts
// each tile's blended pairs and segments so that every backward workgroup
// knows where its pairs go.  Images are bit-identical to the one-wave kernels
// (the same per-pair arithmetic in the same order).
#include "tile8.h"

namespace ts {

namespace {


// The blended features of a pixel (c, zt, n and the opacity, a feature of 1)
// are eight sums that only add up what the recurrence has decided.  They are
// left to waves other than the recurrence's, FeatSums::N of them with G sums
// each per pixel, which add a chunk's terms, in the pixel's order, while the
// first wave lists the next chunk's pairs (with the next alpha read ahead in
// the recurrence: forward 76 to 73 us at 4 x 512^2, 695 to 684 us at
// 8 x 1024^2).
template <int NWV>
struct FeatSums {
  static constexpr int N = NWV >= 4 ? 2 : 1, G = 8 / N, W0 = NWV > 1 ? 1 : 0;   // waves W0 .. W0 + N - 1
};
constexpr int FEATS = 8;

// Forward sweep over [start, end) with NWV waves; wave 0 ends with the
// pixel's blend state, and with ACC the waves of FeatSums with its sums.  Used
// by the forward kernel and by the backward's state replay.  rp: the first
// chunk's indexes are in flight.
//   Per chunk: the records into LDS; the first wave lists the pairs that may
// hit; all waves evaluate them; the first wave runs the recurrence.  Both
// one-wave phases are as short as they can be made: the recurrence decides who
// blends and with what weight (left in place of alpha), and nothing else.
//   A tile takes some 14 us at 8 x 1024^2 (five workgroups per CU): 2 until its
// slot and view are there, 1.5 until its first records are, then 5.5 a chunk of
// 64 (5 to 6.5 k of 13 k cycles the evaluation, 4 k before its split the
// recurrence, 2.6 k the pair list).  VALU issue 60 to 70% busy.  Chunks of 32
// and 48 at six workgroups per CU: 67 and 63 us against 64 at 4 x 512^2, 613 and
// 565 against 579 at 8 x 1024^2, one frame 31 and 26 against 25.
template <int NWV, int CHN, bool ACC, class Rec>
__device__ __forceinline__ void forward_sweep(RecPipe<CHN, 64 * NWV>& rp, const ViewRec* __restrict__ vrec,
                                              const uint32_t* __restrict__ srec, uint32_t start, uint32_t end,
                                              const Tile8& c, float s, float alpha_min, float alpha_clamp, float t_min,
                                              Rec* recs, float (*alds)[64], PairMap<CHN>& pm, uint64_t* hm,
                                              float (*feat)[CHN] /* FEATS rows, twice with ACC */,
                                              unsigned long long* done_mask, float& T, float& Tb, int& last,
                                              uint32_t& nblend, float (&acc)[FeatSums<NWV>::G],
                                              unsigned long long* bmask = nullptr,
                                              unsigned long long* bml = nullptr) {
  constexpr int NT = 64 * NWV;
  using FS = FeatSums<NWV>;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bool done = !c.inside;
  if (wave == 0) {
    const unsigned long long m = __ballot(done);
    if (lane == 0) *done_mask = m;
  }
  if (start < end) {
    rp.fetch_rec(vrec);
    rp.fetch_idx(srec, start + CHN, end - 1);
  }
  // the last chunk's blended entries per pixel are still in LDS: the last wave
  // turns them into the pixels per entry (what the backward's pairs are) and
  // writes these out (not before the next chunk's wait for its loads: loads and
  // stores share one counter), the waves of FeatSums add their terms
  uint32_t mbase = start;
  int mn = 0;
  const auto finish_chunk = [&] {
    if (mn == 0) return;
    if (bmask && wave == NWV - 1) {
      const uint64_t m = wave_transpose64(bml[lane]);
      if (lane < mn) bmask[mbase + lane] = m;
    }
    if (ACC && wave >= FS::W0 && wave < FS::W0 + FS::N) {
      const float(*ft)[CHN] = feat + ((mbase - start) / CHN & 1u) * FEATS + (wave - FS::W0) * FS::G;
      uint64_t b = bml[lane];
      while (__ballot(b != 0ull) != 0ull) {
        if (b != 0ull) {
          const int e = __ffsll((unsigned long long)b) - 1;
          b &= b - 1ull;
          const float w = alds[e][lane];
#pragma unroll
          for (int k = 0; k < FS::G; ++k) acc[k] = fmaf(w, ft[k][e], acc[k]);
        }
      }
    }
  };
  for (uint32_t base = start; base < end; base += CHN) {
    __syncthreads();
    if (*done_mask == ~0ull) break;
    const int n = (int)min((uint32_t)CHN, end - base);
    rp.store(recs, n, ACC ? feat + ((base - start) / CHN & 1u) * FEATS : feat);
    rp.fetch_rec(vrec);
    rp.fetch_idx(srec, base + 2 * CHN, end - 1);
    __syncthreads();
    // phase A: coverage and Eq. 1 of the live (entry, pixel) pairs, packed;
    // hm[pixel] collects the chunk entries the pixel may blend
    if (wave == NWV - 1) hm[lane] = 0ull;
    if (wave == 0) chunk_pairs<CHN>(recs, n, c, ~*done_mask, pm);
    finish_chunk();
    __syncthreads();
    for_each_pair<CHN>(pm, NT, [&](int e, int x, int y) {
      const float qx = (float)(c.tx * 8 + x) + 0.5f, qy = (float)(c.ty * 8 + y) + 0.5f;
      PixHit h;
      if (pixel_hit(recs[e], qx, qy, s, h) && h.alpha >= alpha_min) {
        const int pix = y * 8 + x;
        alds[e][pix] = h.alpha;
        atomicOr(&hm[pix], 1ull << e);
      }
    });
    __syncthreads();
    if (wave == 0) {
      // each pixel visits only its candidate entries, front to back; the next
      // one's alpha is read before this one is decided
      uint64_t cand = done ? 0ull : hm[lane];
      uint64_t blended = 0ull;   // this lane's blended entries of the chunk
      int e = (__ffsll((unsigned long long)cand) - 1) & 63;
      float araw = alds[e & (CHN - 1)][lane];
      while (__ballot(cand != 0ull) != 0ull) {
        if (cand != 0ull) {
          cand &= cand - 1ull;
          const int en = (__ffsll((unsigned long long)cand) - 1) & 63;
          const float anext = alds[en & (CHN - 1)][lane];
          const float a = fminf(araw, alpha_clamp);
          const float Tn = T * (1.0f - a);
          if (Tn < t_min) {
            done = true;
          } else {
            if (ACC) alds[e][lane] = T * a;   // the blend weight
            Tb = T;
            T = Tn;
            blended |= 1ull << e;
            if (T == 0.0f) done = true;
          }
          if (done) cand = 0ull;
          e = en;
          araw = anext;
        }
      }
      if (blended != 0ull) last = (int)base + 63 - __clzll((long long)blended);
      nblend += (uint32_t)__popcll(blended);   // the chunk's blended pairs (per lane)
      if (ACC) bml[lane] = blended;
      const unsigned long long m = __ballot(done);
      if (lane == 0) *done_mask = m;
    }
    mbase = base;
    mn = n;
  }
  if (ACC && wave == 0) reinterpret_cast<float*>(hm)[lane] = T;   // for whoever writes the sums
  __syncthreads();
  finish_chunk();
}

// Background of `count` tiles with an empty list (the dispatch slots from
// `first`; a workgroup takes up to EMPTY_PER_WG of them): the outputs of a
// pixel no record reaches (T = 1), no blended entry, and the tile's end of
// blended prefix at its start.
constexpr uint32_t EMPTY_PER_WG = 16;
template <int NT>
__device__ __forceinline__ void background_tiles(void* ws, const Layout& L, const DevView* vw, uint32_t first,
                                                 uint32_t count) {
  const TileSlot* slots = at<const TileSlot>(ws, L.o_tile_order);
  uint32_t* tpend = at<uint32_t>(ws, L.o_tile_pend);
  int32_t* last_out = at<int32_t>(ws, L.o_last);
  float* tlast_out = at<float>(ws, L.o_tlast);
  for (uint32_t q = threadIdx.x; q < count * 64u; q += NT) {
    const uint32_t slot = first + (q >> 6);
    const int pix = (int)(q & 63u);
    const TileSlot sl = slots[slot];
    const DevView& V = vw[sl.view];
    if (pix == 0) tpend[slot] = sl.start;
    const int lt = (int)sl.tile - V.tile_base;
    const int i = (lt % V.tiles_x) * 8 + (pix & 7), j = (lt / V.tiles_x) * 8 + (pix >> 3);
    if (i >= V.W || j >= V.H) continue;
    const size_t plane = (size_t)V.W * V.H;
    const size_t px = (size_t)j * V.W + i;
    auto* out = gmem(V.out);
    out[0 * plane + px] = V.bg[0];
    out[1 * plane + px] = V.bg[1];
    out[2 * plane + px] = V.bg[2];
#pragma unroll
    for (int k = 3; k < 8; ++k) out[k * plane + px] = 0.0f;
    if (keeps_pixel_state(L)) {
      const size_t g = (size_t)V.pix_base + px;
      last_out[g] = -1;
      tlast_out[g] = 1.0f;
    }
  }
}

}  // namespace

template <int NWV, int CHN>
__global__ __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_composite_mw(void* ws, Layout L, float alpha_min, float alpha_clamp,
                                                           float t_min) {
  const DevView* vw = at<const DevView>(ws, L.o_view);
  const uint32_t* srec = at<const uint32_t>(ws, blend_entry_records(L));
  const ViewRec* vrec = at<const ViewRec>(ws, L.o_vrec);
  int32_t* last_out = at<int32_t>(ws, L.o_last);
  float* tlast_out = at<float>(ws, L.o_tlast);
  __shared__ EvalRec recs[CHN];
  __shared__ float alds[CHN][64];
  __shared__ PairMap<CHN> pm;
  __shared__ uint64_t hm[64];
  __shared__ float feat[2 * FEATS][CHN];   // a chunk's features, and the last one's: c, zt, n and 1
  __shared__ unsigned long long bml[64];
  __shared__ unsigned long long done_mask;

  // a tile has some two chunks, so the chain of loads before the first counts:
  // the slot, then the first records' indexes, then whatever the view gives
  const TileSlot sl = tile_slot(at<const TileSlot>(ws, L.o_tile_order));
  // the tiles with an empty list take the last slots (length bucket 0):
  // workgroups past the others write their background, EMPTY_PER_WG tiles
  // each, and the rest of the grid leaves at once
  {
    const uint32_t n_empty = *cmem(at<const uint32_t>(ws, L.o_tile_hist));
    const uint32_t n_work = (uint32_t)L.total_tiles - n_empty;
    if (blockIdx.x >= n_work) {
      const uint32_t first = n_work + (blockIdx.x - n_work) * EMPTY_PER_WG;
      if (first < (uint32_t)L.total_tiles)
        background_tiles<64 * NWV>(ws, L, vw, first, min(EMPTY_PER_WG, (uint32_t)L.total_tiles - first));
      return;
    }
  }
  PairSelect<CHN, 64 * NWV> ps;
  RecPipe<CHN, 64 * NWV> rp;
  ps.load();
  if (sl.start < sl.end) rp.fetch_idx(srec, sl.start, sl.end - 1);
  const Tile8 c = tile8(vw, sl);
  ps.store(pm);
  for (int q = threadIdx.x; q < 2 * CHN; q += 64 * NWV) feat[q < CHN ? FEATS - 1 : 2 * FEATS - 1][q % CHN] = 1.0f;
  const auto& V = cmem(vw)[c.view];
  const float s = V.s;
  // what the end needs of the view, loaded here (not behind the sweep's stores)
  const size_t plane = (size_t)V.W * V.H;
  const size_t px = (size_t)c.j * V.W + c.i;
  const float bg[3] = {V.bg[0], V.bg[1], V.bg[2]};
  const int32_t pix_base = V.pix_base;
  auto* out = gmem(V.out);
  const uint32_t start = c.start, end = c.end;
  float T = 1.0f, Tb = 1.0f;
  using FS = FeatSums<NWV>;
  float acc[FS::G] = {};
  int last = -1;
  uint32_t nblend = 0;
  const bool count = L.o_pairs != 0;
  forward_sweep<NWV, CHN, true>(rp, vrec, srec, start, end, c, s, alpha_min, alpha_clamp, t_min, recs, alds, pm, hm,
                                feat, &done_mask, T, Tb, last, nblend, acc,
                                L.o_bmask ? at<unsigned long long>(ws, L.o_bmask) : nullptr, bml);
  // the pixel's state, before the atomics below (a load after them would be
  // waited for with them, 2 us of a tile's 14)
  if ((threadIdx.x >> 6) == 0 && c.inside && keeps_pixel_state(L)) {
    const size_t g = (size_t)pix_base + px;
    last_out[g] = last < 0 ? -1 : (int)at<const uint32_t>(ws, blend_entry_index(L))[last];
    tlast_out[g] = Tb;
  }
  if ((threadIdx.x >> 6) == 0) {
    // end of the tile's blended prefix: where the backward starts its walk
    const uint32_t pend = wave_max((uint32_t)(last + 1 > (int)start ? last + 1 : (int)start));
    nblend = wave_scan_add(nblend);
    if ((threadIdx.x & 63) == 63) {
      at<uint32_t>(ws, L.o_tile_pend)[blockIdx.x] = pend;
      if (count) at<uint32_t>(ws, L.o_slot_pairs)[blockIdx.x] = nblend;
      // the backward dispatch order's histograms of walked lengths and of
      // blended pairs (bucket 0, nothing walked, is not counted)
      if (pend > start) {
        uint32_t* bh = at<uint32_t>(ws, L.o_bwd_hist);
        const int b = len_bucket(pend - start);
        atomicAdd(bh + b, 1u);
        if (count) {
          atomicAdd(bh + 2 * TILE_BUCKETS + b, nblend);
          atomicAdd((unsigned long long*)&at<DevHeader>(ws, L.o_hdr)->pairs_needed, (unsigned long long)nblend);
        }
      }
    }
  }
  const int wave = threadIdx.x >> 6;
  if (wave >= FS::W0 && wave < FS::W0 + FS::N && c.inside) {
    const float Tend = reinterpret_cast<const float*>(hm)[threadIdx.x & 63];
    const int f0 = (wave - FS::W0) * FS::G;
#pragma unroll
    for (int k = 0; k < FS::G; ++k) {
      // features c, zt, n and the opacity to the planes c, opacity, zt, n
      const int f = f0 + k, p = f < 3 ? f : f < 7 ? f + 1 : 3;
      out[p * plane + px] = f < 3 ? fmaf(Tend, f == 0 ? bg[0] : f == 1 ? bg[1] : bg[2], acc[k]) : acc[k];
    }
  }
}

// Backward, walk and recurrence: per chunk, faces and Eq. 1 of every (entry,
// pixel) that the forward blended (its masks), packed, then the reverse
// recurrence of Eq. 2 (one wave).  Every blended pair's dL/df_prev,
// dL/df_next and blend weight go to the pair buffer, entry-major inside the
// chunk, and every entry with a blended pixel gets a segment (its record, its
// per-(record, tile) gradient slot, its first pair and pair count); the
// tile's pairs and segments start at the bases the forward's counts gave
// this backward slot.
//   Bound by its one-wave phase: of 8.3 k cycles a chunk of 32 the recurrence
// with the pairs' writes is 3.7 k, the evaluation 2 k, the lists 1 k.  With the
// transpose, the pairs' places and the entries per pixel taken by other waves:
// 69 to 62 us at 4 x 512^2.  (The first wave without any load, so that it never
// waits for its own stores: 67 us at the same five waves per SIMD; six waves
// per SIMD: 64.)
template <int NWV, int CHB>
__global__ __launch_bounds__(64 * NWV) void k_composite_bwd_mw(void* ws, Layout L, float alpha_min,
                                                               float alpha_clamp, float t_min, int recompute) {
  static_assert(CHB <= 32, "a pixel's chunk candidates are a 32-bit mask");
  constexpr int NT = 64 * NWV;
  const DevView* vw = at<const DevView>(ws, L.o_view);
  const uint32_t* srec = at<const uint32_t>(ws, blend_entry_records(L));
  const ViewRec* vrec = at<const ViewRec>(ws, L.o_vrec);
  const float* tlast_in = at<const float>(ws, L.o_tlast);
  const unsigned long long* bmask = at<const unsigned long long>(ws, L.o_bmask);
  uint4* pairs = at<uint4>(ws, L.o_pairs);
  __shared__ ViewRec recs[CHB];
  __shared__ uint4 eseg[CHB];        // per entry with a blended pixel: record, view, tile, gradient slot
  __shared__ uint32_t ridx[CHB];     // per entry: its record
  __shared__ float abuf[CHB][64];    // raw alpha
  __shared__ float e2buf[CHB][64];   // exp(s f_next)
  __shared__ uint8_t sel[CHB][64];   // entry face | exit face << 2
  __shared__ PairMap<CHB> pm;        // phase A's pairs
  __shared__ uint64_t pmask[CHB];    // phase B: per entry, the pixels that blended it
  __shared__ uint32_t poff[CHB + 1]; // and the places of its pairs
  __shared__ uint64_t hmask[64];     // per pixel: chunk entries it may have blended (bit e)
  __shared__ float feat[7][CHB];     // per entry: c[3], zt, n[3] (conflict-free gathers)
  __shared__ unsigned long long done_mask;
  __shared__ int smax;

  // dispatch order by the length the forward walked (longest first); the
  // tiles where nothing was blended come last and leave at once
  const TileSlot* bslots = at<const TileSlot>(ws, L.o_bwd_order);
  const TileSlot sl = tile_slot(bslots);
  const uint32_t pend_f = cmem(at<const uint32_t>(ws, L.o_bwd_pend))[blockIdx.x];
  // where this tile's pairs go
  uint32_t pair_run = cmem(at<const uint32_t>(ws, L.o_bwd_base))[blockIdx.x];
  if (!recompute && (blockIdx.x >= cmem(at<const DevHeader>(ws, L.o_hdr))->bwd_work || pend_f == sl.start)) return;
  const uint32_t start = sl.start, end = sl.end;
  const unsigned lane = threadIdx.x & 63u;
  const int wave = threadIdx.x >> 6;
  const uint64_t cap = (uint64_t)L.entry_cap;
  const uint32_t* rfirst = at<const uint32_t>(ws, L.o_rfirst);

  // The chunks run from the one holding pend - 1 down to start; only the first
  // is partial.  pend: end of the tile's blended prefix (from the forward, or
  // the replay).
  RecPipe<CHB, NT, true> rp;
  // lane e of the waves that work on masks: the blend mask of the current
  // chunk's entry e, and of the next chunk's (its load in flight across the
  // current chunk)
  const bool masks = (wave == 0 || wave == NWV / 2 || wave == NWV - 1) && lane < (unsigned)CHB;
  uint64_t bm_cur = 0ull, bm_next = 0ull;
  uint32_t pend = pend_f;
  const auto last_chunk = [&] { return (int64_t)start + (((int64_t)pend - 1 - (int64_t)start) / CHB) * CHB; };
  // The loads before the first chunk are a chain that a tile's few chunks have
  // to carry (it was a third of their time): the slot, the first records'
  // indexes, the records, and beside those two whatever the view leads to.
  const auto first_idx = [&] {
    const uint32_t b = (uint32_t)last_chunk();
    rp.fetch_idx(srec, b, pend - 1u);
    if (masks && lane < pend - b) bm_next = bmask[b + lane];
  };
  if (!recompute) first_idx();
  PairSelect<CHB, NT> ps;
  ps.load();
  const Tile8 c = tile8(vw, sl);
  const auto& V = cmem(vw)[c.view];
  const float s = V.s;
  const size_t plane = (size_t)V.W * V.H;
  const size_t px = c.inside ? (size_t)c.j * V.W + c.i : 0;
  const float bg[3] = {V.bg[0], V.bg[1], V.bg[2]};
  const size_t pix_base = (size_t)V.pix_base;
  const auto* dout = gmem(V.dout);
  ps.store(pm);

  // per-pixel state (wave 0): T before the last blend, upstream gradient
  int last = -1;
  float Tb = 1.0f;
  if (recompute) {
    float T = 1.0f;
    float acc[FeatSums<NWV>::G];
    uint32_t nb_unused = 0;
    RecPipe<CHB, NT> rq;
    if (start < end) rq.fetch_idx(srec, start, end - 1);
    forward_sweep<NWV, CHB, false>(rq, vrec, srec, start, end, c, s, alpha_min, alpha_clamp, t_min, recs, abuf, pm,
                                   hmask, feat, &done_mask, T, Tb, last, nb_unused, acc);
    if (wave == 0) {
      const uint32_t w = wave_max((uint32_t)(last + 1 > (int)start ? last + 1 : (int)start));
      if (lane == 63u) smax = (int)w;
    }
    __syncthreads();
    pend = (uint32_t)smax;
    if (pend > start) first_idx();
  }
  // the chunk starting at b, or below the list the entry pend - 1 again
  const auto below = [&](int64_t b) { return b >= (int64_t)start ? (uint32_t)b : pend - 1u; };
  const int64_t cb0 = last_chunk();
  if (pend > start) {
    rp.fetch_rec(vrec, rfirst);
    rp.fetch_idx(srec, below(cb0 - CHB), pend - 1u);
  }
  // (no load under a lane's condition, but at pixel 0 for a lane outside: each
  // was waited for before the next, eight in a row, 8 to 12 k cycles)
  float gr[8];
  if (wave == 0) {
    float tl = 1.0f;
    if (!recompute) tl = tlast_in[pix_base + px];
#pragma unroll
    for (int q = 0; q < 8; ++q) gr[q] = dout[q * plane + px];
    if (!recompute && c.inside) Tb = tl;
#pragma unroll
    for (int q = 0; q < 8; ++q) gr[q] = c.inside ? gr[q] : 0.0f;
  }
  float Rbehind = 0.0f;   // (before the first chunk's recurrence: gr . background)
  const uint32_t tile_xy = (uint32_t)c.tx | ((uint32_t)c.ty << 16);

  bool first = true;
  float Tnext = 1.0f;
  for (int64_t cb = cb0; cb >= (int64_t)start && pend > start; cb -= CHB) {
    const uint32_t base = (uint32_t)cb;
    const int n = (int)min((uint32_t)CHB, pend - base);
    __syncthreads();
    // the next masks' load is issued before the next records', so taking
    // over the current masks (a wait for their load, a chunk old) does not
    // also wait for the record loads just issued
    bm_cur = bm_next;
    if (masks && cb - CHB >= (int64_t)start) bm_next = bmask[base - CHB + lane];
    rp.store(recs, n, feat, ridx);
    rp.fetch_rec(vrec, rfirst);
    rp.fetch_idx(srec, below(cb - 2 * CHB), pend - 1u);
    __syncthreads();
    // from the masks (lane e: the pixels that blended entry e), a wave each
    // where there are as many: the chunk's pair list, every pixel's entries,
    // and the places of the pairs with what every pair of an entry carries
    if (wave == 0) pair_map<CHB>(n, bm_cur, pm);
    if (wave == NWV - 1) hmask[lane] = (uint32_t)wave_transpose64((int)lane < n ? bm_cur : 0ull);
    if (wave == NWV / 2) {
      pair_offsets<CHB, 1>(n, bm_cur, pmask, poff);
      if ((int)lane < n && bm_cur != 0ull) {
        const ViewRec& R = recs[lane];
        int i0, i1, j0, j1;
        unpack_rect(R, i0, i1, j0, j1);
        const int tx0 = i0 >> 3, ty0 = j0 >> 3, nx = (i1 >> 3) - tx0 + 1;
        const uint32_t d = R.entry0 + (uint32_t)((c.ty - ty0) * nx + (c.tx - tx0));
        eseg[lane] = make_uint4(ridx[lane], (uint32_t)c.view, tile_xy, d);
      }
    }
    __syncthreads();
    // phase A: faces and Eq. 1 of every pair, packed
    for_each_pair<CHB>(pm, NT, [&](int e, int x, int y) {
      const float px_ = (float)(c.tx * 8 + x) + 0.5f, py_ = (float)(c.ty * 8 + y) + 0.5f;
      PixHit h;
      (void)pixel_hit(recs[e], px_, py_, s, h);   // (the forward found that it hits)
      const int pix = y * 8 + x;
      abuf[e][pix] = h.alpha;
      e2buf[e][pix] = h.e2;
      sel[e][pix] = (uint8_t)h.faces;
    });
    __syncthreads();
    // phase B (wave 0): the reverse recurrence writes each pair
    if (wave == 0) {
      const uint32_t m0 = (uint32_t)hmask[lane];   // CHB <= 32 entries
      if (cb == cb0) Rbehind = gr[0] * bg[0] + gr[1] * bg[1] + gr[2] * bg[2];
      const uint64_t lt = (1ull << lane) - 1ull;
      // each pixel visits only the entries it blended, nearest-last first
      uint32_t m = m0;
      while (__ballot(m != 0u) != 0ull) {
        if (m != 0u) {
          const int e = 31 - __clz(m);
          m ^= 1u << e;
          const float araw = abuf[e][lane];
          const float e2 = e2buf[e][lane];
          const float a = fminf(araw, alpha_clamp);
          const float T = first ? Tb : Tnext * rcp(1.0f - a);
          first = false;
          Tnext = T;
          const float sdot = gr[0] * feat[0][e] + gr[1] * feat[1][e] + gr[2] * feat[2][e] + gr[3] +
                             gr[4] * feat[3][e] + gr[5] * feat[4][e] + gr[6] * feat[5][e] + gr[7] * feat[6][e];
          const float da = araw > alpha_clamp ? 0.0f : T * (sdot - Rbehind);
          Rbehind = a * sdot + (1.0f - a) * Rbehind;
          // dL/dalpha chained through Eq. 1 to the entry and exit SDF values
          float dd, dfn;
          eq1_chain(da, araw, e2, s, dd, dfn);
          const uint64_t below = pmask[e] & lt;
          const uint32_t pi = pair_run + poff[e] + (uint32_t)__popcll(below);
          if ((uint64_t)pi < cap) {
            // the segment's first pair carries its pair count
            const uint32_t hw = below == 0ull ? PAIR_HEAD | ((uint32_t)__popcll(pmask[e]) << 11) : 0u;
            pairs[2 * (size_t)pi] = make_uint4(__float_as_uint(dd), __float_as_uint(dfn), __float_as_uint(T * a),
                                               lane | ((uint32_t)sel[e][lane] << 6) | hw);
            pairs[2 * (size_t)pi + 1] = eseg[e];
          }
        }
      }
      pair_run += poff[n];
    }
  }
}

// Backward, per-pair gradients, flat over the pair buffer: each workgroup
// pass takes a window of PG_W consecutive pairs, one per lane.  A lane chains
// its pair to the record's 23 screen-space parameters (colour, depth and
// normal enter linearly with the blend weight; the entry and exit faces
// through App. A.1-A.2) and leaves them in an LDS row; everything it needs
// comes with the pair (one load) and then the record and the view's
// upstream gradient (a second).  The segments whose first pair lies in the
// window are then summed there in a fixed order, a segment per half wave and
// a parameter per lane, into the segment's gradient slot (flagged as reached)
// or, with per-record gradients, added to the record's accumulator.  Only the
// window's last segment runs past it, by at most 63 pairs: the workgroup's
// last wave takes the pairs after the window up to the next segment's first
// pair, and the first wave skips the pairs before the window's first segment,
// which the previous window takes.  Fixed order throughout: reproducible
// bitwise.
//   Bound by VALU issue (61% of its cycles; a pair is some 280 instructions)
// and the pairs' own 32 bytes.  Eight waves of which one takes the tail: with
// four, of which the first took the tail after its own pairs, a fifth of the
// instructions worked for a few lanes and the rest waited for it.  With the
// four faces' products shared (pair_grad_all) and the sums per half wave: 55
// to 38 us for 1.8 M pairs, 818 to 571 us for 27 M (1.5 TB/s of pairs alone).
// (Earlier layouts: a 4-lane group per segment left most lanes idle behind a
// wave's longest segment, 47 us at the training shape against 48 then; one
// workgroup per tile summing its segments through LDS in rounds, 68 us; pairs
// that reached their record and tile through a segment table, 55 us.)
constexpr int PG_T = 512;          // threads: one pair each
constexpr int PG_TAIL = 64;        // the last wave: the last segment's pairs past the window
constexpr int PG_W = PG_T - PG_TAIL;      // pairs per window
constexpr int PG_G = TGRAD_STRIDE - 1;    // the 23 parameters (the slot's last float is padding)
constexpr int PG_LD = PG_G;               // LDS row stride (floats), odd: conflict-free column writes
constexpr int PG_STEP = 8;                // rows a sum reads at a time

struct PairIn {
  uint4 a, b;   // the pair's two halves
  bool ok;
};

// Loads of pair pidx; ok = in range (the buffers of an overflowed forward
// may be stale: the reads then stay in bounds and the result is discarded).
__device__ __forceinline__ PairIn pair_load(const uint4* __restrict__ pairs, uint32_t pidx, const Layout& L) {
  PairIn q;
  q.a = pairs[2 * (size_t)pidx];
  q.b = pairs[2 * (size_t)pidx + 1];
  q.ok = q.b.y < (uint32_t)L.nv && (int64_t)q.b.x < L.rec_cap;
  return q;
}

__device__ __forceinline__ void pair_row(const PairIn& q, const DevView* __restrict__ vw,
                                         const float4* __restrict__ vrec4, float* row) {
  // the record's projected vertices, inverse depths and SDF values (its first 64 bytes)
  ViewRec R;
  const float4* src = vrec4 + (size_t)q.b.x * 8;
  reinterpret_cast<float4*>(&R)[0] = src[0];
  reinterpret_cast<float4*>(&R)[1] = src[1];
  reinterpret_cast<float4*>(&R)[2] = src[2];
  reinterpret_cast<float4*>(&R)[3] = src[3];
  const DevView& V = vw[q.b.y];
  const auto* dout = gmem(V.dout);
  const int W = V.W, H = V.H;
  const int pix = (int)(q.a.w & 63u);
  const int i = (int)(q.b.z & 0xffffu) * 8 + (pix & 7), j = (int)(q.b.z >> 16) * 8 + (pix >> 3);
  // (clamped: a stale pair of an overflowed forward stays in bounds)
  const size_t plane = (size_t)W * H, p = (size_t)min(j, H - 1) * W + min(i, W - 1);
  float gr[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) gr[k] = dout[k * plane + p];
  float g[PG_G];
  pair_grad_all(R, (float)i + 0.5f, (float)j + 0.5f, gr, __uint_as_float(q.a.x), __uint_as_float(q.a.y),
                __uint_as_float(q.a.z), (int)((q.a.w >> 6) & 15u), g);
#pragma unroll
  for (int k = 0; k < PG_G; ++k) row[k] = g[k];
}

__global__ __launch_bounds__(PG_T) void k_pair_grads(void* ws, Layout L) {
  const DevHeader* hdr = at<const DevHeader>(ws, L.o_hdr);
  const DevView* vw = at<const DevView>(ws, L.o_view);
  const float4* vrec4 = at<const float4>(ws, L.o_vrec);
  const uint4* pairs = at<const uint4>(ws, L.o_pairs);
  float* tgrad = at<float>(ws, L.o_tgrad);
  uint8_t* eflag = at<uint8_t>(ws, L.o_eflag);
  const uint64_t cap = (uint64_t)L.entry_cap;
  const uint32_t npair = (uint32_t)min(hdr->pairs_needed, cap);
  const bool per_record = record_grads(L);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  constexpr uint32_t NW = PG_W / 64;   // waves with window pairs; the last one takes the tail
  // one array: the rows, then the window's segments (a sum's last step may
  // read past its segment's rows, up to the last row and STEP - 1 more, and
  // drops what it read there)
  __shared__ float lds[PG_T * PG_LD + 3 * PG_W];
  static_assert((PG_STEP - 1) * PG_LD <= 3 * PG_W, "a sum's last step stays inside the array");
  uint32_t* hrow = reinterpret_cast<uint32_t*>(lds + PG_T * PG_LD);   // first row | pair count << 16
  uint32_t* hrec = hrow + PG_W;                                       // record
  uint32_t* hslot = hrec + PG_W;                                      // gradient slot
  __shared__ uint32_t wheads[NW];

  for (uint32_t w0 = blockIdx.x * PG_W; w0 < npair; w0 += gridDim.x * PG_W) {
    const uint32_t pidx = w0 + threadIdx.x;
    PairIn q;
    q.ok = false;
    q.a.w = 0u;
    if (pidx < npair) q = pair_load(pairs, pidx, L);
    const bool head = q.ok && (q.a.w & PAIR_HEAD) != 0u;
    const uint64_t hb = __ballot(head);
    bool take = q.ok;
    if (wave == 0u) {
      // pairs before the window's first segment start belong to the previous window
      const uint32_t h0 = hb ? (uint32_t)__ffsll((unsigned long long)hb) - 1u : 64u;
      take = take && !(lane < h0 && w0 > 0u);
    } else if (wave == NW) {
      // the pairs after the window up to the next first pair (or the end)
      // belong to the window's last segment
      const uint64_t tb = __ballot(pidx >= npair || (q.a.w & PAIR_HEAD) != 0u);
      const uint32_t tn = tb ? (uint32_t)__ffsll((unsigned long long)tb) - 1u : 64u;
      take = take && lane < tn;
    }
    if (take) pair_row(q, vw, vrec4, lds + threadIdx.x * PG_LD);
    if (lane == 0u && wave < NW) wheads[wave] = (uint32_t)__popcll(hb);
    __syncthreads();
    uint32_t nh = 0u, hbase = 0u;
#pragma unroll
    for (uint32_t w = 0; w < NW; ++w) {
      hbase += w < wave ? wheads[w] : 0u;
      nh += wheads[w];
    }
    if (head && wave < NW) {
      const uint32_t h = hbase + (uint32_t)__popcll(hb & ((1ull << lane) - 1ull));
      hrow[h] = threadIdx.x | (min((q.a.w >> 11) & 127u, 64u) << 16);
      hrec[h] = q.b.x;
      hslot[h] = q.b.w;
    }
    __syncthreads();
    // a segment per half wave, a parameter per lane (24 of 32)
    const uint32_t k = lane & 31u;
    for (uint32_t h = 2u * wave + (lane >> 5); h < nh; h += 2u * (PG_T / 64)) {
      if (k >= (uint32_t)TGRAD_STRIDE) continue;
      const uint32_t rc = hrow[h], cnt = k < (uint32_t)PG_G ? rc >> 16 : 0u;
      const float* row = lds + (rc & 0xffffu) * PG_LD + k;
      // eight rows per step, their reads in flight together (a fixed order)
      float sum = 0.0f;
      for (uint32_t m0 = 0; m0 < cnt; m0 += PG_STEP) {
        float v[PG_STEP];
#pragma unroll
        for (uint32_t u = 0; u < PG_STEP; ++u) v[u] = row[(m0 + u) * PG_LD];
#pragma unroll
        for (uint32_t u = 0; u < PG_STEP; ++u) v[u] = m0 + u < cnt ? v[u] : 0.0f;
        sum += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
      }
      if (per_record) {
        if (k < (uint32_t)PG_G && sum != 0.0f) unsafeAtomicAdd(&tgrad[(size_t)hrec[h] * TGRAD_STRIDE + k], sum);
      } else {
        const uint32_t d = hslot[h];
        if ((uint64_t)d < cap) {
          tgrad[(size_t)d * TGRAD_STRIDE + k] = sum;
          if (k == 0u) eflag[d] = 1;
        }
      }
    }
    __syncthreads();
  }
}

hipError_t launch_pair_grads(void* ws, const Layout& L, hipStream_t st) {
  if (L.o_pairs == 0) return hipErrorInvalidValue;
  const int64_t b = (L.entry_cap + PG_W - 1) / PG_W;   // one window of pairs per block and pass
  const unsigned blocks = (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
  k_pair_grads<<<blocks, PG_T, 0, st>>>(ws, L);
  return hipGetLastError();
}

template <int NWV>
static void launch_fwd_mw(void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  if (p.chunk_fwd == 32)
    k_composite_mw<NWV, 32><<<(unsigned)L.total_tiles, 64 * NWV, 0, st>>>(ws, L, p.alpha_min, p.alpha_clamp, p.t_min);
  else
    k_composite_mw<NWV, 64><<<(unsigned)L.total_tiles, 64 * NWV, 0, st>>>(ws, L, p.alpha_min, p.alpha_clamp, p.t_min);
}
template <int NWV>
static void launch_bwd_mw(void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  const int rc = (p.flags & RENDER_RECOMPUTE_STATE) ? 1 : 0;
  if (p.chunk_bwd == 16)
    k_composite_bwd_mw<NWV, 16><<<working_tiles(L), 64 * NWV, 0, st>>>(ws, L, p.alpha_min, p.alpha_clamp,
                                                                               p.t_min, rc);
  else
    k_composite_bwd_mw<NWV, 32><<<working_tiles(L), 64 * NWV, 0, st>>>(ws, L, p.alpha_min, p.alpha_clamp,
                                                                               p.t_min, rc);
}

hipError_t launch_composite_mw(void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  switch (p.waves) {
    case 2: launch_fwd_mw<2>(ws, L, p, st); break;
    case 4: launch_fwd_mw<4>(ws, L, p, st); break;
    case 8: launch_fwd_mw<8>(ws, L, p, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_composite_backward_mw(void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  switch (p.waves) {
    case 2: launch_bwd_mw<2>(ws, L, p, st); break;
    case 4: launch_bwd_mw<4>(ws, L, p, st); break;
    case 8: launch_bwd_mw<8>(ws, L, p, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ts
