// Per-scene and per-view preparation kernels of the gfx950 tetrahedron
// rasterizer: descriptor upload, the alpha_max pre-filter with order-
// preserving compaction and per-tet normal/colour (Sec. 3.2, App. A.3),
// projection and binning, tile lists, placement, the dispatch orders, depth
// order inside every tile (Sec. 3.3), the backward's gradient clear; and the
// coarse-to-fine bounds and grids (App. B).
#include <algorithm>
#include <cstring>
#include <vector>

#include "ts_device.h"

namespace ts {

// ---------------------------------------------------------------------------
// descriptor upload through kernel arguments (no host-to-device copies, so
// the whole call sequence can be captured in a graph)
// ---------------------------------------------------------------------------
constexpr int BLOB_WORDS = 960;
struct alignas(16) Blob {
  uint32_t w[BLOB_WORDS];
};

__global__ void k_write_blob(Blob b, uint32_t* dst, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) dst[i] = b.w[i];
}

static hipError_t upload(const void* src, size_t bytes, void* dst, hipStream_t st) {
  const uint32_t* s = static_cast<const uint32_t*>(src);
  uint32_t* d = static_cast<uint32_t*>(dst);
  size_t words = bytes / 4;
  for (size_t o = 0; o < words; o += BLOB_WORDS) {
    Blob b;
    int n = (int)((words - o) < (size_t)BLOB_WORDS ? (words - o) : (size_t)BLOB_WORDS);
    for (int i = 0; i < n; ++i) b.w[i] = s[o + i];
    k_write_blob<<<1, 256, 0, st>>>(b, d + o, n);
  }
  return hipGetLastError();
}

// The header (forward only), scenes, views and scene-view lists occupy
// consecutive workspace regions: they go up as one image (alignment gaps
// zeroed).
static hipError_t desc_image(const DevScene* hs, int ns, const DevView* hv, int nv, const int32_t* scene_views,
                             const Layout& L, bool reset_header, std::vector<uint8_t>& img, size_t& first) {
  static_assert(sizeof(DevHeader) % 4 == 0 && sizeof(DevScene) % 4 == 0 && sizeof(DevView) % 4 == 0,
                "descriptors are whole words");
  first = reset_header ? L.o_hdr : L.o_scene;
  const size_t end = L.o_scene_views + 4 * (size_t)nv;
  if (L.o_hdr > L.o_scene || L.o_scene > L.o_view || L.o_view > L.o_scene_views) return hipErrorInvalidValue;
  img.assign(end - first, 0);
  if (reset_header) {
    // fresh counters for a forward pass (its kernels accumulate into them)
    DevHeader h{};
    h.entry_capacity = L.entry_cap;
    h.kept_capacity = L.kept_cap;
    std::memcpy(img.data() + (L.o_hdr - first), &h, sizeof h);
  }
  std::memcpy(img.data() + (L.o_scene - first), hs, sizeof(DevScene) * ns);
  std::memcpy(img.data() + (L.o_view - first), hv, sizeof(DevView) * nv);
  std::memcpy(img.data() + (L.o_scene_views - first), scene_views, sizeof(int32_t) * nv);
  return hipSuccess;
}


// ---------------------------------------------------------------------------
// a1: pre-filter.  alpha_max = Eq. 1 at (max f, min f) over the 4 vertices;
// keep iff alpha_max >= prefilter_tf.  Kept tets are compacted in ascending
// tet id per scene (block counts; each compaction block sums the counts of
// the blocks before it and rescans its own tets).
// ---------------------------------------------------------------------------
constexpr int PF_THREADS = 256;
constexpr int PF_PER_THREAD = PF_TILE / PF_THREADS;  // 4 consecutive tets per thread

__device__ __forceinline__ int find_scene_by_block(const DevScene* sc, int ns, int b) {
  int lo = 0, hi = ns - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (sc[mid].block_base <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Out-of-range vertex indices never reach a memory access: such a tet is
// dropped (and counted in the header when `invalid` is given).
__device__ __forceinline__ bool keep_tet(const DevScene& S, int k, float tf, uint32_t* invalid, int4* vi_out) {
  int4 vi = load_tet(S.tets, k);
  if (vi_out) *vi_out = vi;
  if ((unsigned)vi.x >= (unsigned)S.V || (unsigned)vi.y >= (unsigned)S.V || (unsigned)vi.z >= (unsigned)S.V ||
      (unsigned)vi.w >= (unsigned)S.V) {
    if (invalid) *invalid = 1u;
    return false;
  }
  const auto* sdf = gmem(S.sdf);
  float f0 = sdf[vi.x], f1 = sdf[vi.y], f2 = sdf[vi.z], f3 = sdf[vi.w];
  float fmax = fmaxf(fmaxf(f0, f1), fmaxf(f2, f3));
  float fmin = fminf(fminf(f0, f1), fminf(f2, f3));
  return alpha_eq1(fmax, fmin, S.s) >= tf;
}

__device__ __forceinline__ uint32_t block_exclusive_scan_256(uint32_t v, uint32_t* lds /*[8]*/, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds[wave] = x;
  __syncthreads();
  uint32_t wbase = 0, tot = 0;
  for (int w = 0; w < PF_THREADS / 64; ++w) {
    uint32_t t = lds[w];
    if (w < wave) wbase += t;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return wbase + x - v;
}

// A block's kept count, with PF_INVALID set when one of its tets had a
// vertex index out of range (the totals put it into the header).
constexpr uint32_t PF_INVALID = 1u << 31;

__device__ __forceinline__ void pf_count_body(void* ws, const Layout& L, float tf, const DevScene* sc) {
  uint32_t* cnt = at<uint32_t>(ws, L.o_pf_cnt);
  __shared__ uint32_t lds[8];
  const int b = blockIdx.x;
  const int s = find_scene_by_block(sc, L.ns, b);
  const DevScene S = sc[s];
  const int k0 = (b - S.block_base) * PF_TILE + threadIdx.x * PF_PER_THREAD;
  uint32_t c = 0, nib = 0, bad = 0;
  static_assert(PF_PER_THREAD == 4 && PF_THREADS % 8 == 0, "a thread's four decisions are a nibble of a word");
#pragma unroll
  for (int q = 0; q < PF_PER_THREAD; ++q) {
    int k = k0 + q;
    const bool kp = k < S.K && keep_tet(S, k, tf, &bad, nullptr);
    c += kp ? 1u : 0u;
    nib |= kp ? 1u << q : 0u;
  }
  const int any_bad = __syncthreads_or((int)bad);
  // the decisions, 4 bits per thread: eight threads fill a word
  const int lane = threadIdx.x & 63;
  uint32_t w = nib << (4 * (lane & 7));
  w |= __shfl_xor(w, 1, 64);
  w |= __shfl_xor(w, 2, 64);
  w |= __shfl_xor(w, 4, 64);
  if ((lane & 7) == 0) at<uint32_t>(ws, L.o_pf_keep)[(size_t)b * (PF_TILE / 32) + (threadIdx.x >> 3)] = w;
  uint32_t tot;
  block_exclusive_scan_256(c, lds, &tot);
  if (threadIdx.x == 0) cnt[b] = tot | (any_bad ? PF_INVALID : 0u);
}

__global__ __launch_bounds__(PF_THREADS) void k_pf_count(void* ws, Layout L, float tf) {
  pf_count_body(ws, L, tf, at<const DevScene>(ws, L.o_scene));
}

// The same, with the forward's descriptor image (header, scenes, views and
// scene-view lists) as the argument: block 0 writes it to the workspace for
// the kernels after this one (no block of this one reads the workspace's
// copy or the header), and every block reads its scene from the argument.
__global__ __launch_bounds__(PF_THREADS) void k_pf_count_desc(Blob d, int nwords, void* ws, Layout L, float tf) {
  if (blockIdx.x == 0) {
    uint32_t* dst = at<uint32_t>(ws, L.o_hdr);
    for (int i = threadIdx.x; i < nwords; i += PF_THREADS) dst[i] = d.w[i];
  }
  pf_count_body(ws, L, tf, reinterpret_cast<const DevScene*>(d.w + (L.o_scene - L.o_hdr) / 4));
}

// Per-scene kept ranges, per-view record bases, totals and capacity checks
// from the pre-filter blocks' counts (thread t sums a contiguous range of
// them; a scan of the range sums gives each range's start, and the scene
// whose first block lies in a range takes its base from there).  One block.
__device__ void prefilter_totals(void* ws, const Layout& L, uint32_t* lds /*[8]*/) {
  DevHeader* hdr = at<DevHeader>(ws, L.o_hdr);
  const DevScene* sc = at<const DevScene>(ws, L.o_scene);
  const DevView* vw = at<const DevView>(ws, L.o_view);
  const uint32_t* cnt = at<const uint32_t>(ws, L.o_pf_cnt);
  int32_t* kbase = at<int32_t>(ws, L.o_scene_kept_base);
  int32_t* kcount = at<int32_t>(ws, L.o_scene_kept_count);
  int32_t* rbase = at<int32_t>(ws, L.o_view_rec_base);
  const int n = (int)L.pf_blocks;
  const int per = (n + PF_THREADS - 1) / PF_THREADS;
  const int j0 = min(n, (int)threadIdx.x * per), j1 = min(n, j0 + per);
  uint32_t sum = 0, bad = 0;
  for (int j = j0; j < j1; ++j) {
    sum += cnt[j] & ~PF_INVALID;
    bad |= cnt[j] & PF_INVALID;
  }
  const int any_bad = __syncthreads_or((int)(bad != 0u));
  uint32_t total;
  const uint32_t start = block_exclusive_scan_256(sum, lds, &total);
  const uint32_t cap = (uint32_t)L.kept_cap;
  // scene s starts at block block_base (a scene with no blocks shares the
  // next one's; past the last block: the total)
  for (int s = 0; s < L.ns; ++s) {
    const int bb = sc[s].block_base;
    const bool mine = (bb >= j0 && bb < j1) || (bb >= n && threadIdx.x == PF_THREADS - 1);
    if (mine) {
      uint32_t x = start;
      for (int j = j0; j < min(bb, j1); ++j) x += cnt[j] & ~PF_INVALID;
      kbase[s] = (int32_t)min(x, cap);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    hdr->kept_total = total;
    uint32_t ovf = total > cap ? 1u : 0u;
    for (int s = 0; s < L.ns; ++s) {
      const uint32_t b0 = (uint32_t)kbase[s];
      const uint32_t b1 = s + 1 < L.ns ? (uint32_t)kbase[s + 1] : min(total, cap);
      kcount[s] = (int32_t)(b1 - b0);
    }
    uint64_t r = 0;
    for (int v = 0; v < L.nv; ++v) {
      rbase[v] = (int32_t)r;
      r += (uint64_t)kcount[vw[v].scene];
    }
    if (r > (uint64_t)L.rec_cap) { ovf |= 1u; r = (uint64_t)L.rec_cap; }
    hdr->records_total = (uint32_t)r;
    hdr->overflow = ovf;
    hdr->entries_total = 0;
    if (any_bad) hdr->invalid_index = 1u;
  }
}

// rescan and write the kept tets' records: vertices, SDF, normal (App. A.3 via
// the equivalent 3x3 edge system), mean colour.  Each block finds the kept
// tets before it by summing the counts of the blocks before it (all threads
// at once); block 0 also writes the per-scene and per-view totals.
__global__ __launch_bounds__(PF_THREADS) void k_pf_scatter(void* ws, Layout L) {
  const DevScene* sc = at<const DevScene>(ws, L.o_scene);
  const uint32_t* cnt = at<const uint32_t>(ws, L.o_pf_cnt);
  TetRec* trec = at<TetRec>(ws, L.o_trec);
  int32_t* kept_tet = at<int32_t>(ws, L.o_kept_tet);
  __shared__ uint32_t lds[8];
  const int b = blockIdx.x;
  {
    // the per-tile entry counters and the dispatch-order histograms and
    // cursors (forward and backward) start cleared for the kernels that follow
    uint32_t* tcnt = at<uint32_t>(ws, L.o_tile_cnt);
    for (uint64_t i = (uint64_t)b * PF_THREADS + threadIdx.x; i < 32u * tile_counter_row(L);
         i += (uint64_t)gridDim.x * PF_THREADS)
      tcnt[i] = 0u;
    if (b == 0) {
      uint32_t* th = at<uint32_t>(ws, L.o_tile_hist);
      for (int i = threadIdx.x; i < 2 * TILE_BUCKETS; i += PF_THREADS) th[i] = 0u;
      uint32_t* bh = at<uint32_t>(ws, L.o_bwd_hist);
      for (int i = threadIdx.x; i < BWD_HIST_WORDS; i += PF_THREADS) bh[i] = 0u;
    }
  }
  if (b == 0) prefilter_totals(ws, L, lds);
  if (b >= (int)L.pf_blocks) return;   // (these only clear; without tets block 0 also writes the totals)
  uint32_t part = 0;
  for (int j = threadIdx.x; j < b; j += PF_THREADS) part += cnt[j] & ~PF_INVALID;
  uint32_t before;
  block_exclusive_scan_256(part, lds, &before);
  const int s = find_scene_by_block(sc, L.ns, b);
  const DevScene S = sc[s];
  const int k0 = (b - S.block_base) * PF_TILE + threadIdx.x * PF_PER_THREAD;
  // the count kernel's decisions (this thread's nibble); only kept tets are read
  const uint32_t nib =
      (at<const uint32_t>(ws, L.o_pf_keep)[(size_t)b * (PF_TILE / 32) + (threadIdx.x >> 3)] >> (4 * (threadIdx.x & 7))) & 15u;
  bool kp[PF_PER_THREAD];
  int4 vi[PF_PER_THREAD];
  uint32_t c = 0;
#pragma unroll
  for (int q = 0; q < PF_PER_THREAD; ++q) {
    kp[q] = (nib >> q) & 1u;
    vi[q] = make_int4(0, 0, 0, 0);
    if (kp[q]) vi[q] = load_tet(S.tets, k0 + q);
    c += kp[q] ? 1u : 0u;
  }
  uint32_t tot;
  uint32_t slot = before + block_exclusive_scan_256(c, lds, &tot);
#pragma unroll
  for (int q = 0; q < PF_PER_THREAD; ++q) {
    if (!kp[q]) continue;
    const uint32_t my = slot++;
    if (my >= (uint32_t)L.kept_cap) continue;
    const int idx[4] = {vi[q].x, vi[q].y, vi[q].z, vi[q].w};
    TetRec r;
    for (int a = 0; a < 4; ++a) {
      r.x[a][0] = gmem(S.verts)[3 * (size_t)idx[a] + 0];
      r.x[a][1] = gmem(S.verts)[3 * (size_t)idx[a] + 1];
      r.x[a][2] = gmem(S.verts)[3 * (size_t)idx[a] + 2];
      r.f[a] = gmem(S.sdf)[idx[a]];
    }
    // g = E^-1 (f_k - f_0), E rows e_k = x_k - x_0 (k = 1..3)
    float e[3][3], df[3];
    for (int a = 0; a < 3; ++a) {
      for (int j = 0; j < 3; ++j) e[a][j] = r.x[a + 1][j] - r.x[0][j];
      df[a] = r.f[a + 1] - r.f[0];
    }
    float c23[3] = {e[1][1] * e[2][2] - e[1][2] * e[2][1], e[1][2] * e[2][0] - e[1][0] * e[2][2],
                    e[1][0] * e[2][1] - e[1][1] * e[2][0]};
    float c31[3] = {e[2][1] * e[0][2] - e[2][2] * e[0][1], e[2][2] * e[0][0] - e[2][0] * e[0][2],
                    e[2][0] * e[0][1] - e[2][1] * e[0][0]};
    float c12[3] = {e[0][1] * e[1][2] - e[0][2] * e[1][1], e[0][2] * e[1][0] - e[0][0] * e[1][2],
                    e[0][0] * e[1][1] - e[0][1] * e[1][0]};
    float det = e[0][0] * c23[0] + e[0][1] * c23[1] + e[0][2] * c23[2];
    float g[3];
    for (int j = 0; j < 3; ++j) g[j] = (det != 0.0f) ? (c23[j] * df[0] + c31[j] * df[1] + c12[j] * df[2]) / det : 0.0f;
    float gn = sqrtf(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
    for (int j = 0; j < 3; ++j) r.n[j] = (gn > 0.0f) ? g[j] / gn : 0.0f;
    for (int j = 0; j < 3; ++j) {
      const auto* C = gmem(S.colors);
      r.c[j] = ((C[3 * (size_t)idx[0] + j] + C[3 * (size_t)idx[1] + j]) +
                (C[3 * (size_t)idx[2] + j] + C[3 * (size_t)idx[3] + j])) * 0.25f;
    }
    r.tet = k0 + q;
    r.scene = s;
    trec[my] = r;
    kept_tet[my] = k0 + q;
  }
}

// The scatter's blocks: one per block of tets, more where those would be few for
// the tile counters that it clears (16 words a thread).
static unsigned pf_scatter_blocks(const Layout& L) {
  const int64_t words = 32 * (int64_t)tile_counter_row(L);
  return (unsigned)std::max(std::max<int64_t>(L.pf_blocks, 1), std::min<int64_t>(words / (16 * PF_THREADS), 1024));
}

hipError_t launch_prefilter(void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  if (L.pf_blocks > 0) k_pf_count<<<(unsigned)L.pf_blocks, PF_THREADS, 0, st>>>(ws, L, p.prefilter_tf);
  k_pf_scatter<<<pf_scatter_blocks(L), PF_THREADS, 0, st>>>(ws, L);
  return hipGetLastError();
}

// The forward's descriptor upload and pre-filter: when the descriptor image
// fits one kernel argument, the pre-filter's counting launch carries it (one
// launch fewer); otherwise it goes up first.
hipError_t launch_desc_prefilter(const DevScene* hs, int ns, const DevView* hv, int nv, const int32_t* scene_views,
                                 void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  std::vector<uint8_t> img;
  size_t first;
  hipError_t e = desc_image(hs, ns, hv, nv, scene_views, L, true, img, first);
  if (e != hipSuccess) return e;
  const size_t words = img.size() / 4;
  if (words > (size_t)BLOB_WORDS || L.pf_blocks == 0 || first != L.o_hdr) {
    e = upload(img.data(), img.size(), at<void>(ws, first), st);
    if (e != hipSuccess) return e;
    return launch_prefilter(ws, L, p, st);
  }
  Blob b;
  std::memcpy(b.w, img.data(), img.size());
  k_pf_count_desc<<<(unsigned)L.pf_blocks, PF_THREADS, 0, st>>>(b, (int)words, ws, L, p.prefilter_tf);
  k_pf_scatter<<<pf_scatter_blocks(L), PF_THREADS, 0, st>>>(ws, L);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a2, a3: per (view, kept tet) record: camera transform, near-plane cull,
// projection, pixel rectangle, tile count, depth key (float32, fixed op
// sequence), 2D face determinants, shading features; then the binning of its
// entries, one per tile that its rectangle touches.
// ---------------------------------------------------------------------------
// One block projects 256 consecutive kept tets of one view per step.  The
// 96-byte tet records come in and the 128-byte view records go out through
// LDS, so that every HBM access of the records is contiguous across the
// block.  A record takes 9 x 16 bytes in LDS: when each thread reads or
// writes its own record 16 bytes at a time, sixteen neighbouring threads
// touch 64 distinct banks.
//   The step's entries are binned while its rectangles are in LDS.  The block
// takes its entries' places (the records' gradient slots, contiguous per
// record) from one global counter, and every entry its rank inside its tile's
// list from the tile's counter; neighbouring records touch neighbouring tiles,
// so the block's entries are counted per tile in an LDS hash first (integer
// LDS adds are fast on this chip) and each tile costs one global atomic.
// (tile, rank, record and whether it cannot blend) go out per entry; once the
// tiles' counts are scanned, an entry's place in the lists is its tile's start plus its rank.
// The order inside a list is left to the atomics: the per-tile depth sort
// imposes the final one.
//   At the training shape (496k records, 1.75 M entries) this took the place of
// a projection (27 us), a count of every tile's entries (25), the scan of the
// counts (11), and a second pass that found every entry's tile again to place
// it (29): now 51 us here (with the hull spans and never_blends) and 10 us in
// k_emit; 8 x 1024^2: 142 + 91 + 114 to 235 + 78 us.  Bound by the latency of a step's phases (two rounds of four
// workgroups per CU there; LDS, 40 KB, sets the four).  Grouping a wave's
// entries by ballots instead of the hash: 56 us, and 111 against 68 us for six
// mixed scenes.
constexpr int PROJ_STRIDE = 9;   // uint4 per record in LDS
constexpr int BIN_PER = 4;       // entries per thread and binning round
constexpr uint32_t BIN_SLOTS = 1024, BIN_PROBES = 16;
struct BinHash {
  uint32_t key[BIN_SLOTS];       // tile + 1; 0: free
  uint32_t cnt[BIN_SLOTS];       // the round's entries of the tile, then the first one's rank
};
static_assert(sizeof(BinHash) <= 256 * PROJ_STRIDE * 16, "the hash takes the records' place in LDS");
static_assert(sizeof(TetRec) == 6 * 16 && sizeof(ViewRec) == 8 * 16, "record sizes in 16-byte units");
static_assert(BIN_SLOTS == 1u << 10, "the tile hash keeps 10 bits");

__global__ __launch_bounds__(256) void k_project(void* ws, Layout L, int tw_log2, int th_log2, float alpha_min) {
  DevHeader* hdr = at<DevHeader>(ws, L.o_hdr);
  const DevView* vw = at<const DevView>(ws, L.o_view);
  const int32_t* kbase = at<const int32_t>(ws, L.o_scene_kept_base);
  const int32_t* kcount = at<const int32_t>(ws, L.o_scene_kept_count);
  const int32_t* rbase = at<const int32_t>(ws, L.o_view_rec_base);
  const uint4* trec4 = at<const uint4>(ws, L.o_trec);
  uint4* vrec4 = at<uint4>(ws, L.o_vrec);
  uint32_t* count1 = at<uint32_t>(ws, L.o_count1);
  uint32_t* key1 = at<uint32_t>(ws, L.o_key1a);
  uint32_t* rfirst = at<uint32_t>(ws, L.o_rfirst);
  uint32_t* tcnt = at<uint32_t>(ws, L.o_tile_cnt);
  uint32_t* etile = at<uint32_t>(ws, L.o_key2a);
  uint32_t* erank = at<uint32_t>(ws, L.o_key2b);
  uint32_t* erec = at<uint32_t>(ws, L.o_val2b);
  const uint64_t cap = (uint64_t)L.entry_cap;
  __shared__ uint4 sbuf[256 * PROJ_STRIDE];
  __shared__ unsigned long long svalid[4];   // bit: the record covers a pixel
  __shared__ unsigned long long sidle[4];    // bit: and cannot blend
  __shared__ uint32_t loff[256];
  __shared__ uint2 lrect[256];
  __shared__ uint32_t lds[8];
  __shared__ unsigned long long sbase;
  BinHash& H = *reinterpret_cast<BinHash*>(sbuf);
  const int v = blockIdx.y;
  const DevView V = vw[v];
  const float ifx = rcp(fabsf(V.fx)), ify = rcp(fabsf(V.fy));
  const int n = kcount[V.scene];
  const int r0 = rbase[v];
  const int kb = kbase[V.scene];
  if ((uint64_t)r0 + (uint64_t)n > (uint64_t)hdr->records_total) return;  // capacity overflow guard
  const int t = threadIdx.x;
  for (int k0 = blockIdx.x * 256; k0 < n; k0 += gridDim.x * 256) {
    const int nloc = min(256, n - k0);
    // tet records in, contiguous
    const uint4* src = trec4 + (size_t)(kb + k0) * 6;
    for (int q = t; q < nloc * 6; q += 256) sbuf[(q / 6) * PROJ_STRIDE + (q % 6)] = src[q];
    __syncthreads();
    TetRec T;
    if (t < nloc) {
#pragma unroll
      for (int q = 0; q < 6; ++q) reinterpret_cast<uint4*>(&T)[q] = sbuf[t * PROJ_STRIDE + q];
    }
    __syncthreads();
    uint32_t valid = 0, cnt = 0, idle = 0;   // idle: none of the record's pixels can blend it
    if (t < nloc) {
      const int k = k0 + t;
      const int r = r0 + k;
      float X[4], Y[4], Z[4], px[4], py[4];
      bool culled = false;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const float x = T.x[a][0], y = T.x[a][1], z = T.x[a][2];
        X[a] = fmaf(V.R[0], x, fmaf(V.R[1], y, fmaf(V.R[2], z, V.t[0])));
        Y[a] = fmaf(V.R[3], x, fmaf(V.R[4], y, fmaf(V.R[5], z, V.t[1])));
        Z[a] = fmaf(V.R[6], x, fmaf(V.R[7], y, fmaf(V.R[8], z, V.t[2])));
        culled |= (Z[a] < V.znear);
      }
      uint32_t key = 0xffffffffu;
      if (!culled) {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          px[a] = fmaf(V.fx, X[a] / Z[a], V.cx);
          py[a] = fmaf(V.fy, Y[a] / Z[a], V.cy);
        }
        const float zt = ((Z[0] + Z[1]) + (Z[2] + Z[3])) * 0.25f;
        const float xmin = fminf(fminf(px[0], px[1]), fminf(px[2], px[3]));
        const float xmax = fmaxf(fmaxf(px[0], px[1]), fmaxf(px[2], px[3]));
        const float ymin = fminf(fminf(py[0], py[1]), fminf(py[2], py[3]));
        const float ymax = fmaxf(fmaxf(py[0], py[1]), fmaxf(py[2], py[3]));
        const int i0 = (int)fminf(fmaxf(ceilf(xmin - 0.5f), 0.0f), (float)V.W);
        const int i1 = (int)fmaxf(fminf(floorf(xmax - 0.5f), (float)(V.W - 1)), -1.0f);
        const int j0 = (int)fminf(fmaxf(ceilf(ymin - 0.5f), 0.0f), (float)V.H);
        const int j1 = (int)fmaxf(fminf(floorf(ymax - 0.5f), (float)(V.H - 1)), -1.0f);
        if (i0 <= i1 && j0 <= j1) {
          const int tx0 = i0 >> tw_log2, tx1 = i1 >> tw_log2, ty0 = j0 >> th_log2, ty1 = j1 >> th_log2;
          cnt = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
          key = __float_as_uint(zt);
          ViewRec R;
          for (int a = 0; a < 4; ++a) {
            R.px[a] = px[a];
            R.py[a] = py[a];
            R.iz[a] = 1.0f / Z[a];
            R.f[a] = T.f[a];
          }
          float D[4];
          for (int F = 0; F < 4; ++F) {
            const int A = face_vertex(F, 0), B = face_vertex(F, 1), C = face_vertex(F, 2);
            D[F] = (px[B] - px[A]) * (py[C] - py[A]) - (py[B] - py[A]) * (px[C] - px[A]);
            R.rD[F] = D[F] != 0.0f ? rcp(D[F]) : 0.0f;   // once per record, not per pixel
          }
          R.c[0] = T.c[0]; R.c[1] = T.c[1]; R.c[2] = T.c[2];
          R.zt = zt;
          R.n[0] = T.n[0]; R.n[1] = T.n[1]; R.n[2] = T.n[2];
          R.rx = (uint32_t)i0 | ((uint32_t)i1 << 16);
          R.ry = (uint32_t)j0 | ((uint32_t)j1 << 16);
          const float ext = fmaxf(xmax - xmin, ymax - ymin);
          if (!hull_spans(px, py, D, ext, i0, i1, j0, j1, R.span)) idle = 1;
          const float reach = fmaxf(1.0f, fmaxf(fmaxf(fabsf(xmin), fabsf(xmax)) * ifx, fmaxf(fabsf(ymin), fabsf(ymax)) * ify));
          if (never_blends(X, Y, Z, T.f, D, ext, reach, V.s, alpha_min)) idle = 1;
          R.entry0 = 0;
#pragma unroll
          for (int q = 0; q < 8; ++q) sbuf[t * PROJ_STRIDE + q] = reinterpret_cast<const uint4*>(&R)[q];
          valid = 1;
        }
      }
      count1[r] = cnt;
      key1[r] = key;
    }
    uint32_t tot;
    const uint32_t off = block_exclusive_scan_256(cnt, lds, &tot);
    loff[t] = off;
    if (valid) lrect[t] = make_uint2(sbuf[t * PROJ_STRIDE + 6].w, sbuf[t * PROJ_STRIDE + 7].x);
    const uint64_t vb = __ballot(valid != 0u);
    const uint64_t ib = __ballot(idle != 0u);
    if ((t & 63) == 0) {
      svalid[t >> 6] = vb;
      sidle[t >> 6] = ib;
    }
    // (the places' counter is not waited for before the records have gone out)
    unsigned long long place = 0ull;
    if (t == 0 && tot > 0u) place = atomicAdd((unsigned long long*)&hdr->entries_needed, (unsigned long long)tot);
    __syncthreads();
    // view records out, contiguous (records that cover no pixel are skipped)
    uint4* dst = vrec4 + (size_t)(r0 + k0) * 8;
    for (int q = t; q < nloc * 8; q += 256)
      if ((svalid[q >> 9] >> ((q >> 3) & 63)) & 1ull) dst[q] = sbuf[(q >> 3) * PROJ_STRIDE + (q & 7)];
    if (t == 0) sbase = place;
    __syncthreads();
    const uint64_t base = sbase;
    if (cnt) rfirst[r0 + k0 + t] = (uint32_t)min(base + off, (uint64_t)0xffffffffu);
    // the binning, BIN_PER x 256 entries a round
    for (uint32_t e0 = 0; e0 < tot; e0 += 256u * BIN_PER) {
      __syncthreads();   // the records, or the last round's hash, are done with
      for (uint32_t i = t; i < BIN_SLOTS; i += 256u) H.key[i] = H.cnt[i] = 0u;
      __syncthreads();
      uint32_t q[BIN_PER], tile[BIN_PER], rank[BIN_PER], slot[BIN_PER];
#pragma unroll
      for (int i = 0; i < BIN_PER; ++i) {
        const uint32_t e = e0 + 256u * i + (uint32_t)t;
        q[i] = tile[i] = rank[i] = 0u;
        slot[i] = BIN_SLOTS;
        if (e >= tot) continue;
        // the entry's record: the last one whose first entry is at or before it
#pragma unroll
        for (uint32_t step = 128u; step > 0u; step >>= 1) q[i] = loff[q[i] + step] <= e ? q[i] + step : q[i];
        const uint2 rc = lrect[q[i]];
        const int tx0 = (int)(rc.x & 0xffffu) >> tw_log2, tx1 = (int)(rc.x >> 16) >> tw_log2;
        const int ty0 = (int)(rc.y & 0xffffu) >> th_log2;
        const uint32_t nx = (uint32_t)(tx1 - tx0 + 1), j = e - loff[q[i]], jy = j / nx;
        tile[i] = (uint32_t)(V.tile_base + (ty0 + (int)jy) * V.tiles_x + tx0 + (int)(j - jy * nx));
        uint32_t h = (tile[i] * 2654435761u) >> 22;   // 10 bits: BIN_SLOTS
#pragma unroll 1
        for (uint32_t p = 0; p < BIN_PROBES; ++p) {
          uint32_t key = H.key[h];
          if (key == 0u) {
            key = atomicCAS(&H.key[h], 0u, tile[i] + 1u);
            if (key == 0u) key = tile[i] + 1u;
          }
          if (key == tile[i] + 1u) {
            slot[i] = h;
            rank[i] = atomicAdd(&H.cnt[h], 1u);
            break;
          }
          h = (h + 1u) & (BIN_SLOTS - 1u);
        }
        if (slot[i] == BIN_SLOTS) rank[i] = atomicAdd(&tcnt[tile_counter(L, tile[i])], 1u);   // no place: on its own
      }
      __syncthreads();
      {
        // the tiles' counters, a thread's atomics in flight together
        constexpr int NS = BIN_SLOTS / 256;
        uint32_t c[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) c[i] = H.cnt[t + 256 * i];
#pragma unroll
        for (int i = 0; i < NS; ++i)
          if (c[i] != 0u) c[i] = atomicAdd(&tcnt[tile_counter(L, H.key[t + 256 * i] - 1u)], c[i]);
#pragma unroll
        for (int i = 0; i < NS; ++i) H.cnt[t + 256 * i] = c[i];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < BIN_PER; ++i) {
        const uint32_t e = e0 + 256u * i + (uint32_t)t;
        const uint64_t d = base + e;
        if (e >= tot || d >= cap) continue;
        etile[d] = tile[i];
        erank[d] = rank[i] + (slot[i] < BIN_SLOTS ? H.cnt[slot[i]] : 0u);
        erec[d] = ((uint32_t)(r0 + k0) + q[i]) << 1 | (uint32_t)((sidle[q[i] >> 6] >> (q[i] & 63u)) & 1ull);
      }
    }
    __syncthreads();
  }
}

hipError_t launch_project(void* ws, const Layout& L, const render_params& p, hipStream_t st) {
  int twl = __builtin_ctz((unsigned)p.tile_w), thl = __builtin_ctz((unsigned)p.tile_h);
  dim3 grid(512, (unsigned)L.nv);
  k_project<<<grid, 256, 0, st>>>(ws, L, twl, thl, p.alpha_min);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a3: the tile lists.  Each tile's list [start, end) from the exclusive scan of
// the tiles' entry counts, and the dispatch-order histogram of their lengths.
// Up to LISTS_DIRECT blocks of 1024 tiles every block sums the counts of the
// tiles before its own itself (at most 256 KB from L2, some 3 us; a launch
// costs 4.6 us); past that the blocks' sums come from a launch of their own.
// More entries than the capacity: every list is left empty (the forward's
// outputs are invalid then), since entries past it were not kept.
// ---------------------------------------------------------------------------
constexpr int64_t LISTS_DIRECT = 64;

__device__ __forceinline__ uint32_t block_sum_1024(uint32_t x, uint32_t* lds /*[16]*/) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
  __syncthreads();
  uint32_t sum = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) sum += lds[w];
  __syncthreads();
  return sum;
}

__device__ __forceinline__ uint32_t block_exclusive_scan_1024(uint32_t v, uint32_t* lds /*[16]*/) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t x = wave_scan_add(v);
  if (lane == 63) lds[wave] = x;
  __syncthreads();
  uint32_t wbase = 0;
  for (int w = 0; w < wave; ++w) wbase += lds[w];
  __syncthreads();
  return wbase + x - v;
}

// per 1024 tiles: the entry total of the block's tiles
__global__ __launch_bounds__(1024) void k_tile_block_sum(void* ws, Layout L) {
  __shared__ uint32_t lds[16];
  const uint32_t t = blockIdx.x * 1024u + threadIdx.x;
  const uint32_t sum = block_sum_1024(
      t < (uint32_t)L.total_tiles ? at<const uint32_t>(ws, L.o_tile_cnt)[tile_counter(L, t)] : 0u, lds);
  if (threadIdx.x == 0) at<uint32_t>(ws, L.o_tile_bsum)[blockIdx.x] = sum;
}

__global__ __launch_bounds__(1024) void k_tile_lists(void* ws, Layout L, int direct) {
  DevHeader* hdr = at<DevHeader>(ws, L.o_hdr);
  const uint32_t* tcnt = at<const uint32_t>(ws, L.o_tile_cnt);
  uint2* ranges = at<uint2>(ws, L.o_ranges);
  uint32_t* hist = at<uint32_t>(ws, L.o_tile_hist);
  __shared__ uint32_t lds[16];
  __shared__ uint32_t hb[TILE_BUCKETS];
  if (threadIdx.x < TILE_BUCKETS) hb[threadIdx.x] = 0u;
  const uint64_t total = hdr->entries_needed;
  const bool over = total > (uint64_t)L.entry_cap;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    hdr->entries_total = over ? (uint32_t)L.entry_cap : (uint32_t)total;
    if (over) hdr->overflow |= 2u;
  }
  // (without an overflow every sum below is under 2^31)
  uint32_t before = 0u;
  if (direct) {
    // the tiles before 1024 b: the first 32 b counters of each of the 32 rows
    const uint4* t4 = at<const uint4>(ws, L.o_tile_cnt);
    const uint32_t row4 = (uint32_t)(tile_counter_row(L) / 4), n4 = blockIdx.x * 8u;
    for (uint32_t i = threadIdx.x & 31u; i < n4; i += 32u) {
      const uint4 c = t4[(threadIdx.x >> 5) * row4 + i];
      before += (c.x + c.y) + (c.z + c.w);
    }
  } else {
    const uint32_t* bsum = at<const uint32_t>(ws, L.o_tile_bsum);
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 1024u) before += bsum[i];
  }
  before = block_sum_1024(before, lds);
  const uint32_t t = blockIdx.x * 1024u + threadIdx.x;
  const bool in = t < (uint32_t)L.total_tiles;
  const uint32_t c = in && !over ? tcnt[tile_counter(L, t)] : 0u;
  const uint32_t start = before + block_exclusive_scan_1024(c, lds);
  if (in) {
    ranges[t] = c ? make_uint2(start, start + c) : make_uint2(0u, 0u);   // an empty list is (0, 0)
    atomicAdd(&hb[len_bucket(c)], 1u);
  }
  __syncthreads();
  if (threadIdx.x < TILE_BUCKETS && hb[threadIdx.x]) atomicAdd(&hist[threadIdx.x], hb[threadIdx.x]);
}

hipError_t launch_tile_lists(void* ws, const Layout& L, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  const int direct = L.tile_blocks <= LISTS_DIRECT ? 1 : 0;
  if (!direct) k_tile_block_sum<<<(unsigned)L.tile_blocks, 1024, 0, st>>>(ws, L);
  k_tile_lists<<<(unsigned)L.tile_blocks, 1024, 0, st>>>(ws, L, direct);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// dispatch order of the compositing workgroups: tiles with the longest lists
// first (bucketed by the list length: four buckets per power of two), so the
// longest sequential walks start in the first scheduling round.  The forward
// orders by list length; the backward by the length the forward actually
// walked before every pixel of the tile stopped.  The order inside a bucket is
// whatever the atomics give; results do not depend on it.
// ---------------------------------------------------------------------------

// Every scatter block: first[b] = the number of tiles in buckets above b
// (longest first), from the complete histogram; the block's tiles of bucket
// b then take consecutive places from first[b] + an atomic cursor.
static_assert(TILE_BUCKETS <= 256, "one thread per bucket");
// tiles per thread of the scatter kernels (4 -- a quarter of the blocks and
// of their per-bucket cursor atomics -- was 5 us slower per step: the
// per-block work grew more than the atomics shrank)
constexpr int SC_PER = 1;
__device__ __forceinline__ void bucket_first(const uint32_t* hist, uint32_t* first, uint32_t* lds /*[8]*/) {
  const int t = threadIdx.x;
  const uint32_t v = t < TILE_BUCKETS ? hist[TILE_BUCKETS - 1 - t] : 0u;
  uint32_t tot;
  const uint32_t ex = block_exclusive_scan_256(v, lds, &tot);
  if (t < TILE_BUCKETS) first[TILE_BUCKETS - 1 - t] = ex;
}

// block `blk` of the forward's dispatch order (256 tiles)
__device__ __forceinline__ void tile_scatter_block(void* ws, const Layout& L, uint32_t blk) {
  const uint32_t* ranges = at<const uint32_t>(ws, L.o_ranges);
  const uint32_t* hist = at<const uint32_t>(ws, L.o_tile_hist);
  uint32_t* cursor = at<uint32_t>(ws, L.o_tile_hist) + TILE_BUCKETS;
  TileSlot* order = at<TileSlot>(ws, L.o_tile_order);
  const DevView* vw = at<const DevView>(ws, L.o_view);
  __shared__ uint32_t cnt[TILE_BUCKETS], base[TILE_BUCKETS], first[TILE_BUCKETS], lds[8];
  if (threadIdx.x < TILE_BUCKETS) cnt[threadIdx.x] = 0;
  bucket_first(hist, first, lds);
  __syncthreads();
  int b[SC_PER];
  uint32_t rank[SC_PER];
#pragma unroll
  for (int i = 0; i < SC_PER; ++i) {
    const uint32_t t = (blk * SC_PER + (uint32_t)i) * 256u + threadIdx.x;
    b[i] = 0;
    rank[i] = 0u;
    if (t < (uint32_t)L.total_tiles) {
      b[i] = len_bucket(ranges[2 * t + 1] - ranges[2 * t]);
      rank[i] = atomicAdd(&cnt[b[i]], 1u);
    }
  }
  __syncthreads();
  if (threadIdx.x < TILE_BUCKETS && cnt[threadIdx.x])
    base[threadIdx.x] = first[threadIdx.x] + atomicAdd(&cursor[threadIdx.x], cnt[threadIdx.x]);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SC_PER; ++i) {
    const uint32_t t = (blk * SC_PER + (uint32_t)i) * 256u + threadIdx.x;
    if (t < (uint32_t)L.total_tiles) {
      TileSlot sl;
      sl.tile = t;
      sl.view = (uint32_t)find_view_by_tile(vw, L.nv, (int)t);
      sl.start = ranges[2 * t];
      sl.end = ranges[2 * t + 1];
      order[base[b[i]] + rank[i]] = sl;
    }
  }
}

// ---------------------------------------------------------------------------
// a4: every entry's record into its tile's list, at the list's start plus the
// entry's rank (a4), and the forward's dispatch order (its first blocks): two
// independent steps after the tile lists, in one launch.
// ---------------------------------------------------------------------------
constexpr int EMIT_PER = 4;   // entries per thread and step
__global__ __launch_bounds__(256) void k_emit(void* ws, Layout L, uint32_t scatter_blocks) {
  if (blockIdx.x < scatter_blocks) {
    tile_scatter_block(ws, L, blockIdx.x);
    return;
  }
  const uint64_t total = at<const DevHeader>(ws, L.o_hdr)->entries_needed;
  if (total > (uint64_t)L.entry_cap) return;   // the lists are empty
  const uint32_t n = (uint32_t)total;
  const uint2* ranges = at<const uint2>(ws, L.o_ranges);
  const uint32_t* etile = at<const uint32_t>(ws, L.o_key2a);
  const uint32_t* erank = at<const uint32_t>(ws, L.o_key2b);
  const uint32_t* erec = at<const uint32_t>(ws, L.o_val2b);
  uint32_t* list = at<uint32_t>(ws, sorted_entry_records(L));
  const uint32_t step = 256u * EMIT_PER, blk = blockIdx.x - scatter_blocks, nblk = gridDim.x - scatter_blocks;
  for (uint64_t d0 = (uint64_t)blk * step; d0 < n; d0 += (uint64_t)nblk * step) {
    uint32_t tile[EMIT_PER], rank[EMIT_PER], rec[EMIT_PER], start[EMIT_PER];
#pragma unroll
    for (int i = 0; i < EMIT_PER; ++i) {
      const uint64_t d = d0 + 256u * i + threadIdx.x;
      const bool in = d < n;
      tile[i] = in ? etile[d] : 0u;
      rank[i] = in ? erank[d] : 0u;
      rec[i] = in ? erec[d] : 0u;
    }
#pragma unroll
    for (int i = 0; i < EMIT_PER; ++i) start[i] = ranges[tile[i]].x;
#pragma unroll
    for (int i = 0; i < EMIT_PER; ++i)
      if (d0 + 256u * i + threadIdx.x < n) list[start[i] + rank[i]] = rec[i];
  }
}

hipError_t launch_emit(void* ws, const Layout& L, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  const unsigned ns = (unsigned)((L.total_tiles + 256 * SC_PER - 1) / (256 * SC_PER));
  const int64_t nb = (L.entry_cap + 256 * EMIT_PER - 1) / (256 * EMIT_PER);
  // (the length histogram was counted by k_tile_lists)
  k_emit<<<ns + (unsigned)(nb < 4096 ? nb : 4096), 256, 0, st>>>(ws, L, ns);
  return hipGetLastError();
}

// backward order: forward slots re-bucketed by the walked length pend - start
// (the forward compositing kernel counted every slot with pend > start; the
// tiles with nothing walked form bucket 0, placed last, whose own count the
// offsets never need).  Every slot also gets the base of its blended pairs in
// the backward's pair buffer, by the same bucket scheme (the forward counted
// them per slot and per bucket).  256 tiles per block and step.
__device__ __forceinline__ void bwd_scatter(void* ws, const Layout& L, uint32_t blk, uint32_t nblk) {
  const TileSlot* slots = at<const TileSlot>(ws, L.o_tile_order);
  const uint32_t* pend = at<const uint32_t>(ws, L.o_tile_pend);
  const uint32_t* slot_pairs = at<const uint32_t>(ws, L.o_slot_pairs);
  const uint32_t* hist = at<const uint32_t>(ws, L.o_bwd_hist);
  uint32_t* cursor = at<uint32_t>(ws, L.o_bwd_hist) + TILE_BUCKETS;
  uint32_t* pcursor = at<uint32_t>(ws, L.o_bwd_hist) + 3 * TILE_BUCKETS;
  TileSlot* bslots = at<TileSlot>(ws, L.o_bwd_order);
  uint32_t* bpend = at<uint32_t>(ws, L.o_bwd_pend);
  uint32_t* bbase = at<uint32_t>(ws, L.o_bwd_base);
  __shared__ uint32_t cnt[TILE_BUCKETS], base[TILE_BUCKETS], first[TILE_BUCKETS], lds[8];
  __shared__ uint32_t pcnt[TILE_BUCKETS], pbase[TILE_BUCKETS], pfirst[TILE_BUCKETS];
  bucket_first(hist, first, lds);
  __syncthreads();
  bucket_first(hist + 2 * TILE_BUCKETS, pfirst, lds);
  __syncthreads();
  // the slots before bucket 0 are the tiles with something walked
  if (blk == 0 && threadIdx.x == 0) at<DevHeader>(ws, L.o_hdr)->bwd_work = first[0];
  for (uint32_t t0 = blk * 256u; t0 < (uint32_t)L.total_tiles; t0 += nblk * 256u) {
    if (threadIdx.x < TILE_BUCKETS) cnt[threadIdx.x] = pcnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t t = t0 + threadIdx.x;
    const bool in = t < (uint32_t)L.total_tiles;
    TileSlot sl{};
    uint32_t pe = 0u, rank = 0u, prank = 0u;
    int b = 0;
    if (in) {
      sl = slots[t];
      pe = pend[t];
      b = len_bucket(pe - sl.start);
      rank = atomicAdd(&cnt[b], 1u);
      if (pe > sl.start) prank = atomicAdd(&pcnt[b], slot_pairs[t]);
    }
    __syncthreads();
    if (threadIdx.x < TILE_BUCKETS && cnt[threadIdx.x]) {
      base[threadIdx.x] = first[threadIdx.x] + atomicAdd(&cursor[threadIdx.x], cnt[threadIdx.x]);
      pbase[threadIdx.x] = pfirst[threadIdx.x] + atomicAdd(&pcursor[threadIdx.x], pcnt[threadIdx.x]);
    }
    __syncthreads();
    if (in) {
      const uint32_t q = base[b] + rank;
      bslots[q] = sl;
      bpend[q] = pe;
      bbase[q] = pbase[b] + prank;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// a5b: depth order inside each tile.  The tile lists hold every tile's entries
// in no particular order; each is sorted by the key (depth float bits,
// record), which is unique and gives the (tile, depth, tet id) order of Sec.
// 3.3 with the tie broken by tet id (records of a view ascend with the tet
// id).  One workgroup per tile with entries, longest lists first (the forward
// dispatch order).
//   A list is sorted by counting: its keys go to DS_BUCKETS buckets of equal
// width over the list's own depth range (monotone in the depth bits), the
// buckets are scanned, and a key's place inside its bucket is the number of
// smaller keys there, mostly none or a few.  That is some ten LDS operations
// per key and five barriers; the merge sort below, a binary search per key and
// doubling, is bound by the latency of its dependent LDS reads (775 lists of
// 295 entries on average: 17 to 7 us; 27k of 446: 218 to 121 us).
// Lists past DS_LIST (the keys a workgroup keeps in LDS: at 20 KB eight fit a
// CU) take the buckets in groups of at most that many keys; the merge sort's
// runs merged in HBM made the few lists past 1,024 a tail (3.5k lists of 499, up
// to 1,129: 37 us with the merge sort, 35 with counting up to 1,024, 19 so).
//   Depths that agree in almost all their bits share a bucket (the layers of a
// grid seen along an axis): past DS_CROWD keys in one, or DS_CROWD_LONG in a list
// past DS_LIST, the list is merge sorted instead, in runs of DS_RUN keys in LDS
// merged pairwise in HBM.  A key costs its bucket's length by counting, and so
// the lines lie: lists of 1000 in layers of 60 equal depths 22 against 28 us,
// of 200 49 against 28; of 40,000 in layers of 200 2374 against 2823.
// ---------------------------------------------------------------------------
constexpr int DS_RUN = 1024;
constexpr int DS_LIST = 2 * DS_RUN;
constexpr int DS_BUCKETS = 1024;
constexpr int DS_PER = DS_LIST / 256;   // keys per thread
constexpr uint32_t DS_CROWD = 96, DS_CROWD_LONG = 256;

// Where element i (key `key`) of a run of length w goes when runs are merged
// pairwise: `get(j)` reads the key at index j of the current array of length n.
template <class Get>
__device__ __forceinline__ uint32_t merge_position(uint32_t i, unsigned long long key, uint32_t w, uint32_t n,
                                                   Get&& get) {
  const uint32_t lo = i - i % w;
  const bool left = ((i / w) & 1u) == 0u;
  uint32_t a = left ? min(lo + w, n) : lo - w;   // the other run [a, b)
  const uint32_t a0 = a;
  uint32_t b = left ? min(lo + 2 * w, n) : lo;
  while (a < b) {
    const uint32_t mid = (a + b) >> 1;
    if (get(mid) < key) a = mid + 1;
    else b = mid;
  }
  return (left ? lo : lo - w) + (i - lo) + (a - a0);
}

// Sort k[0, m) (m <= DS_RUN) in LDS, t as the second buffer; returns the
// buffer that holds the result.
__device__ __forceinline__ unsigned long long* lds_merge_sort(unsigned long long* k, unsigned long long* t,
                                                              uint32_t m) {
  for (uint32_t w = 1; w < m; w <<= 1) {
    for (uint32_t i = threadIdx.x; i < m; i += blockDim.x) {
      const unsigned long long key = k[i];
      t[merge_position(i, key, w, m, [&](uint32_t j) { return k[j]; })] = key;
    }
    __syncthreads();
    unsigned long long* x = k; k = t; t = x;
  }
  return k;
}

// The merge sort of a tile's list: items rv[0, n) by (zkey[record], item),
// through the scratch pair xk, xv, with the tile keys rk as scratch too
// (rewritten by the caller).
__device__ __forceinline__ void merge_sort_list(uint32_t* rk, uint32_t* rv, uint32_t* xk, uint32_t* xv,
                                                const uint32_t* zkey, uint32_t n, unsigned long long* lds) {
  for (uint32_t r0 = 0; r0 < n; r0 += DS_RUN) {
    const uint32_t m = min((uint32_t)DS_RUN, n - r0);
    for (uint32_t i = threadIdx.x; i < m; i += blockDim.x) {
      const uint32_t r = rv[r0 + i];
      lds[i] = ((unsigned long long)zkey[r >> 1] << 32) | r;
    }
    __syncthreads();
    const unsigned long long* srt = lds_merge_sort(lds, lds + DS_RUN, m);
    if (n <= (uint32_t)DS_RUN) {
      for (uint32_t i = threadIdx.x; i < m; i += blockDim.x) rv[i] = (uint32_t)srt[i];
      __syncthreads();
      return;
    }
    for (uint32_t i = threadIdx.x; i < m; i += blockDim.x) {
      xk[r0 + i] = (uint32_t)(srt[i] >> 32);
      xv[r0 + i] = (uint32_t)srt[i];
    }
    __syncthreads();
  }
  // pairwise merges of the runs in HBM: scratch -> result pair -> scratch ...
  uint32_t *ak = xk, *av = xv, *bk = rk, *bv = rv;
  for (uint32_t w = DS_RUN; w < n; w <<= 1) {
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
      const unsigned long long key = ((unsigned long long)ak[i] << 32) | av[i];
      const uint32_t pos = merge_position(i, key, w, n, [&](uint32_t j) {
        return ((unsigned long long)ak[j] << 32) | av[j];
      });
      bk[pos] = (uint32_t)(key >> 32);
      bv[pos] = (uint32_t)key;
    }
    __syncthreads();
    uint32_t* t = ak; ak = bk; bk = t;
    t = av; av = bv; bv = t;
  }
  if (av != rv)
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) rv[i] = av[i];
  __syncthreads();
}

struct DepthSort {
  unsigned long long key[DS_LIST];   // the keys of the list, or of a group of its buckets
  uint32_t cnt[DS_BUCKETS];          // per bucket its count, then its first place, then its end
  uint32_t red[8];
};

__device__ __forceinline__ void block_min_max(uint32_t& lo, uint32_t& hi, uint32_t* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
  }
  if ((threadIdx.x & 63u) == 0u) {
    red[threadIdx.x >> 6] = lo;
    red[4 + (threadIdx.x >> 6)] = hi;
  }
  __syncthreads();
  lo = min(min(red[0], red[1]), min(red[2], red[3]));
  hi = max(max(red[4], red[5]), max(red[6], red[7]));
}

// exclusive scan of the bucket counts in place (every thread; ends with a barrier)
__device__ __forceinline__ void scan_buckets(DepthSort& S) {
  constexpr int PER = DS_BUCKETS / 256;
  const uint32_t t = threadIdx.x, wave = t >> 6;
  uint32_t c[PER], sum = 0u;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    c[i] = sum;
    sum += S.cnt[t * PER + i];
  }
  const uint32_t x = wave_scan_add(sum);
  __syncthreads();   // (red is also block_min_max's)
  if ((t & 63u) == 63u) S.red[wave] = x;
  __syncthreads();
  uint32_t base = x - sum;
  for (uint32_t w = 0; w < wave; ++w) base += S.red[w];
#pragma unroll
  for (int i = 0; i < PER; ++i) S.cnt[t * PER + i] = base + c[i];
  __syncthreads();
}

struct BucketOf {
  uint32_t lo;
  float scale;
  __device__ __forceinline__ uint32_t operator()(uint32_t z) const {
    return min((uint32_t)((float)(z - lo) * scale), (uint32_t)DS_BUCKETS - 1u);
  }
};

// The place of a key among the list's (or group's) keys in bucket order:
// [p0, p1) are its bucket's.
__device__ __forceinline__ uint32_t bucket_place(const unsigned long long* k, uint32_t p0, uint32_t p1,
                                                 unsigned long long key) {
  uint32_t p = p0;
  for (uint32_t j = p0; j < p1; ++j) p += k[j] < key ? 1u : 0u;
  return p;
}

// n <= DS_LIST; false, with rv unchanged, if a bucket is crowded
__device__ __forceinline__ bool bucket_sort_list(uint32_t* rv, const uint32_t* zkey, uint32_t n, DepthSort& S) {
  const uint32_t t = threadIdx.x;
  uint32_t z[DS_PER], r[DS_PER], lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int i = 0; i < DS_PER; ++i) {
    if (256u * i >= n) break;
    r[i] = t + 256u * i < n ? rv[t + 256u * i] : 0u;
  }
#pragma unroll
  for (int i = 0; i < DS_PER; ++i) {
    if (256u * i >= n) break;
    const bool in = t + 256u * i < n;
    z[i] = in ? zkey[r[i] >> 1] : 0u;
    lo = min(lo, in ? z[i] : 0xffffffffu);
    hi = max(hi, in ? z[i] : 0u);
  }
  for (uint32_t i = t; i < (uint32_t)DS_BUCKETS; i += 256u) S.cnt[i] = 0u;
  block_min_max(lo, hi, S.red);
  const BucketOf bucket{lo, (float)DS_BUCKETS / ((float)(hi - lo) + 1.0f)};
  uint32_t rank[DS_PER], crowd = 0u;
#pragma unroll
  for (int i = 0; i < DS_PER; ++i) {
    if (256u * i >= n) break;
    rank[i] = t + 256u * i < n ? atomicAdd(&S.cnt[bucket(z[i])], 1u) : 0u;
    crowd = max(crowd, rank[i]);
  }
  if (__syncthreads_or((int)(crowd >= DS_CROWD))) return false;
  scan_buckets(S);
  // into bucket order (inside a bucket: whatever the atomics gave)
#pragma unroll
  for (int i = 0; i < DS_PER; ++i) {
    if (256u * i >= n) break;
    if (t + 256u * i < n) S.key[S.cnt[bucket(z[i])] + rank[i]] = ((unsigned long long)z[i] << 32) | r[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < DS_PER; ++i) {
    if (256u * i >= n) break;
    if (t + 256u * i >= n) continue;
    const uint32_t b = bucket(z[i]);
    rank[i] = bucket_place(S.key, S.cnt[b], b + 1u < (uint32_t)DS_BUCKETS ? S.cnt[b + 1u] : n,
                           ((unsigned long long)z[i] << 32) | r[i]);
  }
  __syncthreads();
  // the records in order, left in LDS
  uint32_t* out = reinterpret_cast<uint32_t*>(S.key);
#pragma unroll
  for (int i = 0; i < DS_PER; ++i) {
    if (256u * i >= n) break;
    if (t + 256u * i < n) out[rank[i]] = r[i];
  }
  __syncthreads();
  return true;
}

// any n: the depths go to xk once, then each group of consecutive buckets
// with at most DS_LIST keys is picked out of the list and sorted into xv
__device__ __forceinline__ bool bucket_sort_long(uint32_t* rv, uint32_t* xk, uint32_t* xv, const uint32_t* zkey,
                                                 uint32_t n, DepthSort& S) {
  const uint32_t t = threadIdx.x;
  uint32_t lo = 0xffffffffu, hi = 0u;
  for (uint32_t i = t; i < n; i += 256u) {
    const uint32_t z = zkey[rv[i] >> 1];
    xk[i] = z;
    lo = min(lo, z);
    hi = max(hi, z);
  }
  for (uint32_t i = t; i < (uint32_t)DS_BUCKETS; i += 256u) S.cnt[i] = 0u;
  block_min_max(lo, hi, S.red);
  const BucketOf bucket{lo, (float)DS_BUCKETS / ((float)(hi - lo) + 1.0f)};
  uint32_t crowd = 0u;
  for (uint32_t i = t; i < n; i += 256u) crowd = max(crowd, atomicAdd(&S.cnt[bucket(xk[i])], 1u));
  if (__syncthreads_or((int)(crowd >= DS_CROWD_LONG))) return false;
  scan_buckets(S);
  for (uint32_t g0 = 0; g0 < (uint32_t)DS_BUCKETS;) {
    // cnt still holds first places from g0 on: the group ends before the
    // first bucket whose end is past the group's room
    const uint32_t p0 = S.cnt[g0];
    uint32_t a = g0 + 1u, b = (uint32_t)DS_BUCKETS;
    while (a < b) {
      const uint32_t mid = (a + b + 1u) >> 1;
      if ((mid < (uint32_t)DS_BUCKETS ? S.cnt[mid] : n) - p0 <= (uint32_t)DS_LIST) a = mid;
      else b = mid - 1u;
    }
    const uint32_t g1 = a;
    __syncthreads();
    for (uint32_t i = t; i < n; i += 256u) {
      const uint32_t z = xk[i], q = bucket(z);
      // (after its additions a bucket's cnt is its end, the next one's start)
      if (q >= g0 && q < g1) S.key[atomicAdd(&S.cnt[q], 1u) - p0] = ((unsigned long long)z << 32) | rv[i];
    }
    __syncthreads();
    const uint32_t m = S.cnt[g1 - 1u] - p0;
    for (uint32_t i = t; i < m; i += 256u) {
      const unsigned long long key = S.key[i];
      const uint32_t q = bucket((uint32_t)(key >> 32));
      xv[p0 + bucket_place(S.key, (q > g0 ? S.cnt[q - 1u] : p0) - p0, S.cnt[q] - p0, key)] = (uint32_t)key;
    }
    __syncthreads();
    g0 = g1;
  }
  for (uint32_t i = t; i < n; i += 256u) rv[i] = xv[i];
  return true;
}

// An item of a list is its record's index, shifted up, and in bit 0 whether the
// record cannot blend.  With blend_lists the records that can also go to a list
// of their own (their index in the full list beside them), which the
// compositing kernels walk: half the entries or more face away from the camera
// or cover no pixel's centre, and a tile's walk is a serial chain of chunks.
// 19 to 21 us at 4 x 512^2, 122 to 140 at 8 x 1024^2, for 69 to 67 and 59 to 50
// us in the two walks there (634 to 594 in the forward, the backward's pairs
// bound at 590), 151 + 237 to 138 + 217 with the resort window of five.
//   Past DS_GRID lists a workgroup takes several, far apart in the dispatch order:
// a workgroup per tile, most of which only leave, cost 97 us of a 4096^2 frame
// (262k tiles) of an object a fifth as wide, 22 so.
constexpr unsigned DS_GRID = 32768;
__global__ __launch_bounds__(256) void k_tile_depth_sort(void* ws, Layout L, int blend_lists) {
  __shared__ DepthSort S;
  static_assert(DS_LIST >= 2 * DS_RUN, "the merge sort's two LDS buffers");
  const uint32_t n_empty = at<const uint32_t>(ws, L.o_tile_hist)[0];
  const uint32_t t = threadIdx.x, n_work = (uint32_t)L.total_tiles - n_empty;
  for (uint32_t slot = blockIdx.x; slot < n_work; slot += gridDim.x) {
    const TileSlot sl = at<const TileSlot>(ws, L.o_tile_order)[slot];
    const uint32_t s0 = sl.start, n = sl.end - sl.start;
    uint32_t* rk = at<uint32_t>(ws, sorted_tile_keys(L)) + s0;       // result pair: tile keys, records
    uint32_t* rv = at<uint32_t>(ws, sorted_entry_records(L)) + s0;
    const uint32_t* zkey = at<const uint32_t>(ws, L.o_key1a);        // depth bits per record
    // scratch pair, then the blend lists
    uint32_t* xk = at<uint32_t>(ws, blend_entry_index(L)) + s0;
    uint32_t* xv = at<uint32_t>(ws, blend_entry_records(L)) + s0;
    const uint32_t* src = rv;
    if (n > 1u) {
      bool done;
      if (n <= (uint32_t)DS_LIST) {
        done = bucket_sort_list(rv, zkey, n, S);
        if (done) src = reinterpret_cast<const uint32_t*>(S.key);
      } else {
        done = bucket_sort_long(rv, xk, xv, zkey, n, S);
      }
      if (!done) merge_sort_list(rk, rv, xk, xv, zkey, n, S.key);
    }
    __syncthreads();
    uint32_t m = 0u;   // of the blend list so far
    for (uint32_t i0 = 0; i0 < n; i0 += 256u) {
      const uint32_t i = i0 + t, v = i < n ? src[i] : 1u;
      if (i < n) {
        rv[i] = v >> 1;
        rk[i] = sl.tile;   // the list's tile keys
      }
      if (!blend_lists) continue;
      const uint64_t b = __ballot((v & 1u) == 0u);
      if ((t & 63u) == 0u) S.red[t >> 6] = (uint32_t)__popcll(b);
      __syncthreads();
      uint32_t o = m + (uint32_t)__popcll(b & ((1ull << (t & 63u)) - 1ull));
#pragma unroll
      for (uint32_t w = 0; w < 4u; ++w) {
        o += w < t >> 6 ? S.red[w] : 0u;
        m += S.red[w];
      }
      if ((v & 1u) == 0u) {
        xv[o] = v >> 1;
        xk[o] = s0 + i;
      }
      __syncthreads();
    }
    if (blend_lists && t == 0u) at<TileSlot>(ws, L.o_tile_order)[slot].end = s0 + m;
    __syncthreads();   // the next list takes the LDS
  }
}

hipError_t launch_tile_depth_sort(void* ws, const Layout& L, bool blend_lists, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  k_tile_depth_sort<<<std::min(working_tiles(L), DS_GRID), 256, 0, st>>>(ws, L, blend_lists ? 1 : 0);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// gradient buffers are overwritten: clear them first
// ---------------------------------------------------------------------------
// The scenes' gradients (row y: scene y); row 0 also clears the entry flags
// of the last forward's entries (the backward sets the ones it reaches).
__device__ __forceinline__ void zero_grads_body(const DevScene& S, void* ws, const Layout& L) {
  const size_t n3 = 3 * (size_t)S.V;
  const size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = i0; i < n3; i += stride) {
    S.dverts[i] = 0.0f;
    S.dcolors[i] = 0.0f;
    if (i < (size_t)S.V) S.dsdf[i] = 0.0f;
  }
  if (blockIdx.y != 0) return;
  const DevHeader* hdr = at<const DevHeader>(ws, L.o_hdr);
  uint32_t* f = at<uint32_t>(ws, L.o_eflag);
  const uint32_t words = (hdr->entries_total + 3u) / 4u;
  for (size_t i = i0; i < words; i += stride) f[i] = 0u;
  if (record_grads(L)) {
    // the records' gradient accumulators
    float4* acc = at<float4>(ws, L.o_tgrad);
    const size_t n4 = (size_t)min(hdr->records_total, (uint32_t)L.rec_cap) * (TGRAD_STRIDE / 4);
    for (size_t i = i0; i < n4; i += stride) acc[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
}

// Row ns of the grid (where the backward goes through pairs) writes the
// backward's dispatch order, which only needs the forward.  (In a launch of
// its own at the end of the forward it cost 8 us at the training shape.)
__global__ __launch_bounds__(256) void k_zero_grads(void* ws, Layout L) {
  if (blockIdx.y == (unsigned)L.ns) bwd_scatter(ws, L, blockIdx.x, gridDim.x);
  else zero_grads_body(at<const DevScene>(ws, L.o_scene)[blockIdx.y], ws, L);
}

// The same, taking the backward's descriptor image (scenes first) as the
// kernel argument: row 0 also writes it to the workspace for the kernels
// after this one, and every block reads its scene from the argument.
__global__ __launch_bounds__(256) void k_zero_grads_desc(Blob b, int nwords, void* ws, Layout L) {
  if (blockIdx.y == (unsigned)L.ns) {
    bwd_scatter(ws, L, blockIdx.x, gridDim.x);
    return;
  }
  if (blockIdx.y == 0) {
    uint32_t* dst = at<uint32_t>(ws, L.o_scene);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += gridDim.x * blockDim.x) dst[i] = b.w[i];
  }
  zero_grads_body(reinterpret_cast<const DevScene*>(b.w)[blockIdx.y], ws, L);
}

// Descriptor upload and gradient clearing of a backward pass: one launch when
// the descriptors fit in one kernel argument, else the upload launches and
// then the clearing kernel.
hipError_t launch_desc_zero_grads(const DevScene* hs, int ns, const DevView* hv, int nv, const int32_t* scene_views,
                                  void* ws, const Layout& L, hipStream_t st) {
  std::vector<uint8_t> img;
  size_t first;
  hipError_t e = desc_image(hs, ns, hv, nv, scene_views, L, false, img, first);
  if (e != hipSuccess) return e;
  dim3 grid(256, (unsigned)L.ns + (L.o_pairs != 0 && L.total_tiles > 0 ? 1u : 0u));
  const size_t words = img.size() / 4;
  if (words <= (size_t)BLOB_WORDS) {
    static_assert(alignof(DevScene) <= 16, "scenes start the image, which starts the argument");
    Blob b;
    std::memcpy(b.w, img.data(), img.size());
    k_zero_grads_desc<<<grid, 256, 0, st>>>(b, (int)words, ws, L);
  } else {
    e = upload(img.data(), img.size(), at<void>(ws, first), st);
    if (e != hipSuccess) return e;
    k_zero_grads<<<grid, 256, 0, st>>>(ws, L);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Coarse-to-fine pre-filtering (App. B): bounding box of the vertices of the
// kept tets.  Coordinates are reduced as order-preserving integer images of
// their float bits (min/max are exact and order-independent).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t ord_bits(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ord_float(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

__global__ void k_bounds_init(uint32_t* box, unsigned long long* kept) {
  const int t = threadIdx.x;
  if (t < 3) box[t] = 0xffffffffu;
  if (t >= 3 && t < 6) box[t] = 0u;
  if (t == 0 && kept) *kept = 0ull;
}

// Same-address atomics are what bounds a reduction like this one (one set of
// seven per wave: 284 us at 12.6 M tets, 70 us so): each block combines its
// waves first, and its first lanes then update only the bounds that it
// widens (a bound read here is at worst an older, narrower one).  What is
// left is the four SDF gathers per tet: four tets of a thread in flight took
// 83 us, the exponentials skipped well outside the surface 75 us.
__global__ __launch_bounds__(256) void k_pf_bounds(DevScene S, float tf, uint32_t* box, unsigned long long* kept) {
  __shared__ uint32_t red[7][4];
  uint32_t mn[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, mx[3] = {0u, 0u, 0u};
  uint32_t cnt = 0;
  for (int k = blockIdx.x * 256 + threadIdx.x; k < S.K; k += gridDim.x * 256) {
    int4 vi;
    if (!keep_tet(S, k, tf, nullptr, &vi)) continue;
    ++cnt;
    const int idx[4] = {vi.x, vi.y, vi.z, vi.w};
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const uint32_t u = ord_bits(S.verts[3 * (size_t)idx[a] + c]);
        mn[c] = min(mn[c], u);
        mx[c] = max(mx[c], u);
      }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mn[c] = min(mn[c], (uint32_t)__shfl_xor((int)mn[c], o, 64));
      mx[c] = max(mx[c], (uint32_t)__shfl_xor((int)mx[c], o, 64));
    }
    cnt += (uint32_t)__shfl_xor((int)cnt, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      red[c][w] = mn[c];
      red[3 + c][w] = mx[c];
    }
    red[6][w] = cnt;
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 3) {
    const uint32_t x = min(min(red[t][0], red[t][1]), min(red[t][2], red[t][3]));
    if (x < __hip_atomic_load(&box[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&box[t], x);
  } else if (t < 6) {
    const uint32_t x = max(max(red[t][0], red[t][1]), max(red[t][2], red[t][3]));
    if (x > __hip_atomic_load(&box[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&box[t], x);
  } else if (t == 6 && kept) {
    const uint32_t n = (red[6][0] + red[6][1]) + (red[6][2] + red[6][3]);
    if (n > 0u) atomicAdd(kept, (unsigned long long)n);
  }
}

// in place: integer images back to floats; NaN where nothing was kept
__global__ void k_bounds_final(uint32_t* box) {
  const int t = threadIdx.x;
  if (t < 6) {
    const uint32_t u = box[t];
    const bool empty = (t < 3) ? (u == 0xffffffffu) : (u == 0u);
    reinterpret_cast<float*>(box)[t] = empty ? __uint_as_float(0x7fc00000u) : ord_float(u);
  }
}

hipError_t launch_prefilter_bounds(const DevScene& S, float tf, float* bounds, int64_t* kept, hipStream_t st) {
  uint32_t* box = reinterpret_cast<uint32_t*>(bounds);
  unsigned long long* kp = reinterpret_cast<unsigned long long*>(kept);
  k_bounds_init<<<1, 64, 0, st>>>(box, kp);
  const unsigned g = (unsigned)std::max(1, std::min((S.K + 255) / 256, 2048));
  if (S.K > 0) k_pf_bounds<<<g, 256, 0, st>>>(S, tf, box, kp);
  k_bounds_final<<<1, 64, 0, st>>>(box);
  return hipGetLastError();
}



// ---------------------------------------------------------------------------
// Coarse-to-fine grid (App. B).  The second pass keeps the resolution R and
// cubic cells: a cube centred on the first pass's kept box, whose side is the
// box's largest extent plus one coarse cell on each side.  Arithmetic of the
// cube: extents in float32, side rounded to float32 from the double sum, the
// centre and low corner in double (rounded to float32 at the end), cell size
// side / R in float32.  An empty kept set (NaN box) keeps the input cube.
// ---------------------------------------------------------------------------
__global__ void k_refit_cube(const float* __restrict__ box, const float* __restrict__ cube_in, int R,
                             float* __restrict__ cube_out) {
  if (threadIdx.x != 0) return;
  float lo[3], hi[3];
  bool empty = false;
  for (int c = 0; c < 3; ++c) {
    lo[c] = box[c];
    hi[c] = box[3 + c];
    empty = empty || !(lo[c] == lo[c]) || !(hi[c] == hi[c]);
  }
  if (empty) {
    for (int c = 0; c < 4; ++c) cube_out[c] = cube_in[c];
    return;
  }
  float ext = hi[0] - lo[0];
  ext = fmaxf(ext, hi[1] - lo[1]);
  ext = fmaxf(ext, hi[2] - lo[2]);
  const double pad = 2.0 * (double)cube_in[3];
  const float side = (float)((double)ext + pad);
  const double half = (double)side * 0.5;
  for (int c = 0; c < 3; ++c) {
    const double mid = ((double)lo[c] + (double)hi[c]) * 0.5;
    cube_out[c] = (float)(mid - half);
  }
  cube_out[3] = side / (float)R;
}

// Vertex (x, y, z) = x + (R+1)(y + (R+1) z) at low + (x, y, z) h (float32:
// one product, one sum, no fused multiply-add); cell q = x + R(y + R z) holds
// tets 6q + p, p over the six axis orders (a, b, c) in lexicographic order,
// with vertices (v0, v0 + e_a, v0 + e_a + e_b, v0 + (1, 1, 1)).
// One row (y, z) of the grid per wave and step: a row's positions and its
// 6 R tets are contiguous, and its threads take consecutive words (float,
// int4) of them, so that no index needs a 64-bit division by the grid's size
// and every store is contiguous across the wave (R = 128, with and without
// tets: 73 us to 43 us together).
__global__ __launch_bounds__(256) void k_cube_grid(int R, const float* __restrict__ cube, float* __restrict__ verts,
                                                   int4* __restrict__ tets) {
  const uint32_t n = (uint32_t)R + 1u, rows = n * n;
  const float low[3] = {cube[0], cube[1], cube[2]}, h = cube[3];
  const uint32_t lane = threadIdx.x & 63u;
  const int sx = 1, sy = (int)n, sz = (int)rows, diag = sx + sy + sz;
  for (uint32_t row = blockIdx.x * 4u + (threadIdx.x >> 6); row < rows; row += gridDim.x * 4u) {
    const uint32_t z = row / n, y = row - z * n;
    float* vr = verts + 3 * (size_t)row * n;
    const float py = low[1] + (float)y * h, pz = low[2] + (float)z * h;
    for (uint32_t i = lane; i < 3u * n; i += 64u) {
      const uint32_t x = i / 3u, c = i - 3u * x;
      vr[i] = c == 0u ? low[0] + (float)x * h : c == 1u ? py : pz;
    }
    if (!tets || y == (uint32_t)R || z == (uint32_t)R) continue;
    int4* tr = tets + 6 * ((size_t)z * R + y) * R;
    for (uint32_t i = lane; i < 6u * (uint32_t)R; i += 64u) {
      const uint32_t x = i / 6u, p = i - 6u * x;
      const int v0 = (int)(row * n + x);
      // axis orders (0,1,2) (0,2,1) (1,0,2) (1,2,0) (2,0,1) (2,1,0): first axis, and
      // the one left out of the first two
      const int a1 = p < 2u ? sx : p < 4u ? sy : sz;
      const int last = (p == 0u || p == 2u) ? sz : (p == 1u || p == 4u) ? sy : sx;
      tr[i] = make_int4(v0, v0 + a1, v0 + (diag - last), v0 + diag);
    }
  }
}

hipError_t launch_refit_cube(const float* bounds, const float* cube_in, int R, float* cube_out, hipStream_t st) {
  k_refit_cube<<<1, 64, 0, st>>>(bounds, cube_in, R, cube_out);
  return hipGetLastError();
}

hipError_t launch_cube_grid(int R, const float* cube, float* verts, int32_t* tets, hipStream_t st) {
  const uint32_t rows = (uint32_t)(R + 1) * (uint32_t)(R + 1);
  const unsigned blocks = std::min((rows + 3u) / 4u, 8192u);
  k_cube_grid<<<blocks, 256, 0, st>>>(R, cube, verts, reinterpret_cast<int4*>(tets));
  return hipGetLastError();
}

}  // namespace ts
