// raster.hip — front-to-back compositing (3D-GS rasteriser that the paper's
// Sec. II "Parallel Training" runs per partition) and its reverse replay.
//
// Layout on gfx950: one wave64 per bin tile.  A 16x16 tile gives each lane 4
// pixels of one column, so every Gaussian staged in LDS is read once per 4
// evaluations and the backward's wave reduction is amortised over 256
// pixels.  Gaussians are staged 64 at a time (one gathered record per lane).
// The forward can also split a tile's pixels over 2 or 4 waves of one
// work-group (each wave walks the whole list for its rows, with its own LDS
// batch): all tiles of a 1080p view are resident at once, so the forward's
// time is set by its longest lists, and more waves per tile shorten them.
// Work-group ids are remapped so that neighbouring tiles run on the same
// XCD and share its L2.
//
// The backward recovers each pixel's transmittance by dividing T_final by
// (1 - alpha) in reverse order (STORED) or first replays the forward for its
// blocks (RECOMPUTE).  The 9 gradient components of an entry are summed over
// the wave with lane swaps and DPP and added with one FP32 atomic each.
#include <algorithm>

#include "gs_device.h"

namespace gsmi {

constexpr int kRasterWave = 64;
// A forward wave's LDS batch: 64 entries and the two that its loop reads ahead.
constexpr int kFwdSlots = kRasterWave + 2;

// XCD-aware tile order: work-group i runs on XCD (i mod 8), and the XCDs take
// runs of consecutive tiles in turn: neighbours that share Gaussians share an
// L2.  Of a few images the runs are kXcdTiles long, so that an image's middle
// rows, whose lists are the longest, do not all fall to two XCDs (an eighth of
// the image to each instead: 1M Gaussians at 1920x1080, whole forward 389 us,
// runs of 4, 8 or 32 tiles 223-227 us; two images 368 / 309, six 802 / 779).
// Of a multiple of 8 images each XCD takes whole ones: the XCDs' shares are
// equal then, and an image's Gaussians stay in one L2 (runs of 8 tiles / whole
// images: backward of 32 images of 640x360 2861 / 2672 us, with stored sums
// 4910 / 4215; 64 of 128x128, forward 118 / 87).
constexpr int64_t kXcdTiles = 8;

__device__ __forceinline__ int64_t tile_of_block(uint32_t i, uint32_t run) {
  const uint32_t j = i >> 3;
  return (int64_t)(j / run * 8 + (i & 7)) * run + j % run;
}
static int64_t xcd_run(int64_t n_tiles, int64_t tiles_per_slot) {
  const int64_t slots = n_tiles / std::max<int64_t>(tiles_per_slot, 1);
  return slots > 0 && slots % 8 == 0 ? slots / 8 * tiles_per_slot : kXcdTiles;
}

// A projected record as three 16-byte words (mean, conic, opacity, rgb).
struct RawSplat {
  float4 a, b, c;
};

__device__ __forceinline__ RawSplat fetch_splat(const float* __restrict__ rec, uint32_t id) {
  const float4* r = reinterpret_cast<const float4*>(rec + (int64_t)id * GS_REC_STRIDE);
  return RawSplat{r[0], r[1], r[2]};
}

__device__ __forceinline__ Splat make_splat(const RawSplat& raw) {
  const float4 a = raw.a, b = raw.b, c = raw.c;
  Splat s;
  s.pad1 = s.pad2 = 0.0f;
  s.mx = a.x;
  s.my = a.y;
  s.A = -0.5f * kLog2e * a.z;
  s.B = -kLog2e * a.w;
  s.C = -0.5f * kLog2e * b.x;
  s.o = b.y;
  s.r = b.z;
  s.g = b.w;
  s.b = c.x;
  s.thr = -__builtin_amdgcn_logf(255.0f * b.y);   // -log2(255 o)
  return s;
}

__device__ __forceinline__ Splat load_splat(const float* __restrict__ rec, uint32_t id) {
  return make_splat(fetch_splat(rec, id));
}

template <int TW, int TH>
struct TileGeom {
  static constexpr int PX = TW * TH / kRasterWave;      // pixels per lane
  static constexpr int RSTEP = kRasterWave / TW;        // rows between a lane's pixels
  static_assert(TW * TH % kRasterWave == 0 && kRasterWave % TW == 0, "tile shape");
};

// Orders one wave's LDS accesses: the wave's staged batch is private to it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Pixel-centre box of the pixels a wave owns (for the entry cull).
struct PixBox {
  float x0, x1, y0, y1;
};

// The forward's walk over one staged batch.  Only entries that may reach the
// wave's box are kept, packed in list order, so that a visit costs an address
// increment and no bit scan; pad1 carries the list position.  Entry i + 1 is
// read while i is composited (two register sets alternate), its colour with
// the words of the skip test: read behind the test's branch, it made a lone
// wave wait for the LDS at every blend.  What a visit costs in instructions,
// scalar ones included, is what counts: the longest lists' waves run on alone
// after the others (1080p: 150 us of 360 for lists of 6400 entries), and there
// a wave issues one instruction in about 5 cycles.  70 -> 45 instructions a
// blending visit: 1920x1080 forward 361 -> 308 us, 8 partitions x 4 views 595
// -> 519, 3-band colour at 1024x830 216 -> 176; split forward at 4K, part 745
// -> 624.
struct FwdEntry {
  float4 g;                 // mx, my, A, B
  float2 h;                 // C, thr
  float4 col;               // o, r, g, b
};

__device__ __forceinline__ FwdEntry fwd_entry(const Splat* s) {
  return FwdEntry{*reinterpret_cast<const float4*>(s), *reinterpret_cast<const float2*>(&s->C),
                  *reinterpret_cast<const float4*>(&s->o)};
}

// Packs the lanes' hits into s_splat (kFwdSlots entries); returns their number.
__device__ __forceinline__ int fwd_pack(Splat& s, bool hit, int pos, Splat* s_splat) {
  const uint64_t hits = __ballot(hit);
  const int cnt = __builtin_popcountll(hits);
  wave_sync();
  if (hit) {
    s.pad1 = __builtin_bit_cast(float, pos);
    s_splat[__builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u))] = s;
  }
  s_splat[cnt].thr = INFINITY;        // an odd count's partner passes no test
  wave_sync();
  return cnt;
}

// body(entry, packed index) for the cnt packed entries, in order.
template <typename F>
__device__ __forceinline__ void fwd_for_each(const Splat* s_splat, int cnt, F&& body) {
  if (cnt) {
    FwdEntry ea = fwd_entry(s_splat);
    for (int i = 0;; i += 2) {
      const FwdEntry eb = fwd_entry(s_splat + i + 1);
      body(ea, i);
      ea = fwd_entry(s_splat + i + 2);
      body(eb, i + 1);
      if (i + 2 >= cnt) break;
    }
  }
}

// Falloff exponents of the lane's pixels and, per pixel, the lanes of mask
// live whose skip tests entry e passes; returns the union of the masks.
template <int PX>
__device__ __forceinline__ uint64_t fwd_test(const FwdEntry& e, float fx, const float* fy,
                                             const uint64_t (&live)[PX], float (&p2)[PX],
                                             uint64_t (&pass)[PX]) {
  // keeps the read of the colour with the others, ahead of the branch
  asm volatile("" ::"v"(e.col.x), "v"(e.col.y), "v"(e.col.z), "v"(e.col.w));
  Splat sp;
  sp.mx = e.g.x;
  sp.my = e.g.y;
  sp.A = e.g.z;
  sp.B = e.g.w;
  sp.C = e.h.x;
  sp.thr = e.h.y;
  splat_p2_column<PX>(sp, __fsub_rn(fx, sp.mx), fy, p2);
  uint64_t any = 0;
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    pass[k] = splat_pass_lanes(sp, p2[k]) & live[k];
    any |= pass[k];
  }
  return any;
}

// List position after the packed entry i.
__device__ __forceinline__ int fwd_pos(const Splat* s_splat, int i) {
  return __builtin_bit_cast(int, s_splat[i].pad1);
}

// Forward pass of one tile for one lane's PX pixels (pixel slots q0 + 64 k
// of the tile, slot = row * TW + column), which lie in the wave's box.
// WITH_COLOR=false is the replay used by the backward in RECOMPUTE mode.
// s_splat: this wave's LDS batch of kFwdSlots entries.
// CHUNKED (with colour) also prepares the chunked backward: boundary c is
// the list position (c+1)*chunk; for each pixel the forward stores at slot c
// of `ck` (ck[c * TW*TH + pixel]) the transmittance T_c there and the colour
// still to come behind it, normalised by T_c:
//   U_c = (sum over later blends of rgb alpha T + bg T_final) / T_c,
// built without cancellation from chunk-local composites (P = prod(1-alpha),
// L = sum rgb alpha T_local over a chunk) by U_c = L_{c+1} + P_{c+1} U_{c+1}
// after the tile is done.
template <int TW, int TH, int PX, bool WITH_COLOR, bool CHUNKED = false>
__device__ __forceinline__ void tile_forward(const float* __restrict__ rec,
                                             const uint32_t* __restrict__ ids, uint32_t start,
                                             uint32_t end, const float fx, const float* fy,
                                             const bool* inside, Splat* s_splat, float* T,
                                             float (*C)[3], int* last, const PixBox& box,
                                             float4* ck = nullptr, int chunk = 0, float bg0 = 0.f,
                                             float bg1 = 0.f, float bg2 = 0.f, int q0 = 0) {
  // one pixel a lane: the wave's pixels are an 8x8 block, row by row
  constexpr bool kBlock8 = PX == 1 && TW % 8 == 0 && TH % 8 == 0;
  const int lane = threadIdx.x & (kRasterWave - 1);
  // lanes whose pixel k still composites: inside the image and not stopped
  uint64_t live[PX];
  float Tl[PX], Lc[PX][3];
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    T[k] = 1.0f;
    last[k] = 0;
    live[k] = __ballot(inside[k]);
    if (WITH_COLOR) C[k][0] = C[k][1] = C[k][2] = 0.0f;
    if (CHUNKED) {
      Tl[k] = 1.0f;
      Lc[k][0] = Lc[k][1] = Lc[k][2] = 0.0f;
    }
  }
  uint32_t reached = 0;     // list entries processed (CHUNKED bookkeeping)
  // the next batch's records and the id of the one after are loaded while a
  // batch is composited, so a batch boundary does not wait on the two
  // dependent loads (id, then record)
  RawSplat nraw{};
  uint32_t nid2 = 0;
  if (start + lane < end) nraw = fetch_splat(rec, ids[start + lane]);
  if (start + kRasterWave + lane < end) nid2 = ids[start + kRasterWave + lane];
  for (uint32_t b0 = start; b0 < end; b0 += kRasterWave) {
    uint64_t any_live = 0;
#pragma unroll
    for (int k = 0; k < PX; ++k) any_live |= live[k];
    if (!any_live) break;
    const int n = (int)min((uint32_t)kRasterWave, end - b0);
    const RawSplat raw = nraw;
    const uint32_t nid = nid2;
    if (b0 + kRasterWave + lane < end) nraw = fetch_splat(rec, nid);
    if (b0 + 2 * kRasterWave + lane < end) nid2 = ids[b0 + 2 * kRasterWave + lane];
    // the cull's box: the wave's pixels, or of an 8x8 block the box of those
    // that still composite.  A long list's tail is for a few pixels only (at
    // 1080p the last wave to end visited 2628 entries, 823 of which blended
    // somewhere): forward 308 -> 233 us there, 176 -> 158 with 3-band colour.
    PixBox bx = box;
    if (kBlock8) {
      const uint64_t m = live[0];
      uint32_t c = (uint32_t)(m | (m >> 32));
      c |= c >> 16;
      c = (c | (c >> 8)) & 0xff;
      bx = PixBox{box.x0 + (float)__builtin_ctz(c), box.x0 + (float)(31 - __builtin_clz(c)),
                  box.y0 + (float)(__builtin_ctzll(m) >> 3),
                  box.y0 + (float)((63 - __builtin_clzll(m)) >> 3)};
    }
    Splat s = make_splat(raw);
    const bool hit = lane < n && splat_may_hit(s, bx.x0, bx.x1, bx.y0, bx.y1);
    const int cnt = fwd_pack(s, hit, (int)(b0 - start) + lane + 1, s_splat);
    int lastc[PX];            // packed index of the lane's last blend in the batch
#pragma unroll
    for (int k = 0; k < PX; ++k) lastc[k] = -1;
    fwd_for_each(s_splat, cnt, [&](const FwdEntry& e, int i) {
      float p2[PX];
      uint64_t pass[PX];
      if (!fwd_test<PX>(e, fx, fy, live, p2, pass)) return;
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        if (PX > 1 && !pass[k]) continue;
        const float alpha = fminf(kAlphaMax, e.col.x * splat_gauss(p2[k]));
        const float Tn = T[k] * (1.0f - alpha);
        const uint64_t stop = pass[k] & lanes_lt(Tn, kTMin);
        if (__builtin_expect(stop != 0, 0)) {   // rare: a branch, not mask operations a visit
          asm volatile("");
          live[k] &= ~stop;
          pass[k] &= ~stop;
        }
        if (lane_in(pass[k])) {
          if (WITH_COLOR) {
            const float w = alpha * T[k];
            C[k][0] = fmaf(e.col.y, w, C[k][0]);
            C[k][1] = fmaf(e.col.z, w, C[k][1]);
            C[k][2] = fmaf(e.col.w, w, C[k][2]);
          }
          if (CHUNKED) {
            const float wl = alpha * Tl[k];
            Lc[k][0] = fmaf(e.col.y, wl, Lc[k][0]);
            Lc[k][1] = fmaf(e.col.z, wl, Lc[k][1]);
            Lc[k][2] = fmaf(e.col.w, wl, Lc[k][2]);
            Tl[k] = Tl[k] * (1.0f - alpha);
          }
          T[k] = Tn;
          lastc[k] = i;
        }
      }
    });
#pragma unroll
    for (int k = 0; k < PX; ++k)
      if (lastc[k] >= 0) last[k] = fwd_pos(s_splat, lastc[k]);
    if (CHUNKED) {
      reached = b0 + (uint32_t)n - start;
      if (reached % (uint32_t)chunk == 0) {
        // chunk ce just ended: its local composite goes to slot ce-1
        const int ce = (int)(reached / chunk) - 1;
        if (ce >= 1) {
          float4* dst = ck + (int64_t)(ce - 1) * (TW * TH);
#pragma unroll
          for (int k = 0; k < PX; ++k)
            dst[q0 + k * kRasterWave] = make_float4(Tl[k], Lc[k][0], Lc[k][1], Lc[k][2]);
        }
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          Tl[k] = 1.0f;
          Lc[k][0] = Lc[k][1] = Lc[k][2] = 0.0f;
        }
      }
    }
  }
  if (CHUNKED && reached > 0) {
    // the partly processed last chunk (if any) and the reverse recursion
    int clast = (int)((reached - 1) / chunk);          // last chunk touched
    if (reached % (uint32_t)chunk != 0 && clast >= 1) {
      float4* dst = ck + (int64_t)(clast - 1) * (TW * TH);
#pragma unroll
      for (int k = 0; k < PX; ++k)
        dst[q0 + k * kRasterWave] = make_float4(Tl[k], Lc[k][0], Lc[k][1], Lc[k][2]);
    }
    float Tn[PX], U[PX][3];
#pragma unroll
    for (int k = 0; k < PX; ++k) {
      Tn[k] = T[k];
      U[k][0] = bg0;
      U[k][1] = bg1;
      U[k][2] = bg2;
    }
    for (int c = clast - 1; c >= 0; --c) {
      float4* slot = ck + (int64_t)c * (TW * TH);
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        const int q = q0 + k * kRasterWave;
        const float4 pl = slot[q];                          // (P, L) of chunk c+1
        const float Te = Tn[k] / pl.x;
        U[k][0] = fmaf(pl.x, U[k][0], pl.y);
        U[k][1] = fmaf(pl.x, U[k][1], pl.z);
        U[k][2] = fmaf(pl.x, U[k][2], pl.w);
        slot[q] = make_float4(Te, U[k][0], U[k][1], U[k][2]);
        Tn[k] = Te;
      }
    }
  }
}

// Per-call arguments shared by the forward and backward rasterisers.
struct RasterDev {
  const float* rec;
  const uint32_t* ids;
  const uint32_t* ranges;
  int W, H, tiles_x, tiles_per_slot;
  int64_t n_tiles;
  float bg0, bg1, bg2;
  // deterministic backward (NULL dup_grads: atomics into d_rec): emit[q]
  // is the emission index (gradient slot) of sorted entry q
  const uint32_t* emit;
  float* dup_grads;
  int64_t dup_cap;
};

// Deterministic mode: zero the gradient slots of list indices [lo, hi) of a
// tile (entries no pixel reaches), one entry per lane.
__device__ __forceinline__ void zero_dup_slots(const RasterDev& a, uint32_t start, int lo, int hi) {
  const int lane = threadIdx.x & (kRasterWave - 1);
  for (int q = lo + lane; q < hi; q += kRasterWave) {
    const uint32_t e = a.emit[start + q];
    if ((int64_t)e >= a.dup_cap) continue;
    float* g = a.dup_grads + (int64_t)e * GS_DREC_STRIDE;
#pragma unroll
    for (int c = 0; c < GS_DREC_STRIDE; ++c) g[c] = 0.0f;
  }
}

// Which tile a work-group processes: default XCD-aware order, a precomputed
// (longest-first) order, or a persistent grid pulling from an atomic queue.
struct TileSched {
  const uint32_t* order;   // NULL: XCD-aware default order
  uint32_t* queue;         // non-NULL: persistent launch, items pulled atomically
  uint32_t run;            // default order: consecutive tiles of an XCD (xcd_run)
};

// Chunked backward: every tile list is cut into `chunk`-entry work items;
// offset[t] is the first item of tile t (offset[n_tiles] = item count),
// items[i] the tile of item i; ck the forward checkpoints (T_c, U_c), one
// TW*TH float4 block per item.
struct ChunkDev {
  int chunk;
  const uint32_t* offset;
  const uint32_t* items;
  float4* ck;
};

// Calls body(tile, b) for the work-group's tiles; 1 << lg work-groups, b = 0 ..
// (1 << lg) - 1, share a tile (adjacent launches, or adjacent queue items).
template <typename F>
__device__ __forceinline__ void for_each_tile(const TileSched& sch, int64_t n_tiles, int lg,
                                              F&& body) {
  const uint32_t part = (1u << lg) - 1;
  if (sch.queue) {
    for (;;) {
      uint32_t item = 0;
      if (threadIdx.x == 0) item = atomicAdd(sch.queue, 1u);
      item = __builtin_amdgcn_readfirstlane(item);
      if ((int64_t)item >= n_tiles << lg) break;
      body((int64_t)(sch.order ? sch.order[item >> lg] : item >> lg), (int)(item & part));
    }
  } else if (sch.order) {
    const uint32_t i = blockIdx.x >> lg;
    if ((int64_t)i < n_tiles) body((int64_t)sch.order[i], (int)(blockIdx.x & part));
  } else {
    // consecutive work-groups of one XCD (ids 8 apart) share a tile
    const uint32_t j = blockIdx.x >> 3;
    const int64_t tile = tile_of_block((j >> lg) * 8 + (blockIdx.x & 7), sch.run);
    if (tile < n_tiles) body(tile, (int)(j & part));
  }
}

// Forward of one tile by wave w = threadIdx.x / 64 of NW; PX = TW TH / (64 NW)
// pixels per lane.  With one pixel per lane the wave owns an 8x8 block of
// the tile (blocks in row-major order), the most compact box for the entry
// cull; otherwise the rows ty TH + (w PX + k) RSTEP + lane / TW of column
// lane % TW.
template <int TW, int TH, int NW>
__device__ __forceinline__ void fwd_tile(const RasterDev& a, const ChunkDev& ch, int64_t tile,
                                         Splat* s_splat, float* __restrict__ image,
                                         float* __restrict__ T_final,
                                         int32_t* __restrict__ n_contrib) {
  constexpr int PX = TileGeom<TW, TH>::PX / NW, RSTEP = TileGeom<TW, TH>::RSTEP;
  static_assert(PX >= 1 && TileGeom<TW, TH>::PX % NW == 0, "waves per tile");
  constexpr bool kBlock8 = PX == 1 && TW % 8 == 0 && TH % 8 == 0;
  const int W = a.W, H = a.H;
  const int slot = (int)(tile / a.tiles_per_slot);
  const int t = (int)(tile - (int64_t)slot * a.tiles_per_slot);
  const int ty = t / a.tiles_x, tx = t - ty * a.tiles_x;
  const int lane = threadIdx.x & (kRasterWave - 1);
  const int w = threadIdx.x / kRasterWave;
  // the lane's column and first row inside the tile, and the wave's box
  const int lx = kBlock8 ? (w % (TW / 8)) * 8 + lane % 8 : lane % TW;
  const int ly0 = kBlock8 ? (w / (TW / 8)) * 8 + lane / 8 : lane / TW + w * PX * RSTEP;
  const int bxo = kBlock8 ? (w % (TW / 8)) * 8 : 0, bw = kBlock8 ? 8 : TW;
  const int byo = kBlock8 ? (w / (TW / 8)) * 8 : w * PX * RSTEP, bh = kBlock8 ? 8 : PX * RSTEP;
  const PixBox box{(float)(tx * TW + bxo) + 0.5f, (float)(tx * TW + bxo + bw - 1) + 0.5f,
                   (float)(ty * TH + byo) + 0.5f, (float)(ty * TH + byo + bh - 1) + 0.5f};
  const int px = tx * TW + lx;
  const int py0 = ty * TH + ly0;
  const float fx = (float)px + 0.5f;
  float fy[PX];
  bool inside[PX];
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    const int py = py0 + k * RSTEP;
    fy[k] = (float)py + 0.5f;
    inside[k] = (px < W) && (py < H);
  }
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  float T[PX], C[PX][3];
  int last[PX];
  if (ch.ck) {
    float4* ck = ch.ck + (int64_t)ch.offset[tile] * (TW * TH);
    tile_forward<TW, TH, PX, true, true>(a.rec, a.ids, start, end, fx, fy, inside, s_splat, T, C,
                                         last, box, ck, ch.chunk, a.bg0, a.bg1, a.bg2,
                                         ly0 * TW + lx);
  } else {
    tile_forward<TW, TH, PX, true>(a.rec, a.ids, start, end, fx, fy, inside, s_splat, T, C, last,
                                   box);
  }
  const int64_t HW = (int64_t)H * W;
  float* img = image + (int64_t)slot * 3 * HW;
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    if (!inside[k]) continue;
    const int64_t o = (int64_t)(py0 + k * RSTEP) * W + px;
    img[o] = C[k][0] + T[k] * a.bg0;
    img[HW + o] = C[k][1] + T[k] * a.bg1;
    img[2 * HW + o] = C[k][2] + T[k] * a.bg2;
    if (T_final) T_final[(int64_t)slot * HW + o] = T[k];
    if (n_contrib) n_contrib[(int64_t)slot * HW + o] = last[k];
  }
}

// Waves per SIMD that two 16x16 rasterisers are compiled for: 7 caps them at
// 72 VGPRs (80 unconstrained, i.e. 6 waves); the few spilled registers are
// reloaded at most once per 64-entry batch, never per entry.  Measured 2%
// faster for the forward on four waves (one pixel per lane) and for the
// chunked backward.  1 leaves the compiler free (other shapes spill heavily
// under the cap).
template <int TW, int TH, int NW>
constexpr int kFwdWavesPerEU = (TW == 16 && TH == 16 && NW == 4) ? 7 : 1;
template <int TW, int TH>
constexpr int kBwdWavesPerEU = (TW == 16 && TH == 16) ? 7 : 1;

template <int TW, int TH, int NW>
__global__ __launch_bounds__(kRasterWave * NW)
__attribute__((amdgpu_waves_per_eu(kFwdWavesPerEU<TW, TH, NW>)))
void k_raster_fwd(RasterDev a, TileSched sch,
                                                                 ChunkDev ch,
                                                                 float* __restrict__ image,
                                                                 float* __restrict__ T_final,
                                                                 int32_t* __restrict__ n_contrib) {
  __shared__ Splat s_splat[kFwdSlots * NW];
  // wave-uniform base (scalar), so per-entry LDS addresses stay scalar too
  Splat* mine = s_splat + __builtin_amdgcn_readfirstlane(threadIdx.x / kRasterWave) * kFwdSlots;
  for_each_tile(sch, a.n_tiles, 0, [&](int64_t tile, int) {
    fwd_tile<TW, TH, NW>(a, ch, tile, mine, image, T_final, n_contrib);
  });
}

__device__ __forceinline__ int wave_max_int(int v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = max(v, __shfl_xor(v, d, 64));
  return v;
}

// Reduce-scatter of the 9 gradient components of one list entry over the
// wave.  Stage 1 pairs lanes l and l ^ 32 with v_permlane32_swap, stage 2
// pairs l and l ^ 16 with v_permlane16_swap: swapping the halves of two
// component registers and adding gives, in every lane, one component summed
// over the lane pair, with no selects.  Stages 3-4 (partners l ^ 8 via
// row_ror:8, and l <-> 7 - (l mod 8) via row_half_mirror) keep one of two
// components per lane, and two quad_perm steps finish the sum.  Afterwards
// each group of 4 lanes holds the wave total of one component: 9 of the 16
// groups hold one each, and lanes 4k issue a single 9-lane atomic.
struct Scatter9 {
  int slot;       // component this lane's group holds (-1: none)
  float scale;    // its constant factor in d_rec
};

__device__ __forceinline__ Scatter9 scatter9_setup() {
  const int lane = threadIdx.x & (kRasterWave - 1);
  // which operand a lane keeps after each swap: push 0 / 1 through it
  const auto p32 = __builtin_amdgcn_permlane32_swap(0u, 1u, false, false);
  const auto p16 = __builtin_amdgcn_permlane16_swap(0u, 1u, false, false);
  const bool first32 = p32[0] == 0u, first16 = p16[0] == 0u;
  const int b3 = (lane >> 3) & 1, b2 = (lane >> 2) & 1;
  const int u = b2 == 0 ? (b3 ? 2 : 0) : (b3 ? -1 : 1);           // after stage 2
  const int w = u < 0 ? -1 : (first16 ? u : (u + 3 <= 4 ? u + 3 : -1));   // after stage 1
  const int v = w < 0 ? -1 : (first32 ? w : (w + 5 <= 8 ? w + 5 : -1));  // component
  // d mean2d carry -2 ln2 (the log2-scaled falloff), d Q11 and d Q22 -1/2,
  // d Q12 -1; opacity and colour 1
  const float sc[9] = {-2.0f * kLn2, -2.0f * kLn2, -0.5f, -1.0f, -0.5f, 1.0f, 1.0f, 1.0f, 1.0f};
  Scatter9 r;
  r.slot = ((lane & 3) == 0) ? v : -1;
  r.scale = v >= 0 ? sc[v] : 0.0f;
  return r;
}

__device__ __forceinline__ float swap_add32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float swap_add16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// v[0..8]: this lane's partial components; returns the wave total of the
// component named by scatter9_setup().slot (valid in every lane of its group).
__device__ __forceinline__ float reduce_scatter9(const float (&v)[9]) {
  const int lane = threadIdx.x & (kRasterWave - 1);
  // stage 1: 9 -> 5 (pairs (i, i + 5), v[9] = 0)
  const float w0 = swap_add32(v[0], v[5]);
  const float w1 = swap_add32(v[1], v[6]);
  const float w2 = swap_add32(v[2], v[7]);
  const float w3 = swap_add32(v[3], v[8]);
  const float w4 = swap_add32(v[4], 0.0f);
  // stage 2: 5 -> 3 (pairs (i, i + 3), w[5] = 0)
  const float u0 = swap_add16(w0, w3);
  const float u1 = swap_add16(w1, w4);
  const float u2 = swap_add16(w2, 0.0f);
  // stage 3: 3 -> 2 across l ^ 8: bit 3 clear keeps (u0, u1), set keeps (u2, -)
  const bool b3 = (lane >> 3) & 1;
  const float k0 = b3 ? u2 : u0, s0 = b3 ? u0 : u2;
  const float k1 = b3 ? 0.0f : u1, s1 = b3 ? u1 : 0.0f;
  const float t0 = k0 + dpp_f<kDppRowRor8>(s0);
  const float t1 = k1 + dpp_f<kDppRowRor8>(s1);
  // stage 4: 2 -> 1 across l <-> 7 - (l mod 8): bit 2 clear keeps t0
  const bool b2 = (lane >> 2) & 1;
  const float kk = b2 ? t1 : t0, ss = b2 ? t0 : t1;
  float z = kk + dpp_f<kDppRowHalfMirror>(ss);
  // stages 5-6: sum over the quad
  z += dpp_f<kDppQuadSwap1>(z);
  z += dpp_f<kDppQuadSwap2>(z);
  return z;
}

// ---------------------------------------------------------------- backward

// The backward walks 8x8 blocks of pixels, one pixel of each block per lane
// (lane l: column l mod 8, row l / 8).  A wave owns NK blocks, side by side
// in rows of BX: the blocks of a whole tile, or one of them.
template <int BX, int NK>
struct BwdPixels {
  float fx, fy;                   // the lane's pixel centre in block 0
  float T[NK], dIacc[NK];         // transmittance behind the walk's position; dI . colour behind it
  float dI[NK][3];
  int last[NK];                   // list position after the last blended entry (0: takes no part)
  bool inside[NK];
  int64_t o0, HW;                 // offset of the block-0 pixel in a plane; pixels per plane
  int W;
  // The pixels of the blocks from pixel (x0, y0).
  __device__ __forceinline__ BwdPixels(const RasterDev& a, int x0, int y0) {
    const int lane = threadIdx.x & (kRasterWave - 1);
    const int px = x0 + (lane & 7), py = y0 + (lane >> 3);
    W = a.W;
    HW = (int64_t)a.H * a.W;
    o0 = (int64_t)py * a.W + px;
    fx = (float)px + 0.5f;
    fy = (float)py + 0.5f;
#pragma unroll
    for (int k = 0; k < NK; ++k) inside[k] = px + 8 * (k % BX) < a.W && py + 8 * (k / BX) < a.H;
  }
  __device__ __forceinline__ int64_t offset(int k) const {
    return o0 + (int64_t)(8 * (k / BX)) * W + 8 * (k % BX);
  }
  // Loads the image gradients (dimg: the slot's planes) after last is set; a
  // pixel whose gradient is zero (a masked one) adds exactly zero to every
  // gradient and takes no part.  Returns the wave's largest last position.
  __device__ __forceinline__ int load_gradient(const float* __restrict__ dimg) {
    int lmax = 0;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int64_t o = offset(k);
      dI[k][0] = inside[k] ? dimg[o] : 0.0f;
      dI[k][1] = inside[k] ? dimg[HW + o] : 0.0f;
      dI[k][2] = inside[k] ? dimg[2 * HW + o] : 0.0f;
      if (dI[k][0] == 0.0f && dI[k][1] == 0.0f && dI[k][2] == 0.0f) last[k] = 0;
      lmax = max(lmax, last[k]);
    }
    return __builtin_amdgcn_readfirstlane(wave_max_int(lmax));
  }
  // State behind the whole list: dI . (I - C) = dI . bg T_final.
  __device__ __forceinline__ void final_state(int k, float T_fin, const RasterDev& a) {
    T[k] = T_fin;
    dIacc[k] = T_fin * (dI[k][0] * a.bg0 + dI[k][1] * a.bg1 + dI[k][2] * a.bg2);
  }
};

// Reverse replay of list positions (lo, hi] of one tile (entries start+lo ..
// start+hi-1, last first) for the wave's blocks, the first of which starts at
// pixel (x0, y0).  With a.dup_grads (the wave owns the whole tile) an entry's
// components go to its emission slot, else they are added atomically to
// d_rec.  mine: the entries (by slot of their batch) whose sums this wave
// takes; the others only move its pixels' transmittance on.
// The walk is bound by vector instruction issue.  A footprint reaches 1.3 of
// a 16x16 tile's four blocks on average (28 of 256 pixels blend at 1080p), so
// staging tests every block's box and a visit evaluates only the blocks that
// the entry may reach (a wave-uniform branch per block); the lanes then sum
// their blocks and one reduction over the wave serves the whole tile.
template <int BX, int NK>
__device__ __forceinline__ void reverse_pass(const RasterDev& a, uint32_t start, int lo, int hi,
                                             int x0, int y0, BwdPixels<BX, NK>& p, Splat* s_splat,
                                             float* __restrict__ d_rec, uint2* s_meta = nullptr,
                                             uint64_t mine = ~0ull) {
  const int lane = threadIdx.x & (kRasterWave - 1);
  const bool det = a.dup_grads != nullptr;
  float* const gbase = det ? a.dup_grads : d_rec;
  const Scatter9 red = scatter9_setup();
  const float bx = (float)x0 + 0.5f, by = (float)y0 + 0.5f;
  for (int top = hi; top > lo; top -= kRasterWave) {
    const int bot = max(lo, top - kRasterWave);
    const int n = top - bot;
    wave_sync();
    uint32_t reach = 0;               // blocks the lane's entry may reach
    uint32_t eid = 0;                 // its pair, or gradient slot
    Splat staged{};
    if (lane < n) {
      const uint32_t id = a.ids[start + bot + lane];
      eid = det ? a.emit[start + bot + lane] : id;
      Splat s = load_splat(a.rec, id);
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const float gx = bx + (float)(8 * (k % BX)), gy = by + (float)(8 * (k / BX));
        if (splat_may_hit(s, gx, gx + 7.0f, gy, gy + 7.0f)) reach |= 1u << k;
      }
      s.pad1 = __builtin_amdgcn_rcpf(s.o);
      s.pad2 = 0.5f * s.B;
      if (NK == 1) staged = s;
      else s_splat[lane] = s;
      // an entry that cannot reach the tile gets zero gradients
      if (det && !reach && (mine >> lane & 1) && (int64_t)eid < a.dup_cap) {
        float* g = gbase + (int64_t)eid * GS_DREC_STRIDE;
#pragma unroll
        for (int c = 0; c < GS_DREC_STRIDE; ++c) g[c] = 0.0f;
      }
    }
    // moves pixel k's state in front of an entry that it blends
    struct Step {
      float aa, alpha, w, dLda;
    };
    auto step = [&](const Splat& sp, int k, float p2) {
      Step b;
      b.aa = sp.o * splat_gauss(p2);
      b.alpha = fminf(kAlphaMax, b.aa);
      const float inv = __builtin_amdgcn_rcpf(1.0f - b.alpha);
      const float Tb = p.T[k] * inv;                 // transmittance in front of it
      b.w = b.alpha * Tb;
      const float dIc = fmaf(p.dI[k][2], sp.b, fmaf(p.dI[k][1], sp.g, p.dI[k][0] * sp.r));
      b.dLda = fmaf(Tb, dIc, -inv * p.dIacc[k]);
      p.dIacc[k] = fmaf(b.w, dIc, p.dIacc[k]);
      p.T[k] = Tb;
      return b;
    };
    // an entry whose sums another wave takes
    auto pass_by = [&](const Splat& sp, uint32_t blocks, int pos) {
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        if (NK > 1 && !(blocks & (1u << k))) continue;
        const float p2 = splat_p2(sp, __fsub_rn(p.fx + (float)(8 * (k % BX)), sp.mx),
                                  __fsub_rn(p.fy + (float)(8 * (k / BX)), sp.my));
        if (lane_in(splat_pass_lanes(sp, p2) & lanes_le(pos, p.last[k]))) step(sp, k, p2);
      }
    };
    // one entry, its blocks, pair (or gradient slot) and list position
    auto visit = [&](const Splat& sp, uint32_t blocks, uint32_t entry, int pos, bool take) {
      if (!take) {
        pass_by(sp, blocks, pos);
        return;
      }
      // sums over the lane's pixels of G = dL/d(exponent) times 1, dx, dy,
      // dx^2, dx dy, dy^2 and of the blend weight times dI
      float sG = 0.f, sGx = 0.f, sGy = 0.f, sGxx = 0.f, sGxy = 0.f, sGyy = 0.f;
      float sr = 0.f, sg = 0.f, sb = 0.f;
      uint64_t hit = 0;
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        if (NK > 1 && !(blocks & (1u << k))) continue;
        const float dx = __fsub_rn(p.fx + (float)(8 * (k % BX)), sp.mx);
        const float dy = __fsub_rn(p.fy + (float)(8 * (k / BX)), sp.my);
        const float p2 = splat_p2(sp, dx, dy);
        const uint64_t pass = splat_pass_lanes(sp, p2) & lanes_le(pos, p.last[k]);
        hit |= pass;
        if (lane_in(pass)) {
          const Step b = step(sp, k, p2);
          sr = fmaf(p.dI[k][0], b.w, sr);
          sg = fmaf(p.dI[k][1], b.w, sg);
          sb = fmaf(p.dI[k][2], b.w, sb);
          // (the derivative through a clamped alpha is zero)
          const float G = b.aa < kAlphaMax ? b.dLda * b.alpha : 0.0f;
          const float Gx = G * dx, Gy = G * dy;
          sG += G;
          sGx += Gx;
          sGy += Gy;
          sGxx = fmaf(Gx, dx, sGxx);
          sGxy = fmaf(Gx, dy, sGxy);
          sGyy = fmaf(Gy, dy, sGyy);
        }
      }
      if (!hit) {
        if (det && lane < GS_DREC_STRIDE && (int64_t)entry < a.dup_cap)
          gbase[(int64_t)entry * GS_DREC_STRIDE + lane] = 0.0f;
        return;
      }
      // (constant factors applied per component after the reduction)
      const float comp[9] = {fmaf(sp.A, sGx, sp.pad2 * sGy),    // d mx / -2 ln2
                             fmaf(sp.C, sGy, sp.pad2 * sGx),    // d my / -2 ln2
                             sGxx,                              // d Q11 / -1/2
                             sGxy,                              // d Q12 / -1
                             sGyy,                              // d Q22 / -1/2
                             sG * sp.pad1,                      // d o
                             sr, sg, sb};
      const float tot = reduce_scatter9(comp);
      if (red.slot >= 0) {
        float* dst = gbase + (int64_t)entry * GS_DREC_STRIDE + red.slot;
        if (!det) atomicAdd(dst, red.scale * tot);
        else if ((int64_t)entry < a.dup_cap) *dst = red.scale * tot;
      }
    };
    const uint64_t hits = __ballot(reach != 0);
    if constexpr (NK == 1) {
      // packed last entry first, the next one read while one is visited
      const int cnt = __builtin_popcountll(hits);
      if (reach) {
        const int i = cnt - 1 - (int)__builtin_amdgcn_mbcnt_hi(
                                    (uint32_t)(hits >> 32),
                                    __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
        s_splat[i] = staged;
        s_meta[i] = make_uint2(eid, (uint32_t)(bot + lane + 1));
      }
      wave_sync();
      if (cnt) {
        Splat ea = s_splat[0], eb;
        uint2 ma = s_meta[0], mb;
        for (int i = 0;; i += 2) {
          eb = s_splat[i + 1];
          mb = s_meta[i + 1];
          visit(ea, 1u, __builtin_amdgcn_readfirstlane(ma.x), (int)ma.y, mine >> i & 1);
          if (i + 1 >= cnt) break;
          ea = s_splat[i + 2];
          ma = s_meta[i + 2];
          visit(eb, 1u, __builtin_amdgcn_readfirstlane(mb.x), (int)mb.y, mine >> (i + 1) & 1);
          if (i + 2 >= cnt) break;
        }
      }
    } else {
      uint64_t todo = hits;
      wave_sync();
      while (todo) {
        const int j = 63 - (int)__builtin_clzll(todo);
        todo &= ~(1ull << j);
        const Splat sp = s_splat[j];
        visit(sp, __builtin_amdgcn_readlane(reach, j), __builtin_amdgcn_readlane(eid, j),
              bot + j + 1, mine >> j & 1);
      }
    }
  }
}

// Tile coordinates of a tile index.
struct TilePos {
  int slot, tx, ty;
  __device__ __forceinline__ TilePos(const RasterDev& a, int64_t tile) {
    slot = (int)((uint32_t)tile / (uint32_t)a.tiles_per_slot);
    const uint32_t t = (uint32_t)tile - (uint32_t)slot * (uint32_t)a.tiles_per_slot;
    ty = (int)(t / (uint32_t)a.tiles_x);
    tx = (int)(t - (uint32_t)ty * (uint32_t)a.tiles_x);
  }
};

// Whole-list backward of NK blocks of a tile from its block b; the wave takes
// the sums of the entries in `mine`.
template <int TW, int TH, int NK, bool RECOMPUTE>
__device__ __forceinline__ void bwd_blocks(const RasterDev& a, int64_t tile, int b, uint64_t mine,
                                           Splat* s_splat, uint2* s_meta,
                                           const float* __restrict__ T_final,
                                           const int32_t* __restrict__ n_contrib,
                                           const float* __restrict__ d_image,
                                           float* __restrict__ d_rec) {
  constexpr int BX = TW / 8;
  static_assert(NK == 1 || NK == TW * TH / 64, "a block or the whole tile");
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  if (start >= end) return;
  const TilePos tp(a, tile);
  const int x0 = tp.tx * TW + (b % BX) * 8, y0 = tp.ty * TH + (b / BX) * 8;
  BwdPixels<BX, NK> p(a, x0, y0);
  float T_fin[NK];
  if constexpr (RECOMPUTE) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const float kx = (float)(8 * (k % BX)), ky = (float)(8 * (k / BX));
      const PixBox box{(float)x0 + kx + 0.5f, (float)x0 + kx + 7.5f, (float)y0 + ky + 0.5f,
                       (float)y0 + ky + 7.5f};
      const float fy = p.fy + ky;
      tile_forward<TW, TH, 1, false>(a.rec, a.ids, start, end, p.fx + kx, &fy, &p.inside[k],
                                     s_splat, &T_fin[k], nullptr, &p.last[k], box);
    }
  } else {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int64_t o = (int64_t)tp.slot * p.HW + p.offset(k);
      T_fin[k] = p.inside[k] ? T_final[o] : 1.0f;
      p.last[k] = p.inside[k] ? n_contrib[o] : 0;
    }
  }
  const int lmax = min(p.load_gradient(d_image + (int64_t)tp.slot * 3 * p.HW), (int)(end - start));
#pragma unroll
  for (int k = 0; k < NK; ++k) p.final_state(k, T_fin[k], a);
  reverse_pass<BX, NK>(a, start, 0, lmax, x0, y0, p, s_splat, d_rec, s_meta, mine);
  if (a.dup_grads) zero_dup_slots(a, start, lmax, (int)(end - start));
}

// Waves are added up to 32 a CU, eight a SIMD, as many as can be resident: with
// a limit of 16, 512x512 images (1 against 2 waves a block) took 136 against
// 125 us for 20K Gaussians, 353 / 307 for 100K and 828 / 781 for 400K, 400x300
// (2 / 4) 337 / 283 for 100K.
constexpr int kBwdShareLgMax = 3;
constexpr int64_t kBwdShareWavesPerCu = 32;

// Whole-list backward.  Without chunks a tile's list is one serial walk, and
// the call takes as long as its longest lists; in the atomic form every block
// of a tile therefore has its own wave (NK = 1; the NB waves of a tile are
// adjacent launches).  The deterministic form stores an entry's sums over the
// whole tile, so one wave takes the tile (NK = NB).
// Where that leaves the chip mostly idle, 1 << lg_share waves walk the same
// pixels, every wave all entries but each the sums of every (1 << lg_share)-th
// only: those, their reduction and the atomics are two thirds of a visit.
// 128x128 with 64 tiles (8 waves a block): 131 -> 76 us; 333x251 with 336
// tiles (4): 174 -> 130.
// Four blocks a wave are compiled for five waves a SIMD (at 97 VGPRs, one too
// many, the replaying form had four: 16 sparse images of 1920x1080 1352 -> 1249).
template <int TW, int TH, int NK, bool RECOMPUTE>
__global__ __launch_bounds__(kRasterWave)
__attribute__((amdgpu_waves_per_eu(NK == 4 ? 5 : 1))) void k_raster_bwd(RasterDev a, TileSched sch,
                                                            int lg_share,
                                                            const float* __restrict__ T_final,
                                                            const int32_t* __restrict__ n_contrib,
                                                            const float* __restrict__ d_image,
                                                            float* __restrict__ d_rec) {
  constexpr int NB = TW * TH / 64 / NK;
  __shared__ Splat s_splat[kFwdSlots];
  __shared__ uint2 s_meta[kFwdSlots];
  constexpr int kLgNB = NB == 1 ? 0 : (NB == 2 ? 1 : (NB == 4 ? 2 : 3));
  static_assert(1 << kLgNB == NB, "blocks of a tile");
  for_each_tile(sch, a.n_tiles, kLgNB + lg_share, [&](int64_t tile, int b) {
    // bits q, q + Q, q + 2 Q, ... of Q = 1 << lg_share waves
    const int Q = 1 << lg_share;
    const uint64_t every = Q == 1 ? ~0ull : ~0ull / ((1ull << Q) - 1);
    bwd_blocks<TW, TH, NK, RECOMPUTE>(a, tile, b >> lg_share, every << (b & (Q - 1)), s_splat,
                                      s_meta, T_final, n_contrib, d_image, d_rec);
  });
}

// Chunked backward: one wave per (tile, chunk) item.  Chunk c covers list
// positions (c*chunk, min((c+1)*chunk, len)]; the state after its last
// position is the forward's final state for pixels whose last blended entry
// lies at or before it, else the checkpoint (T_c, U_c) the forward stored
// there (dI . acc = T_c dI . U_c).
template <int TW, int TH>
__global__ __launch_bounds__(kRasterWave)
__attribute__((amdgpu_waves_per_eu(kBwdWavesPerEU<TW, TH>)))
void k_raster_bwd_chunked(
    RasterDev a, ChunkDev ch, const float* __restrict__ T_final,
    const int32_t* __restrict__ n_contrib, const float* __restrict__ d_image,
    float* __restrict__ d_rec) {
  constexpr int BX = TW / 8, NK = TW * TH / 64;
  __shared__ Splat s_splat[NK == 1 ? kFwdSlots : kRasterWave];
  __shared__ uint2 s_meta[NK == 1 ? kFwdSlots : 1];
  const uint32_t item = blockIdx.x;
  if (item >= ch.offset[a.n_tiles]) return;
  const int64_t tile = ch.items[item];
  const uint32_t c0 = ch.offset[tile];
  const int c = (int)(item - c0);
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  const int len = (int)(end - start);
  const int lo = c * ch.chunk, hi_pos = min(lo + ch.chunk, len);
  const TilePos tp(a, tile);
  const int x0 = tp.tx * TW, y0 = tp.ty * TH;
  BwdPixels<BX, NK> p(a, x0, y0);
#pragma unroll
  for (int k = 0; k < NK; ++k)
    p.last[k] = p.inside[k] ? n_contrib[(int64_t)tp.slot * p.HW + p.offset(k)] : 0;
  const int hi = min(p.load_gradient(d_image + (int64_t)tp.slot * 3 * p.HW), hi_pos);
  if (hi <= lo) {
    if (a.dup_grads) zero_dup_slots(a, start, lo, hi_pos);
    return;
  }
  const int lane = threadIdx.x;
  const float4* ck = ch.ck + ((int64_t)c0 + c) * (TW * TH) + (lane >> 3) * TW + (lane & 7);
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    if (!p.inside[k] || p.last[k] <= hi_pos) {
      // nothing blended after this chunk: final state
      p.final_state(k, p.inside[k] ? T_final[(int64_t)tp.slot * p.HW + p.offset(k)] : 1.0f, a);
    } else {
      const float4 s = ck[8 * (k / BX) * TW + 8 * (k % BX)];   // (T_c, U_c)
      p.T[k] = s.x;
      p.dIacc[k] = s.x * (p.dI[k][0] * s.y + p.dI[k][1] * s.z + p.dI[k][2] * s.w);
    }
  }
  reverse_pass<BX, NK>(a, start, lo, hi, x0, y0, p, s_splat, d_rec, s_meta);
  if (a.dup_grads) zero_dup_slots(a, start, hi, hi_pos);
}

// ---------------------------------------------------------------- quadrant groups

// Reduce-scatter of the 9 gradient components over each 16-lane row of the
// wave (the rows work on different entries): row_ror:8 pairs l and l ^ 8,
// row_half_mirror l and 7 - l, and two quad_perm steps l ^ 2 and l ^ 1;
// each step keeps, per lane, about half of the components summed over the
// lane pair.  Afterwards 9 lanes of every row hold the row total of one
// component each (row_slot9 names which).
template <int CTRL>
__device__ __forceinline__ float keep_add(bool hi, float lo_v, float hi_v) {
  const float mine = hi ? hi_v : lo_v, other = hi ? lo_v : hi_v;
  return mine + dpp_f<CTRL>(other);
}

__device__ __forceinline__ float reduce_scatter9_row(const float (&v)[9]) {
  const int l = threadIdx.x & 15;
  const bool b3 = (l >> 3) & 1, b2 = (l >> 2) & 1, b1 = (l >> 1) & 1, b0 = l & 1;
  // 9 -> 5: bit 3 clear keeps 0..4, set keeps 5..8
  const float w0 = keep_add<kDppRowRor8>(b3, v[0], v[5]);
  const float w1 = keep_add<kDppRowRor8>(b3, v[1], v[6]);
  const float w2 = keep_add<kDppRowRor8>(b3, v[2], v[7]);
  const float w3 = keep_add<kDppRowRor8>(b3, v[3], v[8]);
  const float w4 = keep_add<kDppRowRor8>(b3, v[4], 0.0f);
  // 5 -> 3: bit 2 clear keeps w0..w2, set keeps w3, w4
  const float u0 = keep_add<kDppRowHalfMirror>(b2, w0, w3);
  const float u1 = keep_add<kDppRowHalfMirror>(b2, w1, w4);
  const float u2 = keep_add<kDppRowHalfMirror>(b2, w2, 0.0f);
  // 3 -> 2: bit 1 clear keeps u0, u1, set keeps u2
  const float t0 = keep_add<kDppQuadSwap2>(b1, u0, u2);
  const float t1 = keep_add<kDppQuadSwap2>(b1, u1, 0.0f);
  // 2 -> 1: bit 0 clear keeps t0, set keeps t1
  return keep_add<kDppQuadSwap1>(b0, t0, t1);
}

// Component (0-8) whose row total reduce_scatter9_row leaves in row lane l,
// or -1.
__device__ __forceinline__ int row_slot9(int l) {
  const int b3 = (l >> 3) & 1, b2 = (l >> 2) & 1, b1 = (l >> 1) & 1, b0 = l & 1;
  int L1[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) L1[k] = b3 ? (k < 4 ? 5 + k : -1) : k;
  const int L2[3] = {b2 ? L1[3] : L1[0], b2 ? L1[4] : L1[1], b2 ? -1 : L1[2]};
  const int L3[2] = {b1 ? L2[2] : L2[0], b1 ? -1 : L2[1]};
  return b0 ? L3[1] : L3[0];
}

// ---- pairs of an entry and a pixel (8x8 tiles)
//
// A lane owns pixel p = lane: quadrant p / 16 (2 x 2 of them), in it column
// p % 4 and row p % 16 / 4.

// The pixels (bit p) of the 8x8 block with pixel-centre origin (x0, y0) that
// may pass the alpha test: of every row the interval in which A dx^2 + B dx dy
// + C dy^2 >= thr, widened by splat_may_hit's margin in the exponent, which
// covers the rounding of both sides, and by 1e-3 pixels.
__device__ __forceinline__ void splat_pixels(const Splat& s, float x0, float y0, uint32_t& lo,
                                             uint32_t& hi) {
  lo = hi = 0u;
  if (!(s.A < 0.0f)) {
    lo = hi = ~0u;
    return;
  }
  const float dx0 = x0 - s.mx, dy0 = y0 - s.my;
  const float X = fmaxf(fabsf(dx0), fabsf(dx0 + 7.0f)), Y = fmaxf(fabsf(dy0), fabsf(dy0 + 7.0f));
  const float M = -s.A * X * X + fabsf(s.B) * X * Y - s.C * Y * Y;
  const float thr = s.thr - (0.02f + 4e-6f * M);
  const float K1 = s.B * s.B - 4.0f * s.A * s.C, K2 = 4.0f * s.A * thr;
  const float iA = -0.5f * __builtin_amdgcn_rcpf(s.A);          // 1 / (-2A) > 0
  const float cB = s.B * iA;                                    // interval centre per dy
#pragma unroll
  for (int y = 0; y < 8; ++y) {
    const float dy = dy0 + (float)y;
    const float t = fmaf(K1 * dy, dy, K2);                      // discriminant
    const float h = __builtin_amdgcn_sqrtf(t) * iA + 1e-3f;     // NaN below zero
    const float c = cB * dy - dx0;
    const int i0 = (int)ceilf(__builtin_amdgcn_fmed3f(c - h, 0.0f, 8.0f));
    const int i1 = (int)floorf(__builtin_amdgcn_fmed3f(c + h, -1.0f, 7.0f));
    const uint32_t m = t >= 0.0f && i1 >= i0 ? (2u << i1) - (1u << i0) : 0u;
    const uint32_t w = ((m | (m << 12)) & 0x000f000fu) << (4 * (y & 3));
    if (y < 4) lo |= w;
    else hi |= w;
  }
}

// Transposes the 64x64 bit matrix whose row l is lane l's (hi, lo).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t transpose32_step(uint32_t x, uint32_t other, uint32_t keep,
                                                     int rot) {
  // keep: the bits that stay; the partner's come from `rot` bits to the right
  const uint32_t t = __builtin_amdgcn_alignbit(other, other, (uint32_t)rot);
  return (x & keep) | (t & ~keep);
}
__device__ __forceinline__ void transpose64(uint32_t& lo, uint32_t& hi) {
  const int l = threadIdx.x & 63;
  const auto s32 = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
  uint32_t w[2] = {s32[0], s32[1]};
  const bool b4 = l & 16, b3 = l & 8, b2 = l & 4, b1 = l & 2, b0 = l & 1;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t x = w[i];
    const auto s16 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = transpose32_step(x, b4 ? s16[0] : s16[1], b4 ? 0xffff0000u : 0x0000ffffu, 16);
    x = transpose32_step(x, dpp_u<kDppRowRor8>(x), b3 ? 0xff00ff00u : 0x00ff00ffu, b3 ? 8 : 24);
    x = transpose32_step(x, dpp_u<kDppQuadReverse>(dpp_u<kDppRowHalfMirror>(x)),
                         b2 ? 0xf0f0f0f0u : 0x0f0f0f0fu, b2 ? 4 : 28);
    x = transpose32_step(x, dpp_u<kDppQuadSwap2>(x), b1 ? 0xccccccccu : 0x33333333u, b1 ? 2 : 30);
    x = transpose32_step(x, dpp_u<kDppQuadSwap1>(x), b0 ? 0xaaaaaaaau : 0x55555555u, b0 ? 1 : 31);
    w[i] = x;
  }
  lo = w[0];
  hi = w[1];
}

constexpr int kPairCap = 512;        // pairs of a batch that are taken pair by pair

struct PairLds {
  uint4 pix[kRasterWave];            // entries of the pixel (64 bits), its first pair, last position
  float4 dI[kRasterWave];            // image gradient; place in the tile, x | y << 8
  uint16_t pair[kPairCap];           // entry | pixel << 6
  float2 gw[kPairCap];               // alpha and dI . colour of each pair, then G = dL/d(exponent)
                                     // and blend weight; then the entries' sums
};

// Chunked backward on quadrant lane groups: row q of the wave (lanes 16q ..
// 16q+15) owns the (TW/2) x (TH/2) quadrant (q mod 2, q / 2) of the tile,
// PXQ pixels of one column per lane (column r mod QW, rows r / QW + k RS),
// and walks in reverse list order only the entries of the chunk that may
// reach its quadrant (the staging cull against each quadrant's box); the
// four rows work on different entries at once, and an entry's 9 components
// are reduced over its row and added atomically.  Splats that reach part of
// a tile then cost their fixed share (the reduction) on 16 lanes instead of
// 64.  Per pixel the arithmetic and the skip and stop decisions are those of
// reverse_pass.  Atomic gradient sums only.
// That walk is for batches of more than kPairCap pairs of an entry and a pixel
// it may reach.  Dense views of an 8x8 tile blend an entry into one to four of
// its 64 pixels, and the quadrants ran 3 to 10% of their lanes; batches of few
// pairs are taken pair by pair: the pixels' bits of all entries at once (a
// lane per entry), transposed to the entries' bits of all pixels, the pairs
// listed by pixel, evaluated 64 at a time, walked by a lane per pixel for the
// transmittance and the colour behind, and each entry's sums taken by its own
// lane.  Every term is the one that the walk by quadrants forms, to the bit
// (products and sums by scans over 64 pairs instead of the walk per pixel: 519M
// instructions and 1666 us, but gradients 3.5e-6 off); only an entry's sum
// over its pixels has another order.  13.3M Gaussians at 3840x2160: 1823M ->
// 602M vector instructions, 2529 -> 1672 us; now bound by the 32M memory-side
// atomic requests of the random gradient rows (973 us without them; fewer
// registers and earlier loads measured the same).  10,240 bytes of LDS: 16
// waves a CU, the four a SIMD that the registers allow.  The cap, measured with
// 1280 bytes more: 512 pairs (14 waves a CU) 1662 us, 768 (11) 1764; 320 (16)
// 2193 in views with larger footprints, whose batches then fall to the walk by
// quadrants.
template <int TW, int TH>
__global__ __launch_bounds__(kRasterWave)
__attribute__((amdgpu_waves_per_eu(4))) void k_raster_bwd_chunked_q(
    RasterDev a, ChunkDev ch, const float* __restrict__ T_final,
    const int32_t* __restrict__ n_contrib, const float* __restrict__ d_image,
    float* __restrict__ d_rec) {
  constexpr int QW = TW / 2, QH = TH / 2, PXQ = QW * QH / 16, RS = 16 / QW;
  static_assert(QW * QH % 16 == 0 && 16 % QW == 0, "quadrant shape");
  __shared__ Splat s_splat[kRasterWave];       // pad1: the entry's pair
  static_assert(TW == 8 && TH == 8, "pairs");
  __shared__ PairLds s_p;
  const uint32_t item = blockIdx.x;
  if (item >= ch.offset[a.n_tiles]) return;
  const int64_t tile = ch.items[item];
  const int c = (int)(item - ch.offset[tile]);
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  const int len = (int)(end - start);
  const int lo = c * ch.chunk, hi_pos = min(lo + ch.chunk, len);
  const int lane = threadIdx.x, q = lane >> 4, r = lane & 15;
  const int slot = (int)(tile / a.tiles_per_slot);
  const int tt = (int)(tile - (int64_t)slot * a.tiles_per_slot);
  const int ty = tt / a.tiles_x, tx = tt - ty * a.tiles_x;
  const int lx = (q & 1) * QW + r % QW, ly0 = (q >> 1) * QH + r / QW;   // in the tile
  const int px = tx * TW + lx;
  const float fx = (float)px + 0.5f;
  const int64_t HW = (int64_t)a.H * a.W;
  const float* dimg = d_image + (int64_t)slot * 3 * HW;
  float fy[PXQ], T[PXQ], dI[PXQ][3], dIacc[PXQ];
  int last[PXQ];
  bool inside[PXQ];
  int lmax = 0;
#pragma unroll
  for (int k = 0; k < PXQ; ++k) {
    const int py = ty * TH + ly0 + k * RS;
    fy[k] = (float)py + 0.5f;
    inside[k] = (px < a.W) && (py < a.H);
    const int64_t o = (int64_t)py * a.W + px;
    last[k] = inside[k] ? n_contrib[(int64_t)slot * HW + o] : 0;
    dI[k][0] = inside[k] ? dimg[o] : 0.0f;
    dI[k][1] = inside[k] ? dimg[HW + o] : 0.0f;
    dI[k][2] = inside[k] ? dimg[2 * HW + o] : 0.0f;
    // a pixel with a zero image gradient (a masked one) adds exactly zero
    if (dI[k][0] == 0.0f && dI[k][1] == 0.0f && dI[k][2] == 0.0f) last[k] = 0;
    lmax = max(lmax, last[k]);
  }
  const int hi = min(wave_max_int(lmax), hi_pos);
  if (hi <= lo) return;
  const float4* ck = ch.ck + ((int64_t)ch.offset[tile] + c) * (TW * TH);
#pragma unroll
  for (int k = 0; k < PXQ; ++k) {
    if (!inside[k] || last[k] <= hi_pos) {
      // nothing blended after this chunk: final state, I - C_final = bg T_final
      const int64_t o = (int64_t)(ty * TH + ly0 + k * RS) * a.W + px;
      T[k] = inside[k] ? T_final[(int64_t)slot * HW + o] : 1.0f;
      dIacc[k] = T[k] * (dI[k][0] * a.bg0 + dI[k][1] * a.bg1 + dI[k][2] * a.bg2);
    } else {
      const float4 sck = ck[(ly0 + k * RS) * TW + lx];   // (T_c, U_c)
      T[k] = sck.x;
      dIacc[k] = sck.x * (dI[k][0] * sck.y + dI[k][1] * sck.z + dI[k][2] * sck.w);
    }
  }
  const int rslot = row_slot9(r);
  // d mean2d (x2) carry -ln2, d Q11 and d Q22 -1/2, d Q12 -1 (log2-scaled
  // falloff); opacity and colour 1
  const float sc[9] = {-kLn2, -kLn2, -0.5f, -1.0f, -0.5f, 1.0f, 1.0f, 1.0f, 1.0f};
  const float rscale = rslot >= 0 ? sc[rslot] : 0.0f;
  const float qx0 = (float)(tx * TW) + 0.5f, qy0 = (float)(ty * TH) + 0.5f;
  s_p.dI[lane] = make_float4(dI[0][0], dI[0][1], dI[0][2], __uint_as_float(lx | ly0 << 8));
  // centre of the pixel with that record (exact: the tile's corner plus 0 .. 7)
  auto centre_x = [&](const float4& di) { return qx0 + (float)(__float_as_uint(di.w) & 0xff); };
  auto centre_y = [&](const float4& di) { return qy0 + (float)(__float_as_uint(di.w) >> 8); };
  for (int top = hi; top > lo; top -= kRasterWave) {
    const int bot = max(lo, top - kRasterWave);
    const int n = top - bot;
    wave_sync();
    // the entry's pixels, among those that blend in this batch
    const uint64_t active = __ballot(last[0] > bot);
    uint32_t plo = 0, phi = 0;
    Splat sp{};
    if (lane < n) {
      const uint32_t id = a.ids[start + bot + lane];
      sp = load_splat(a.rec, id);
      sp.pad1 = __uint_as_float(id);
      s_splat[lane] = sp;
      splat_pixels(sp, qx0, qy0, plo, phi);
      plo &= (uint32_t)active;
      phi &= (uint32_t)(active >> 32);
    }
    uint32_t elo = plo, ehi = phi;           // the pixel's entries
    transpose64(elo, ehi);
    const int cnt = __builtin_popcount(elo) + __builtin_popcount(ehi);
    int upto = cnt;                          // inclusive sum over the pixels
#pragma unroll
    for (int d = 1; d < kRasterWave; d <<= 1) {
      const int o = __shfl_up(upto, d, kRasterWave);
      if (lane >= d) upto += o;
    }
    const int total = __builtin_amdgcn_readlane(upto, kRasterWave - 1);
    if (total == 0) continue;
    if (total <= kPairCap) {
      const int lrel = min(max(last[0] - bot, 0), kRasterWave), first = upto - cnt;
      s_p.pix[lane] = make_uint4(elo, ehi, (uint32_t)first, (uint32_t)lrel);
      wave_sync();
      // the pairs by pixel, last entry first
      const uint64_t above = lane == 63 ? 0ull : ~0ull << (lane + 1);
      const uint32_t alo = (uint32_t)above, ahi = (uint32_t)(above >> 32);
      auto place = [&](const uint4& px_) {
        return (int)px_.z + __builtin_popcount(px_.x & alo) + __builtin_popcount(px_.y & ahi);
      };
      for (uint64_t m = (uint64_t)phi << 32 | plo; m; m &= m - 1) {
        const int p = (int)__builtin_ctzll(m);
        s_p.pair[place(s_p.pix[p])] = (uint16_t)(lane | p << 6);
      }
      wave_sync();
      // a lane per pair: what of it needs no transmittance
      for (int i = lane; i < total; i += kRasterWave) {
        const uint32_t code = s_p.pair[i];
        const int e = (int)(code & 63), p = (int)(code >> 6);
        const Splat& se = s_splat[e];
        const float4 di = s_p.dI[p];
        const float p2 = splat_p2(se, __fsub_rn(centre_x(di), se.mx), __fsub_rn(centre_y(di), se.my));
        const bool pass = e < (int)s_p.pix[p].w && splat_pass(se, p2);
        const float alpha = fminf(kAlphaMax, se.o * splat_gauss(p2));
        const float dIc = fmaf(di.z, se.b, fmaf(di.y, se.g, di.x * se.r));
        s_p.gw[i] = pass ? make_float2(alpha, dIc) : make_float2(0.0f, 0.0f);
      }
      wave_sync();
      // a lane per pixel: its pairs one after the other, last entry first, as
      // the walk by quadrants has them (a pair that does not blend, alpha 0,
      // leaves T and dIacc as they are)
      constexpr int kRead = 4;
      for (int i = 0; __any(i < cnt); i += kRead) {
        float2 v[kRead];
#pragma unroll
        for (int k = 0; k < kRead; ++k) v[k] = s_p.gw[min(first + i + k, kPairCap - 1)];
#pragma unroll
        for (int k = 0; k < kRead; ++k) {
          const bool mine = i + k < cnt;
          const float alpha = mine ? v[k].x : 0.0f, dIc = mine ? v[k].y : 0.0f;
          const float inv = __builtin_amdgcn_rcpf(1.0f - alpha);
          const float Tb = T[0] * inv;                 // transmittance in front of it
          const float w = alpha * Tb;
          const float dLda = fmaf(Tb, dIc, -inv * dIacc[0]);
          dIacc[0] = fmaf(w, dIc, dIacc[0]);
          T[0] = Tb;
          // (the derivative through a clamped alpha is zero)
          if (alpha > 0.0f)
            s_p.gw[first + i + k] = make_float2(alpha < kAlphaMax ? dLda * alpha : 0.0f, w);
        }
      }
      wave_sync();
      // sums over an entry's pixels of what the walk by quadrants sums
      float smx = 0.f, smy = 0.f, sG = 0.f, sGxx = 0.f, sGxy = 0.f, sGyy = 0.f;
      float sr = 0.f, sg = 0.f, sb = 0.f, sw = 0.f;
      for (uint64_t m = (uint64_t)phi << 32 | plo; m; m &= m - 1) {
        const int p = (int)__builtin_ctzll(m);
        const float2 gw = s_p.gw[place(s_p.pix[p])];
        if (gw.y == 0.0f) continue;      // not blended: nothing of the pixel, were it infinite
        const float4 di = s_p.dI[p];
        const float dx = __fsub_rn(centre_x(di), sp.mx), dy = __fsub_rn(centre_y(di), sp.my);
        const float Gdy = gw.x * dy;
        smx += fmaf(2.0f * sp.A * dx, gw.x, sp.B * Gdy);
        smy += fmaf(2.0f * sp.C, Gdy, sp.B * dx * gw.x);
        sG += gw.x;
        sGxx = fmaf(dx * dx, gw.x, sGxx);
        sGxy = fmaf(dx, Gdy, sGxy);
        sGyy = fmaf(Gdy, dy, sGyy);
        sr = fmaf(di.x, gw.y, sr);
        sg = fmaf(di.y, gw.y, sg);
        sb = fmaf(di.z, gw.y, sb);
        sw += gw.y;
      }
      wave_sync();
      // through LDS, so that the 9 atomics of an entry are side by side; an
      // entry that blended nowhere adds nothing
      float* out = reinterpret_cast<float*>(s_p.gw);
      const float comp[9] = {-kLn2 * smx, -kLn2 * smy, -0.5f * sGxx, -sGxy, -0.5f * sGyy,
                             sG * __builtin_amdgcn_rcpf(sp.o), sr, sg, sb};
#pragma unroll
      for (int k = 0; k < 9; ++k) out[lane * 9 + k] = comp[k];
      const uint64_t adds = __ballot(sw != 0.0f);
      wave_sync();
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int f = k * kRasterWave + lane, e = f / 9;
        if (adds >> e & 1)
          atomicAdd(d_rec + (int64_t)__float_as_uint(s_splat[e].pad1) * GS_DREC_STRIDE + (f - 9 * e),
                    out[f]);
      }
      continue;
    }
    // many pairs: quadrant by quadrant
    wave_sync();
    uint32_t qm = 0;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if ((g < 2 ? plo : phi) >> (16 * (g & 1)) & 0xffffu) qm |= 1u << g;
    const uint64_t m0 = __ballot(qm & 1u), m1 = __ballot(qm & 2u), m2 = __ballot(qm & 4u),
                   m3 = __ballot(qm & 8u);
    uint64_t todo = q == 0 ? m0 : (q == 1 ? m1 : (q == 2 ? m2 : m3));
    while (__any(todo != 0)) {
      const bool act = todo != 0;
      const int j = act ? 63 - (int)__builtin_clzll(todo) : 0;     // last first
      if (act) todo &= ~(1ull << j);
      const Splat& se = s_splat[j];
      const Splat sp = se;
      const int pos = bot + j + 1;
      const float dx = __fsub_rn(fx, sp.mx);
      float p2[PXQ];
      splat_p2_column<PXQ>(sp, dx, fy, p2);
      bool pass[PXQ], any = false;
#pragma unroll
      for (int k = 0; k < PXQ; ++k) {
        pass[k] = act && (pos <= last[k]) && splat_pass(sp, p2[k]);
        any = any || pass[k];
      }
      if (!__any(any)) continue;
      // per-lane sums over the lane's pixels (dx is shared by its column)
      float sG = 0.f, sGdy = 0.f, sGdy2 = 0.f, so = 0.f, sr = 0.f, sg = 0.f, sb = 0.f;
#pragma unroll
      for (int k = 0; k < PXQ; ++k) {
        if (!pass[k]) continue;
        const float gss = splat_gauss(p2[k]);
        const float aa = sp.o * gss;
        const float alpha = fminf(kAlphaMax, aa);
        const float inv = __builtin_amdgcn_rcpf(1.0f - alpha);
        const float Tb = T[k] * inv;                 // transmittance in front of it
        const float w = alpha * Tb;
        const float dIc = fmaf(dI[k][2], sp.b, fmaf(dI[k][1], sp.g, dI[k][0] * sp.r));
        const float dLda = fmaf(Tb, dIc, -inv * dIacc[k]);
        dIacc[k] = fmaf(w, dIc, dIacc[k]);
        T[k] = Tb;
        sr = fmaf(dI[k][0], w, sr);
        sg = fmaf(dI[k][1], w, sg);
        sb = fmaf(dI[k][2], w, sb);
        if (aa < kAlphaMax) {
          const float G = dLda * alpha;
          const float dy = __fsub_rn(fy[k], sp.my);
          const float Gdy = G * dy;
          so = fmaf(dLda, gss, so);
          sG += G;
          sGdy += Gdy;
          sGdy2 = fmaf(Gdy, dy, sGdy2);
        }
      }
      const float bdx = sp.B * dx;
      const float comp[9] = {fmaf(2.0f * sp.A * dx, sG, sp.B * sGdy),   // d mx / -ln2
                             fmaf(2.0f * sp.C, sGdy, bdx * sG),         // d my / -ln2
                             dx * dx * sG,                              // d Q11 / -1/2
                             dx * sGdy,                                 // d Q12 / -1
                             sGdy2,                                     // d Q22 / -1/2
                             so, sr, sg, sb};
      const float tot = reduce_scatter9_row(comp);
      // rows whose entry no pixel of theirs passed add nothing
      const uint64_t rows = __ballot(any);
      if (rslot >= 0 && ((rows >> (16 * q)) & 0xffffull) != 0)
        atomicAdd(d_rec + (int64_t)__float_as_uint(sp.pad1) * GS_DREC_STRIDE + rslot, rscale * tot);
    }
  }
}

// ---------------------------------------------------------------- split forward

// Pixel geometry of one tile for the calling lane.
template <int TW, int TH>
struct LanePixels {
  static constexpr int PX = TileGeom<TW, TH>::PX, RSTEP = TileGeom<TW, TH>::RSTEP;
  int slot, px, py0, tx, ty;
  float fx, fy[PX];
  bool inside[PX];
  __device__ __forceinline__ LanePixels(const RasterDev& a, int64_t tile) {
    slot = (int)(tile / a.tiles_per_slot);
    const int t = (int)(tile - (int64_t)slot * a.tiles_per_slot);
    ty = t / a.tiles_x;
    tx = t - ty * a.tiles_x;
    const int lane = threadIdx.x;
    px = tx * TW + (lane % TW);
    py0 = ty * TH + lane / TW;
    fx = (float)px + 0.5f;
#pragma unroll
    for (int k = 0; k < PX; ++k) {
      const int py = py0 + k * RSTEP;
      fy[k] = (float)py + 0.5f;
      inside[k] = (px < a.W) && (py < a.H);
    }
  }
  __device__ __forceinline__ int64_t offset(const RasterDev& a, int k) const {
    return (int64_t)(py0 + k * RSTEP) * a.W + px;
  }
};

// Forward of long tile lists in parallel (stored mode with chunk items).
// Part 1: one wave per chunk item (tile, c) composites the chunk's entries
// for the tile's pixels from a local transmittance of 1, ignoring the stop
// rule: P = prod(1 - alpha) and L = sum rgb alpha T_local over the chunk
// (the arithmetic of the sequential forward's chunk composites), and the
// chunk-local position of the last blend.  The (P, L) of chunk c >= 1 go to
// checkpoint slot c - 1, those of chunk 0 to slot nc - 1 (nc = the tile's
// chunks; the backward never reads that slot, the last chunk starting from
// the final state).
template <int TW, int TH>
__global__ __launch_bounds__(kRasterWave) void k_raster_fwd_part(RasterDev a, ChunkDev ch,
                                                                uint16_t* __restrict__ clast) {
  constexpr int PX = TileGeom<TW, TH>::PX;
  __shared__ Splat s_splat[kFwdSlots];
  const uint32_t item = blockIdx.x;
  if (item >= ch.offset[a.n_tiles]) return;
  const int64_t tile = ch.items[item];
  const uint32_t c0 = ch.offset[tile];
  const int c = (int)(item - c0), nc = (int)(ch.offset[tile + 1] - c0);
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  const int len = (int)(end - start);
  const int lo = c * ch.chunk, hi_pos = min(lo + ch.chunk, len);
  const LanePixels<TW, TH> L(a, tile);
  const PixBox box{(float)(L.tx * TW) + 0.5f, (float)(L.tx * TW + TW - 1) + 0.5f,
                   (float)(L.ty * TH) + 0.5f, (float)(L.ty * TH + TH - 1) + 0.5f};
  const int lane = threadIdx.x;
  uint64_t live[PX];
  float Tl[PX], Lc[PX][3];
  int lastl[PX];
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    live[k] = __ballot(L.inside[k]);
    Tl[k] = 1.0f;
    Lc[k][0] = Lc[k][1] = Lc[k][2] = 0.0f;
    lastl[k] = 0;
  }
  for (int b0 = lo; b0 < hi_pos; b0 += kRasterWave) {
    const int n = min(kRasterWave, hi_pos - b0);
    Splat s{};
    bool hit = false;
    if (lane < n) {
      s = load_splat(a.rec, a.ids[start + b0 + lane]);
      hit = splat_may_hit(s, box.x0, box.x1, box.y0, box.y1);
    }
    const int cnt = fwd_pack(s, hit, b0 - lo + lane + 1, s_splat);
    int lastc[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) lastc[k] = -1;
    fwd_for_each(s_splat, cnt, [&](const FwdEntry& e, int i) {
      float p2[PX];
      uint64_t pass[PX];
      if (!fwd_test<PX>(e, L.fx, L.fy, live, p2, pass)) return;
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        if (lane_in(pass[k])) {
          const float alpha = fminf(kAlphaMax, e.col.x * splat_gauss(p2[k]));
          const float wl = alpha * Tl[k];
          Lc[k][0] = fmaf(e.col.y, wl, Lc[k][0]);
          Lc[k][1] = fmaf(e.col.z, wl, Lc[k][1]);
          Lc[k][2] = fmaf(e.col.w, wl, Lc[k][2]);
          Tl[k] = Tl[k] * (1.0f - alpha);
          lastc[k] = i;
        }
      }
    });
#pragma unroll
    for (int k = 0; k < PX; ++k)
      if (lastc[k] >= 0) lastl[k] = fwd_pos(s_splat, lastc[k]);
  }
  float4* ck = ch.ck + ((int64_t)c0 + (c >= 1 ? c - 1 : nc - 1)) * (TW * TH);
  uint16_t* cl = clast + ((int64_t)c0 + c) * (TW * TH);
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    ck[lane + k * kRasterWave] = make_float4(Tl[k], Lc[k][0], Lc[k][1], Lc[k][2]);
    cl[lane + k * kRasterWave] = (uint16_t)lastl[k];
  }
}

// Part 2: one wave per tile joins its chunks in list order.  A pixel whose
// transmittance stays at or above the cut-off through chunk c (T P_c >=
// T_min: the partial products only fall, so no entry of the chunk stops
// it) takes C += T L_c, T = T P_c; where T P_c < T_min the chunk is
// composited again entry by entry from T with the stop rule (all lanes stage
// it and test one such pixel after another, a lane per entry; the pixels
// concerned composite what passed: with the whole wave visiting every entry,
// as the first part does, these few pixels were most of the join, 776 -> 488
// us at 4K), and the pixel ends there.  Then the
// image, T_final and n_contrib are written, and the checkpoints become the
// (T_c, U_c) the backward reads, by the recursion of the sequential forward
// over the chunks' (P, L) (identity after a pixel's stop, the partial
// composite up to it in the stopping chunk).  Both walks over the chunks
// keep D chunks' loads in flight: a long list's join is a chain of
// dependent loads otherwise (lists of 450 chunks at 4K: D 4 -> 8, 945 -> 776
// us).
// MANY: with few large splats most pixels of a tile stop in the same chunk, and
// all lanes visit its entries after all (join_many).
template <int TW, int TH, bool MANY>
__global__ __launch_bounds__(kRasterWave) void k_raster_fwd_join(
    RasterDev a, TileSched sch, ChunkDev ch, const uint16_t* __restrict__ clast,
    float* __restrict__ image, float* __restrict__ T_final, int32_t* __restrict__ n_contrib) {
  constexpr int PX = TileGeom<TW, TH>::PX, NP = TW * TH;
  constexpr int D = PX >= 8 ? 1 : 8 / PX;
  __shared__ Splat s_splat[kRasterWave];
  for_each_tile(sch, a.n_tiles, 0, [&](int64_t tile, int) {
    const LanePixels<TW, TH> L(a, tile);
    const int lane = threadIdx.x;
    const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
    const int len = (int)(end - start);
    const uint32_t c0 = ch.offset[tile];
    const int nc = (int)(ch.offset[tile + 1] - c0);
    float4* ck = ch.ck + (int64_t)c0 * NP;
    const uint16_t* cl = clast + (int64_t)c0 * NP;
    float T[PX], C[PX][3], Ps[PX], Ls[PX][3];
    int last[PX], cs[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) {
      T[k] = 1.0f;
      C[k][0] = C[k][1] = C[k][2] = 0.0f;
      last[k] = 0;
      cs[k] = nc;                       // chunk of the stop (nc: none)
      Ps[k] = 1.0f;
      Ls[k][0] = Ls[k][1] = Ls[k][2] = 0.0f;
    }
    // chunk c's (P, L) sit in slot c - 1, chunk 0's in slot nc - 1
    auto load_chunk = [&](int c, float4 (&pl)[PX], int (&ll)[PX]) {
      const int sl = c >= 1 ? c - 1 : nc - 1;
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        pl[k] = ck[(int64_t)sl * NP + lane + k * kRasterWave];
        ll[k] = cl[(int64_t)c * NP + lane + k * kRasterWave];
      }
    };
    auto join_chunk = [&](int c, const float4 (&pl)[PX], const int (&ll)[PX]) {
      bool fix[PX], any_fix = false;
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        fix[k] = false;
        if (cs[k] < nc || !L.inside[k]) continue;
        const float Tn = T[k] * pl[k].x;
        if (Tn < kTMin) {
          fix[k] = true;
          any_fix = true;
          continue;
        }
        C[k][0] = fmaf(T[k], pl[k].y, C[k][0]);
        C[k][1] = fmaf(T[k], pl[k].z, C[k][1]);
        C[k][2] = fmaf(T[k], pl[k].w, C[k][2]);
        T[k] = Tn;
        if (ll[k]) last[k] = c * ch.chunk + ll[k];
      }
      if (!__any(any_fix)) return;
      // composite chunk c again, entry by entry with the stop rule, for the
      // pixels whose transmittance reaches the cut-off inside it.  Those are
      // few: each is tested by all lanes at once, a lane per entry, and its
      // own lane then composites the entries that passed.
      float Tl[PX], Lc[PX][3];
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        Tl[k] = 1.0f;
        Lc[k][0] = Lc[k][1] = Lc[k][2] = 0.0f;
      }
      const int lo = c * ch.chunk, hi_pos = min(lo + ch.chunk, len);
      for (int b0 = lo; b0 < hi_pos; b0 += kRasterWave) {
        Splat s{};
        s.thr = INFINITY;                  // past the chunk's end: no pass
        wave_sync();
        if (b0 + lane < hi_pos) {
          s = load_splat(a.rec, a.ids[start + b0 + lane]);
          s_splat[lane] = s;
        }
        wave_sync();
        if constexpr (MANY) {
          // a pixel that is done has a NaN row coordinate: it passes no test
          const float x0 = (float)(L.tx * TW) + 0.5f, y0 = (float)(L.ty * TH) + 0.5f;
          float fyk[PX];
#pragma unroll
          for (int k = 0; k < PX; ++k) fyk[k] = fix[k] && cs[k] == nc ? L.fy[k] : __builtin_nanf("");
          uint64_t todo = __ballot(b0 + lane < hi_pos &&
                                   splat_may_hit(s, x0, x0 + (float)(TW - 1), y0, y0 + (float)(TH - 1)));
          while (todo) {
            const int j = (int)__builtin_ctzll(todo);
            todo &= todo - 1;
            const Splat sp = s_splat[j];
            float p2[PX];
            splat_p2_column<PX>(sp, __fsub_rn(L.fx, sp.mx), fyk, p2);
            bool pass[PX], any = false;
#pragma unroll
            for (int k = 0; k < PX; ++k) {
              pass[k] = splat_pass(sp, p2[k]);
              any = any || pass[k];
            }
            if (!__any(any)) continue;
#pragma unroll
            for (int k = 0; k < PX; ++k) {
              if (!pass[k]) continue;
              const float alpha = fminf(kAlphaMax, sp.o * splat_gauss(p2[k]));
              const float Tn = T[k] * (1.0f - alpha);
              if (Tn < kTMin) {            // the pixel stops; this entry is not blended
                fyk[k] = __builtin_nanf("");
                cs[k] = c;
                continue;
              }
              const float w = alpha * T[k];
              C[k][0] = fmaf(sp.r, w, C[k][0]);
              C[k][1] = fmaf(sp.g, w, C[k][1]);
              C[k][2] = fmaf(sp.b, w, C[k][2]);
              const float wl = alpha * Tl[k];
              Lc[k][0] = fmaf(sp.r, wl, Lc[k][0]);
              Lc[k][1] = fmaf(sp.g, wl, Lc[k][1]);
              Lc[k][2] = fmaf(sp.b, wl, Lc[k][2]);
              Tl[k] = Tl[k] * (1.0f - alpha);
              T[k] = Tn;
              last[k] = b0 + j + 1;
            }
          }
          continue;
        }
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          uint64_t todo = __ballot(fix[k] && cs[k] == nc);
          uint64_t list = 0;               // the entries that the lane's pixel passes
          while (todo) {
            const int p = (int)__builtin_ctzll(todo);
            todo &= todo - 1;
            const float qx = lane_f(L.fx, p), qy = lane_f(L.fy[k], p);
            const float p2 = splat_p2(s, __fsub_rn(qx, s.mx), __fsub_rn(qy, s.my));
            const uint64_t pass = splat_pass_lanes(s, p2);
            if (lane == p) list = pass;
          }
          while (list) {
            const int j = (int)__builtin_ctzll(list);
            list &= list - 1;
            const Splat& e = s_splat[j];
            const float p2 = splat_p2(e, __fsub_rn(L.fx, e.mx), __fsub_rn(L.fy[k], e.my));
            const float alpha = fminf(kAlphaMax, e.o * splat_gauss(p2));
            const float Tn = T[k] * (1.0f - alpha);
            if (Tn < kTMin) {              // the pixel stops; this entry is not blended
              cs[k] = c;
              break;
            }
            const float w = alpha * T[k];
            C[k][0] = fmaf(e.r, w, C[k][0]);
            C[k][1] = fmaf(e.g, w, C[k][1]);
            C[k][2] = fmaf(e.b, w, C[k][2]);
            const float wl = alpha * Tl[k];
            Lc[k][0] = fmaf(e.r, wl, Lc[k][0]);
            Lc[k][1] = fmaf(e.g, wl, Lc[k][1]);
            Lc[k][2] = fmaf(e.b, wl, Lc[k][2]);
            Tl[k] = Tl[k] * (1.0f - alpha);
            T[k] = Tn;
            last[k] = b0 + j + 1;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        if (cs[k] != c) continue;
        Ps[k] = Tl[k];
        Ls[k][0] = Lc[k][0];
        Ls[k][1] = Lc[k][1];
        Ls[k][2] = Lc[k][2];
      }
    };
    float4 buf[D][PX];
    int lbuf[D][PX];
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (d < nc) load_chunk(d, buf[d], lbuf[d]);
    for (int cb = 0; cb < nc; cb += D) {
      // every pixel stopped (or outside the image): the rest blends nothing
      bool done = true;
#pragma unroll
      for (int k = 0; k < PX; ++k) done = done && (cs[k] < nc || !L.inside[k]);
      if (__all(done)) break;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const int c = cb + d;
        if (c >= nc) break;
        float4 pl[PX];
        int ll[PX];
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          pl[k] = buf[d][k];
          ll[k] = lbuf[d][k];
        }
        if (c + D < nc) load_chunk(c + D, buf[d], lbuf[d]);
        join_chunk(c, pl, ll);
      }
    }
    const int64_t HW = (int64_t)a.H * a.W;
    float* img = image + (int64_t)L.slot * 3 * HW;
#pragma unroll
    for (int k = 0; k < PX; ++k) {
      if (!L.inside[k]) continue;
      const int64_t o = L.offset(a, k);
      img[o] = C[k][0] + T[k] * a.bg0;
      img[HW + o] = C[k][1] + T[k] * a.bg1;
      img[2 * HW + o] = C[k][2] + T[k] * a.bg2;
      T_final[(int64_t)L.slot * HW + o] = T[k];
      n_contrib[(int64_t)L.slot * HW + o] = last[k];
    }
    // checkpoints: slot c <- (T_c, U_c) from chunk c+1's (P, L), last first.
    // The backward reads slot c only for pixels that blend after chunk c, so
    // the walk starts below the last chunk holding a blend of any pixel
    // (after it T_c = T_final and U_c = bg exactly).
    int lc = 0;
#pragma unroll
    for (int k = 0; k < PX; ++k) lc = max(lc, (last[k] + ch.chunk - 1) / ch.chunk);
    const int c_top = min(nc - 2, wave_max_int(lc) - 2);
#pragma unroll
    for (int k = 0; k < PX; ++k) {
      float Tn = T[k], U[3] = {a.bg0, a.bg1, a.bg2};
      float4* col = ck + lane + k * kRasterWave;
      for (int cb = c_top; cb >= 0; cb -= D) {
        float4 v[D];
#pragma unroll
        for (int d = 0; d < D; ++d)
          if (cb - d >= 0) v[d] = col[(int64_t)(cb - d) * NP];
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const int c = cb - d;
          if (c < 0) break;
          const int e = c + 1;
          const float4 pl = e > cs[k] ? make_float4(1.0f, 0.0f, 0.0f, 0.0f)
                                      : (e == cs[k] ? make_float4(Ps[k], Ls[k][0], Ls[k][1],
                                                                  Ls[k][2])
                                                    : v[d]);
          const float Te = Tn / pl.x;
          U[0] = fmaf(pl.x, U[0], pl.y);
          U[1] = fmaf(pl.x, U[1], pl.z);
          U[2] = fmaf(pl.x, U[2], pl.w);
          col[(int64_t)c * NP] = make_float4(Te, U[0], U[1], U[2]);
          Tn = Te;
        }
      }
    }
  });
}

// ---------------------------------------------------------------- support count

// Per pixel, the number of list entries it blends (alpha test passed,
// transmittance still at or above the cut-off), with the forward's
// decisions: one work-group of 256 threads per tile, up to 2 pixels per
// thread, entries staged 256 at a time.  A measurement of the method's work
// (the pairs an exact rasteriser must composite), not part of the training
// step.
constexpr int kCountThreads = 256;

__global__ __launch_bounds__(kCountThreads) void k_raster_count(RasterDev a, int TW, int TH,
                                                                int32_t* __restrict__ n_blend) {
  __shared__ Splat s_sp[kCountThreads];
  const int64_t tile = blockIdx.x;
  const int slot = (int)(tile / a.tiles_per_slot);
  const int tt = (int)(tile - (int64_t)slot * a.tiles_per_slot);
  const int ty = tt / a.tiles_x, tx = tt - ty * a.tiles_x;
  const int t = threadIdx.x;
  float fx[2], fy[2], T[2];
  int cnt[2];
  bool live[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int p = t + k * kCountThreads;
    const int px = tx * TW + p % TW, py = ty * TH + p / TW;
    fx[k] = (float)px + 0.5f;
    fy[k] = (float)py + 0.5f;
    live[k] = p < TW * TH && px < a.W && py < a.H;
    T[k] = 1.0f;
    cnt[k] = 0;
  }
  const uint32_t start = a.ranges[2 * tile], end = a.ranges[2 * tile + 1];
  for (uint32_t b0 = start; b0 < end; b0 += kCountThreads) {
    if (__syncthreads_count(live[0] || live[1]) == 0) break;
    if (b0 + t < end) s_sp[t] = load_splat(a.rec, a.ids[b0 + t]);
    __syncthreads();
    const int n = (int)min((uint32_t)kCountThreads, end - b0);
    for (int j = 0; j < n; ++j) {
      const Splat sp = s_sp[j];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (!live[k]) continue;
        float p2;
        splat_p2_column<1>(sp, __fsub_rn(fx[k], sp.mx), &fy[k], &p2);
        if (!splat_pass(sp, p2)) continue;
        const float alpha = fminf(kAlphaMax, sp.o * splat_gauss(p2));
        const float Tn = T[k] * (1.0f - alpha);
        if (Tn < kTMin) {
          live[k] = false;
          continue;
        }
        T[k] = Tn;
        ++cnt[k];
      }
    }
    __syncthreads();
  }
  const int64_t HW = (int64_t)a.H * a.W;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int p = t + k * kCountThreads;
    const int px = tx * TW + p % TW, py = ty * TH + p / TW;
    if (p < TW * TH && px < a.W && py < a.H)
      n_blend[(int64_t)slot * HW + (int64_t)py * a.W + px] = cnt[k];
  }
}

__global__ void k_reset_queue(uint32_t* q) {
  if (threadIdx.x == 0) q[0] = 0u;
}

// ---------------------------------------------------------------- deterministic sum

// d_rec[p][c] += sum over pair p's emission slots of component c, in
// emission order; one thread per (pair, component), so the 9 threads of a
// pair read its slots' 36-byte records together.  pair_first [m][2] holds
// each pair's first emission index and its entry count.
__global__ __launch_bounds__(256) void k_dup_reduce(const uint32_t* __restrict__ pair_first,
                                                    int64_t m, const float* __restrict__ dup,
                                                    int64_t dup_cap, float* __restrict__ d_rec) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t p = i / GS_DREC_STRIDE;
  const int c = (int)(i - p * GS_DREC_STRIDE);
  if (p >= m) return;
  const int64_t nt = pair_first[2 * p + 1];
  if (nt <= 0) return;
  const int64_t e0 = pair_first[2 * p];
  if (e0 + nt > dup_cap) return;
  const float* g = dup + e0 * GS_DREC_STRIDE + c;
  float acc = 0.0f;
  for (int k = 0; k < nt; ++k) acc += g[k * GS_DREC_STRIDE];
  d_rec[p * GS_DREC_STRIDE + c] += acc;
}

// ---------------------------------------------------------------- dispatch

struct Launch {
  unsigned blocks;
  TileSched sch;
  ChunkDev ch;
  int64_t max_items;
  int fwd_waves, bwd_blocks;
  bool join_many;
};

// Whether the plan's forward composites chunk items and joins them.
static bool split_forward(const gs_raster_plan* plan) {
  return plan && plan->fwd_split && plan->chunk > 0 && plan->checkpoints;
}

// Whether a launch of `waves` waves for each of n_tiles tiles (and the rounding
// of the default order) holds at most 2^32 - 1 threads.
static bool launch_fits(int64_t n_tiles, int64_t waves) {
  return (n_tiles + 64) * waves * kRasterWave < (int64_t(1) << 32);
}

// Waves per tile of the forward.  Where the plan leaves the choice (fwd_waves
// 0 or 1, no queue): the most that the tile's pixels allow, one 8x8 block each
// for 16x16 tiles.  A wave's time is its list's length times its visits' cost,
// and both the pixels per lane and the entries that reach its box fall with
// more waves (one against the most): 1920x1080 in 16x16 tiles 946 / 225 us, 32
// images of 640x360 1526 / 508, 333x251 224 / 65, 128x128 137 / 48.
static int forward_waves(int tw, int th, int64_t n_tiles, const gs_raster_plan* plan) {
  if (split_forward(plan) || (plan && plan->queue)) return 1;
  if (plan && plan->fwd_waves > 1) return plan->fwd_waves;
  const int px = tw * th / kRasterWave;
  int nw = px % 4 == 0 ? 4 : (px % 2 == 0 ? 2 : 1);
  while (nw > 1 && !launch_fits(n_tiles, nw)) nw /= 2;
  return nw;
}

// The grid of a queue's plan, at most.
static int64_t queue_waves(const gs_raster_plan* plan) {
  return plan->persistent_waves > 0 ? plan->persistent_waves : (int64_t)device_cu_count() * 16;
}

// 8x8 blocks that a wave of the whole-list backward takes: one, or all of its
// tile where gradients are stored, and where the number of waves and not the
// longest lists bounds the call, since every block stages its tile's whole
// list.  That is so
// - with a queue of few waves.  A wave per block / per tile: 1920x1080, 16
//   tiles a wave 2302 / 1952 us, 32 4234 / 3564, but 8 tiles 1273 / 1628;
//   640x360, 14 tiles a wave 1778 / 1562, 4 tiles 514 / 838;
// - of many tiles (from 64 a CU) with few pairs of an image and a Gaussian per
//   tile; the more tiles a CU has, the less a long list stands out.  Earlier in
//   longest-first order, which ends on short lists.  Images of 1920x1080 in
//   16x16 tiles, longest first / default order: 4 images, 127 tiles a CU, 2
//   pairs a tile 398 / 291 and 475 / 391 us, 24 pairs 733 / 613 and 849 / 940,
//   122 pairs 1630 / 1714 and 1815 / 2479; 16 images, 510 tiles a CU, 2 pairs
//   1564 / 930 and 1690 / 1194, 24 pairs 2718 / 2012 and 2823 / 2502, 122 pairs
//   5818 / 5002 and 6074 / 6387; of 3840x2160, one image, 127 tiles a CU, 410
//   pairs 4948 / 14488 and 6702 / 16139; eight, 1012 and 123 in the default
//   order 8486 / 12725.  (An object on a tenth of the image has fewer tiles at
//   work than the call has, and would keep its blocks longer: 4 images of
//   3840x2160 with 31 pairs a tile 1303 / 2906.  The host does not know that;
//   the wave per tile is then as fast as the kernel without blocks was, 2896.
//   Long lists by blocks and short ones by tiles, in two launches, gave none of
//   the cases above its better time.)
constexpr int64_t kQueueTilesPerWave = 12;
static int backward_blocks(int tw, int th, int64_t n_tiles, int64_t pairs,
                           const gs_raster_plan* plan) {
  const int64_t cus = device_cu_count();
  bool per_tile = (plan && plan->dup_grads) || !launch_fits(n_tiles, tw * th / kRasterWave);
  if (plan && plan->queue)
    per_tile |= n_tiles > kQueueTilesPerWave * queue_waves(plan);
  else if (n_tiles >= 64 * cus)
    per_tile |= pairs / n_tiles <= n_tiles / cus / (plan && plan->tile_order ? 2 : 16);
  return per_tile ? tw * th / kRasterWave : 1;
}

// Whether the join visits a stopping chunk's entries with all lanes: up to a
// pair of an image and a Gaussian per 16 pixels, which then are large splats,
// and with several pixels a lane.  Whole split forward, all lanes / pixel by
// pixel, 16x16 tiles of 1920x1080: 20K Gaussians 145 / 178 us, 80K 215 / 235,
// 160K 268 / 269, 1M 699 / 498; 32x16: 20K 240 / 329, 160K 488 / 520, 1M 1547 /
// 1006; 8x8, 20K: 84 / 80.
static bool join_many(int tw, int th, int64_t n_tiles, int64_t pairs) {
  return tw * th > 64 && pairs * 16 <= n_tiles * tw * th;
}

static Launch make_launch(const RasterDev& a, const gs_tiling* tiling, int64_t pairs,
                          const gs_raster_plan* plan) {
  Launch L;
  L.sch.order = plan ? plan->tile_order : nullptr;
  L.sch.queue = plan ? plan->queue : nullptr;
  L.sch.run = (uint32_t)xcd_run(a.n_tiles, a.tiles_per_slot);
  L.ch.chunk = plan ? plan->chunk : 0;
  L.ch.offset = plan ? plan->chunk_offset : nullptr;
  L.ch.items = plan ? plan->chunk_items : nullptr;
  L.ch.ck = plan && plan->chunk > 0 ? reinterpret_cast<float4*>(plan->checkpoints) : nullptr;
  L.max_items = plan ? plan->max_items : 0;
  L.fwd_waves = forward_waves(tiling->tile_w, tiling->tile_h, a.n_tiles, plan);
  L.bwd_blocks = backward_blocks(tiling->tile_w, tiling->tile_h, a.n_tiles, pairs, plan);
  L.join_many = join_many(tiling->tile_w, tiling->tile_h, a.n_tiles, pairs);
  if (L.sch.queue) {
    L.blocks = (unsigned)std::min<int64_t>(queue_waves(plan), std::max<int64_t>(a.n_tiles, 1));
  } else if (L.sch.order) {
    L.blocks = (unsigned)std::max<int64_t>(a.n_tiles, 1);
  } else {
    const int64_t round = 8 * (int64_t)L.sch.run;
    L.blocks = (unsigned)(ceil_div(a.n_tiles, round) * round);
  }
  return L;
}

template <int TW, int TH>
static void launch_fwd(const RasterDev& a, const Launch& L, float* image, float* T_final,
                       int32_t* n_contrib, hipStream_t s) {
  constexpr int PXT = TileGeom<TW, TH>::PX;
  constexpr int kMost = PXT % 4 == 0 ? 4 : (PXT % 2 == 0 ? 2 : 1);
  const int nw = L.fwd_waves;
#define GS_FWD_LAUNCH(NW)                                                                       \
  hipLaunchKernelGGL((k_raster_fwd<TW, TH, NW>), dim3(L.blocks), dim3(NW * kRasterWave), 0, s, a, \
                     L.sch, L.ch, image, T_final, n_contrib)
  if constexpr (kMost >= 4) {
    if (nw == 4) {
      GS_FWD_LAUNCH(4);
      return;
    }
  }
  if constexpr (kMost >= 2) {
    if (nw == 2) {
      GS_FWD_LAUNCH(2);
      return;
    }
  }
  GS_FWD_LAUNCH(1);
#undef GS_FWD_LAUNCH
}

template <int TW, int TH>
static void launch_fwd_split(const RasterDev& a, const Launch& L, uint16_t* chunk_last,
                             float* image, float* T_final, int32_t* n_contrib, hipStream_t s) {
  hipLaunchKernelGGL((k_raster_fwd_part<TW, TH>), dim3((unsigned)L.max_items), dim3(kRasterWave),
                     0, s, a, L.ch, chunk_last);
  constexpr bool kMany = TW * TH > 64;
  if (kMany && L.join_many)
    hipLaunchKernelGGL((k_raster_fwd_join<TW, TH, kMany>), dim3(L.blocks), dim3(kRasterWave), 0, s,
                       a, L.sch, L.ch, chunk_last, image, T_final, n_contrib);
  else
    hipLaunchKernelGGL((k_raster_fwd_join<TW, TH, false>), dim3(L.blocks), dim3(kRasterWave), 0, s,
                       a, L.sch, L.ch, chunk_last, image, T_final, n_contrib);
}

template <int TW, int TH>
static void launch_bwd(const RasterDev& a, const Launch& L, const float* T_final,
                       const int32_t* n_contrib, const float* d_image, int mode, float* d_rec,
                       hipStream_t s) {
  // quadrant groups pay off for the small footprints of 8x8 tiles (the 4K
  // octant: 2.34 -> 1.98 ms); at 16x16 they measured the same as one wave
  // per item (0.421 vs 0.424 ms at 1080p)
  constexpr bool kQuad = TW == 8 && TH == 8;
  if (kQuad && mode == GS_BWD_STORED && L.ch.chunk > 0 && !a.dup_grads)
    hipLaunchKernelGGL((k_raster_bwd_chunked_q<kQuad ? TW : 8, kQuad ? TH : 8>),
                       dim3((unsigned)L.max_items), dim3(kRasterWave), 0, s, a, L.ch, T_final,
                       n_contrib, d_image, d_rec);
  else if (mode == GS_BWD_STORED && L.ch.chunk > 0)
    hipLaunchKernelGGL((k_raster_bwd_chunked<TW, TH>), dim3((unsigned)L.max_items),
                       dim3(kRasterWave), 0, s, a, L.ch, T_final, n_contrib, d_image, d_rec);
  else {
    // whole lists: a wave per 8x8 block, or per tile where gradients are stored
    constexpr int NB = TW * TH / 64;
    const bool rec = mode == GS_BWD_RECOMPUTE;
    // (a queue's grid is persistent and takes the blocks of a tile as items;
    // more waves than tiles measured slower: 336 tiles 183 us, 207 on 1344 waves)
    const bool per_tile = L.bwd_blocks > 1;
    int64_t waves = per_tile || L.sch.queue ? L.blocks : (int64_t)L.blocks * NB;
    int lg_share = 0;
    if (!L.sch.queue)
      while (lg_share < kBwdShareLgMax && 2 * waves <= kBwdShareWavesPerCu * device_cu_count()) {
        ++lg_share;
        waves *= 2;
      }
    const dim3 blocks((unsigned)waves);
#define GS_BWD_LAUNCH(NK, REC)                                                                \
  hipLaunchKernelGGL((k_raster_bwd<TW, TH, NK, REC>), blocks, dim3(kRasterWave), 0, s, a,     \
                     L.sch, lg_share, T_final, n_contrib, d_image, d_rec)
    if (per_tile && rec) GS_BWD_LAUNCH(NB, true);
    else if (per_tile) GS_BWD_LAUNCH(NB, false);
    else if (rec) GS_BWD_LAUNCH(1, true);
    else GS_BWD_LAUNCH(1, false);
#undef GS_BWD_LAUNCH
  }
}

// Tile shapes with a compiled rasteriser.
#define GS_RASTER_SHAPES(X) X(16, 16) X(8, 8) X(16, 8) X(32, 8) X(8, 16) X(32, 16) X(16, 32)

static bool raster_shape_supported(int tw, int th) {
#define GS_SHAPE_CASE(a, b) if (tw == a && th == b) return true;
  GS_RASTER_SHAPES(GS_SHAPE_CASE)
#undef GS_SHAPE_CASE
  return false;
}

static gs_status raster_prepare(const gs_projected* proj, const gs_views* views,
                                const gs_tiling* tiling, const uint32_t* ids,
                                const uint32_t* tile_ranges, const float bg[3], const char* who,
                                RasterDev& a) {
  GS_REQUIRE(proj != nullptr && bg != nullptr, "%s: NULL argument", who);
  gs_status st = check_views(views, tiling, who);
  if (st != GS_OK) return st;
  GS_REQUIRE(raster_shape_supported(tiling->tile_w, tiling->tile_h),
             "%s: tile %dx%d has no rasteriser (16x16, 8x8, 16x8, 32x8, 8x16, 32x16, 16x32)", who,
             tiling->tile_w, tiling->tile_h);
  GS_REQUIRE(tile_ranges != nullptr, "%s: NULL tile_ranges", who);
  GS_REQUIRE(proj->m == 0 || (proj->rec && ids), "%s: NULL rec/ids", who);
  a.rec = proj->rec;
  a.ids = ids;
  a.ranges = tile_ranges;
  a.W = tiling->width;
  a.H = tiling->height;
  a.tiles_x = (int)ceil_div(tiling->width, tiling->tile_w);
  a.tiles_per_slot = a.tiles_x * (int)ceil_div(tiling->height, tiling->tile_h);
  a.n_tiles = (int64_t)a.tiles_per_slot * views->n_slots;
  a.bg0 = bg[0];
  a.bg1 = bg[1];
  a.bg2 = bg[2];
  a.emit = nullptr;
  a.dup_grads = nullptr;
  a.dup_cap = 0;
  return GS_OK;
}

static gs_status plan_prepare(const gs_raster_plan* plan, const gs_tiling* tiling, hipStream_t s,
                              const char* who) {
  if (!plan) return GS_OK;
  GS_REQUIRE(plan->persistent_waves >= 0, "%s: persistent_waves < 0", who);
  const int nw = plan->fwd_waves;
  GS_REQUIRE(nw == 0 || nw == 1 || nw == 2 || nw == 4, "%s: fwd_waves %d not in {0, 1, 2, 4}",
             who, nw);
  GS_REQUIRE(nw <= 1 || (tiling->tile_w * tiling->tile_h / kRasterWave) % nw == 0,
             "%s: fwd_waves %d does not divide the %dx%d tile's %d pixels per lane", who, nw,
             tiling->tile_w, tiling->tile_h, tiling->tile_w * tiling->tile_h / kRasterWave);
  GS_REQUIRE(nw <= 1 || plan->queue == nullptr, "%s: fwd_waves > 1 needs a non-persistent plan",
             who);
  if (plan->chunk > 0) {
    GS_REQUIRE(plan->chunk % kRasterWave == 0, "%s: chunk %d is not a multiple of 64", who,
               plan->chunk);
    GS_REQUIRE(plan->chunk_offset && plan->chunk_items && plan->checkpoints &&
                   plan->max_items > 0 && plan->max_items < (int64_t(1) << 31),
               "%s: chunked plan needs chunk_offset, chunk_items, checkpoints, max_items", who);
  }
  if (plan->queue) {
    hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, s, plan->queue);
    GS_LAUNCH_CHECK(who);
  }
  return GS_OK;
}

}  // namespace gsmi

using namespace gsmi;

extern "C" {

static int64_t call_tiles(const gs_tiling* t, int32_t n_slots) {
  return ceil_div(t->width, t->tile_w) * ceil_div(t->height, t->tile_h) * n_slots;
}

int32_t gs_raster_fwd_waves(const gs_tiling* tiling, int32_t n_slots, const gs_raster_plan* plan) {
  if (!tiling || !raster_shape_supported(tiling->tile_w, tiling->tile_h)) return 0;
  return forward_waves(tiling->tile_w, tiling->tile_h, call_tiles(tiling, n_slots), plan);
}

int32_t gs_raster_join_many(const gs_tiling* tiling, int32_t n_slots, int64_t pairs) {
  if (!tiling || !raster_shape_supported(tiling->tile_w, tiling->tile_h)) return 0;
  return join_many(tiling->tile_w, tiling->tile_h, call_tiles(tiling, n_slots), pairs);
}

int32_t gs_raster_bwd_blocks(const gs_tiling* tiling, int32_t n_slots, int64_t pairs,
                             const gs_raster_plan* plan) {
  if (!tiling || !raster_shape_supported(tiling->tile_w, tiling->tile_h)) return 0;
  return backward_blocks(tiling->tile_w, tiling->tile_h, call_tiles(tiling, n_slots), pairs, plan);
}

gs_status gs_raster_fwd(const gs_projected* proj, const gs_views* views, const gs_tiling* tiling,
                        const uint32_t* ids, const uint32_t* tile_ranges, const float bg[3],
                        float* image, float* T_final, int32_t* n_contrib,
                        const gs_raster_plan* plan, void* stream) {
  clear_error();
  RasterDev a;
  gs_status st = raster_prepare(proj, views, tiling, ids, tile_ranges, bg, "gs_raster_fwd", a);
  if (st != GS_OK) return st;
  GS_REQUIRE(image != nullptr, "gs_raster_fwd: NULL image");
  GS_REQUIRE((T_final == nullptr) == (n_contrib == nullptr),
             "gs_raster_fwd: T_final and n_contrib must both be set or both be NULL");
  hipStream_t s = as_stream(stream);
  st = plan_prepare(plan, tiling, s, "gs_raster_fwd");
  if (st != GS_OK) return st;
  const Launch L = make_launch(a, tiling, proj->m, plan);
  const bool split = split_forward(plan);
  GS_REQUIRE(!split || (plan->chunk_last && T_final),
             "gs_raster_fwd: fwd_split needs chunk_last and the stored state (T_final, n_contrib)");
#define GS_FWD_CASE(a_, b_)                                                          \
  if (tiling->tile_w == a_ && tiling->tile_h == b_) {                                \
    if (split)                                                                       \
      launch_fwd_split<a_, b_>(a, L, plan->chunk_last, image, T_final, n_contrib, s); \
    else                                                                             \
      launch_fwd<a_, b_>(a, L, image, T_final, n_contrib, s);                        \
  } else
  GS_RASTER_SHAPES(GS_FWD_CASE) {}
#undef GS_FWD_CASE
  GS_LAUNCH_CHECK("gs_raster_fwd");
  return GS_OK;
}

gs_status gs_raster_bwd(const gs_projected* proj, const gs_views* views, const gs_tiling* tiling,
                        const uint32_t* ids, const uint32_t* tile_ranges, const float bg[3],
                        const float* T_final, const int32_t* n_contrib, const float* d_image,
                        int32_t mode, float* d_rec, const gs_raster_plan* plan, void* stream) {
  clear_error();
  RasterDev a;
  gs_status st = raster_prepare(proj, views, tiling, ids, tile_ranges, bg, "gs_raster_bwd", a);
  if (st != GS_OK) return st;
  GS_REQUIRE(mode == GS_BWD_STORED || mode == GS_BWD_RECOMPUTE, "gs_raster_bwd: bad mode %d",
             mode);
  GS_REQUIRE(d_image && d_rec, "gs_raster_bwd: NULL d_image/d_rec");
  GS_REQUIRE(mode == GS_BWD_RECOMPUTE || (T_final && n_contrib),
             "gs_raster_bwd: STORED mode needs T_final and n_contrib");
  hipStream_t s = as_stream(stream);
  const bool det = plan && plan->dup_grads;
  if (det) {
    GS_REQUIRE(plan->pair_first && plan->emit_idx && plan->dup_capacity > 0,
               "gs_raster_bwd: deterministic mode needs pair_first, emit_idx, dup_capacity");
    a.emit = plan->emit_idx;
    a.dup_grads = plan->dup_grads;
    a.dup_cap = plan->dup_capacity;
  }
  st = plan_prepare(plan, tiling, s, "gs_raster_bwd");
  if (st != GS_OK) return st;
  const Launch L = make_launch(a, tiling, proj->m, plan);
#define GS_BWD_CASE(a_, b_)                                                   \
  if (tiling->tile_w == a_ && tiling->tile_h == b_)                           \
    launch_bwd<a_, b_>(a, L, T_final, n_contrib, d_image, mode, d_rec, s);    \
  else
  GS_RASTER_SHAPES(GS_BWD_CASE) {}
#undef GS_BWD_CASE
  GS_LAUNCH_CHECK("gs_raster_bwd");
  if (det && proj->m > 0) {
    hipLaunchKernelGGL(k_dup_reduce, dim3((unsigned)ceil_div(proj->m * GS_DREC_STRIDE, 256)),
                       dim3(256), 0, s,
                       plan->pair_first, proj->m, plan->dup_grads,
                       plan->dup_capacity, d_rec);
    GS_LAUNCH_CHECK("gs_raster_bwd/reduce");
  }
  return GS_OK;
}

gs_status gs_raster_count(const gs_projected* proj, const gs_views* views,
                          const gs_tiling* tiling, const uint32_t* ids,
                          const uint32_t* tile_ranges, int32_t* n_blend, void* stream) {
  clear_error();
  RasterDev a;
  const float bg[3] = {0.f, 0.f, 0.f};
  gs_status st = raster_prepare(proj, views, tiling, ids, tile_ranges, bg, "gs_raster_count", a);
  if (st != GS_OK) return st;
  GS_REQUIRE(n_blend != nullptr, "gs_raster_count: NULL n_blend");
  GS_REQUIRE(tiling->tile_w * tiling->tile_h <= 2 * kCountThreads,
             "gs_raster_count: tile of %d pixels (at most %d)", tiling->tile_w * tiling->tile_h,
             2 * kCountThreads);
  if (a.n_tiles == 0) return GS_OK;
  hipLaunchKernelGGL(k_raster_count, dim3((unsigned)a.n_tiles), dim3(kCountThreads), 0,
                     as_stream(stream), a, tiling->tile_w, tiling->tile_h, n_blend);
  GS_LAUNCH_CHECK("gs_raster_count");
  return GS_OK;
}

}  // extern "C"
