// Builds by records: the sort moves one record per <object, segment> instead
// of one pair per <object, cell>.
//
// A segment is up to 256 cells with consecutive ids: a stretch of one row of
// cells, or several whole rows where rows are short.  A record is the part of
// an object's cell box inside one segment, a rectangle of its cells.  The
// objects' boxes in the grid of segments are expanded into records exactly as
// boxes of cells are expanded into pairs (equal work per record); the records
// are radix-sorted by segment, which takes fewer items and fewer digits than
// the pairs would (10M architectural triangles: 20M records of 17-bit segments
// against 51M pairs of 25-bit cells; hundreds of cells per box: a sixth of the
// pairs); and each segment's records, which a stable sort leaves in object
// order, are expanded into its pairs by one wave, which counts them per cell
// in LDS, writes the cells' ranges from those counts and places every pair at
// its rank.  Cells and objects are then written once, in order, and the pairs
// are never read again.
//
// A record's 16 bits of rectangle (first cell, extents) share the sort's 64
// bits with its segment and its object:
//   key = segment << ck | low ck bits of code
//   val = object        | code >> ck << objbits
//   code = (y0 << wx | x0) << (wx + wy) | (my - 1) << wx | (mx - 1)
#pragma once

#include "ranges.hpp"


namespace gb {

struct SegCode {
  uint32_t wx, wy;          // bits of a cell's x and y inside its segment
  uint32_t ck;              // bits of the code kept in the key (at least the wx + wy of the extents)
  uint32_t objbits;         // bits of an object id in the value
  uint32_t nsegs;           // segments of all grids
};

// ---------------------------------------------------------------------------
// Expansion of objects into records.
// ---------------------------------------------------------------------------
struct RecordArgs {
  ExpandOutArgs o;          // cells/objs receive the records' keys and values
  SegCode code;
};

// What the expansion needs of an object's grid.
struct SegParams {
  uint32_t sx, sy, mgx, mgy, nsx, nsxy, seg_base, tri_base;
};

GB_DEV SegParams seg_params(const GridDev& G) {
  return {G.sx, G.sy, G.mgx, G.mgy, G.nsx, G.nsx * G.nsy, G.seg_base, G.tri_base};
}

// Records tile * N .. of one expansion tile (N = Block * K), K consecutive
// ones per thread: keys and values.  Returns the tile's record count.  Where
// (wy = 0): also each record's first cell in the grid, x | y << 10 | z << 20.
template <int Block, int K, bool Batched, bool OneGrid, bool Where = false>
GB_DEV uint32_t record_tile(const ExpandArgs& a, const SegCode& c, uint32_t tile, uint64_t nrec, uint32_t ntiles,
                            uint32_t* s_slot, uint32_t* s_wtot, uint32_t (&keys)[K], uint32_t (&vals)[K],
                            uint32_t* xyz = nullptr) {
  constexpr int N = Block * K;
  const uint32_t tid = threadIdx.x;
  const uint64_t base = static_cast<uint64_t>(tile) * N;
  uint32_t sv[K], t0, s0;
  const uint32_t n = tile_owners<Block, K>(a, tile, nrec, ntiles, s_slot, s_wtot, sv, t0, s0);
  SegParams p;
  uint32_t cur = 0, next_tb = 0xFFFFFFFFu;
  if constexpr (Batched) {
    // the tile's first grid, made visibly uniform so that its parameters are scalar loads
    cur = __builtin_amdgcn_readfirstlane(a.tfg[__builtin_amdgcn_readfirstlane(tile)]);
    p = seg_params(OneGrid ? uniform_grid(a.gs.table + cur) : a.gs.table[cur]);
    if constexpr (!OneGrid) next_tb = cur + 1 < a.gs.ngrids ? a.gs.table[cur + 1].tri_base : 0xFFFFFFFFu;
  } else {
    p = seg_params(a.gs.one);
  }
  uint64_t bx[K];
#pragma unroll
  for (int k = 0; k < K; ++k) bx[k] = a.box[t0 + (sv[k] >> 16)];  // all box loads in flight
  // the object's box in the grid of segments, stepped x fastest along its records
  uint32_t x = 0, y = 0, z = 0;
  const uint32_t kmask = (1u << c.ck) - 1u;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint32_t idx = tid * K + k;
    const uint32_t obj = t0 + (sv[k] >> 16);
    if constexpr (Batched && !OneGrid) {
      if (obj >= next_tb) {  // a thread's objects come in increasing order
        cur = grid_of_tri<true>(a.gs, obj, cur);
        p = seg_params(a.gs.table[cur]);
        next_tb = cur + 1 < a.gs.ngrids ? a.gs.table[cur + 1].tri_base : 0xFFFFFFFFu;
      }
    }
    const Box b = unpack_box(bx[k]);
    const uint32_t hx = b.lo[0] + b.m[0] - 1, hy = b.lo[1] + b.m[1] - 1;
    const uint32_t slx = div_small(b.lo[0], p.mgx), smx = div_small(hx, p.mgx) - slx + 1;
    const uint32_t sly = div_small(b.lo[1], p.mgy), smy = div_small(hy, p.mgy) - sly + 1;
    if (k == 0) {
      const uint32_t ii = tid * K < n ? tid * K : n - 1;
      const uint32_t v = sv[0];
      const uint32_t rid = (v >> 16) == 0 ? static_cast<uint32_t>(base) + ii - s0 : ii - (v & 0xFFFFu);
      const uint32_t sxy = smx * smy;
      z = rid / sxy;
      const uint32_t r2 = rid - z * sxy;
      y = r2 / smx;
      x = r2 - y * smx;
    } else if (sv[k] != sv[k > 0 ? k - 1 : 0]) {
      x = y = z = 0;  // a new owner starts here
    } else {
      ++x;
      const bool cx = x == smx;
      x = cx ? 0u : x;
      y += cx ? 1u : 0u;
      const bool cy = y == smy;
      y = cy ? 0u : y;
      z += cy ? 1u : 0u;
    }
    // the box clipped to segment (slx + x, sly + y): its first cell and extents there
    const uint32_t ox = __umul24(slx + x, p.sx), oy = __umul24(sly + y, p.sy);
    const uint32_t x0 = b.lo[0] > ox ? b.lo[0] - ox : 0u, y0 = b.lo[1] > oy ? b.lo[1] - oy : 0u;
    const uint32_t x1 = hx - ox < p.sx - 1 ? hx - ox : p.sx - 1, y1 = hy - oy < p.sy - 1 ? hy - oy : p.sy - 1;
    const uint32_t seg = p.seg_base + (slx + x) + p.nsx * (sly + y) + p.nsxy * (b.lo[2] + z);
    const uint32_t code = (((y0 << c.wx) | x0) << (c.wx + c.wy)) | ((y1 - y0) << c.wx) | (x1 - x0);
    keys[k] = (seg << c.ck) | (code & kmask);
    vals[k] = (obj - (Batched ? p.tri_base : 0u)) | ((code >> c.ck) << c.objbits);
    if constexpr (Where) xyz[k] = (ox + x0) | ((sly + y) << 10) | ((b.lo[2] + z) << 20);  // (one row: sly + y is y)
    if (idx >= n) {
      keys[k] = 0xFFFFFFFFu;
      vals[k] = 0;
    }
    __builtin_amdgcn_sched_barrier(0);  // one record's temporaries at a time
  }
  __syncthreads();
  return n;
}

// Four records per thread and 1024 threads: 64 VGPRs, so two workgroups fill a CU
// (eight records on 512 threads spilled at six waves per SIMD and took 170 us on
// 20M records, against 95).  Tiles go round by a fixed stride: they are equal work.
template <int Block, int K, int RB, bool Batched>
__global__ __launch_bounds__(Block, 8) void record_kernel(RecordArgs a) {
  constexpr int N = Block * K;
  constexpr int R = 1 << RB;
  __shared__ uint32_t s_owner[padded(N)];
  __shared__ uint32_t s_hist[4 * R];
  __shared__ uint32_t s_wtot[Block / kWave];
  if (build_failed(a.o.ctl)) return;
  const uint64_t nrec = a.o.ctl->nitems;
  const uint32_t ntiles = static_cast<uint32_t>((nrec + N - 1) / N);
  clear_status<Block>(a.o.clear, nrec);
  for (uint32_t i = threadIdx.x; i < a.o.plan.passes * R; i += Block) s_hist[i] = 0;
  __syncthreads();
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    uint32_t keys[K], vals[K];
    uint32_t n;
    if constexpr (Batched) {
      if (tile_straddles(a.o.ex, __builtin_amdgcn_readfirstlane(tile), ntiles)) continue;
    }
    n = record_tile<Block, K, Batched, true>(a.o.ex, a.code, tile, nrec, ntiles, s_owner, s_wtot, keys, vals);
    store_tile<Block, K, RB>(a.o, tile, n, keys, vals, s_hist);
  }
  flush_hist<RB, Block>(a.o.plan, a.o.hist, s_hist);
}

// Batched builds: the tiles whose objects lie in more than one grid.
template <int Block, int K, int RB>
__global__ __launch_bounds__(Block, 2) void record_straddle_kernel(RecordArgs a) {
  constexpr int N = Block * K;
  constexpr int R = 1 << RB;
  __shared__ uint32_t s_owner[padded(N)];
  __shared__ uint32_t s_hist[4 * R];
  __shared__ uint32_t s_wtot[Block / kWave];
  if (build_failed(a.o.ctl)) return;
  const uint64_t nrec = a.o.ctl->nitems;
  const uint32_t ntiles = static_cast<uint32_t>((nrec + N - 1) / N);
  for (uint32_t i = threadIdx.x; i < a.o.plan.passes * R; i += Block) s_hist[i] = 0;
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    if (!tile_straddles(a.o.ex, __builtin_amdgcn_readfirstlane(tile), ntiles)) continue;
    __syncthreads();  // the previous tile's readers of s_owner are done
    uint32_t keys[K], vals[K];
    const uint32_t n =
        record_tile<Block, K, true, false>(a.o.ex, a.code, tile, nrec, ntiles, s_owner, s_wtot, keys, vals);
    store_tile<Block, K, RB>(a.o, tile, n, keys, vals, s_hist);
  }
  flush_hist<RB, Block>(a.o.plan, a.o.hist, s_hist);
}

// ---------------------------------------------------------------------------
// The list of segments that hold records: each one's segment, first record and
// first pair, in segment order (a scan over the sorted records' keys).
// ---------------------------------------------------------------------------
struct alignas(16) SegEntry {
  uint32_t seg, rec, pair, pad;
};

struct SegListArgs {
  const uint32_t* keys;     // [records] sorted
  SegCode code;
  SegEntry* list;           // [list_cap + 1]; entry nlist closes the list: (nsegs, records, pairs)
  uint32_t list_cap;
  uint64_t* status;         // [tiles] look-back words (zeroed): heads << 33 | pairs
  uint32_t vec16;           // keys is 16-byte aligned
  Control* ctl;
};

// Each wave takes 1024 consecutive records in four groups of four per lane, so
// that every load is a whole line, and scans group by group.
template <int Block>
__global__ __launch_bounds__(Block) void seg_list_kernel(SegListArgs a) {
  constexpr int W = Block / kWave;
  constexpr int Q = 4;                       // groups of a wave, 4 records per lane each
  constexpr uint32_t kGroup = 4 * kWave;     // 256 records
  constexpr int N = Block * 4 * Q;
  static_assert(static_cast<uint64_t>(N) * 256 < (uint64_t{1} << 31), "a tile's pairs fit 31 bits");
  __shared__ uint32_t s_heads[W], s_pairs[W];
  __shared__ uint64_t s_prefix;
  __shared__ uint32_t s_tile;
  if (build_failed(a.ctl)) return;
  const uint64_t nrec = a.ctl->nitems;
  const uint32_t ntiles = static_cast<uint32_t>((nrec + N - 1) / N);
  const uint32_t lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t ck = a.code.ck, wx = a.code.wx;
  const uint32_t xmask = (1u << wx) - 1u, ymask = (1u << a.code.wy) - 1u;
  while (true) {
    const uint32_t tile = next_tile(&a.ctl->tile_counter[kCtrSplit], &s_tile);
    if (tile >= ntiles) return;
    const uint64_t wbase = static_cast<uint64_t>(tile) * N + static_cast<uint64_t>(w) * (Q * kGroup);
    // the wave's records that exist; past them a lane repeats the last record of
    // the list, which is no head and whose pairs are left out
    const uint32_t n = static_cast<uint32_t>(wbase >= nrec ? 0 : nrec - wbase < Q * kGroup ? nrec - wbase : Q * kGroup);
    const uint32_t* keys = a.keys + (wbase < nrec ? wbase : 0);
    uint32_t key[Q][4];
    if (n == Q * kGroup && a.vec16) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint4 v = reinterpret_cast<const uint4*>(keys)[q * kWave + lane];
        key[q][0] = v.x;
        key[q][1] = v.y;
        key[q][2] = v.z;
        key[q][3] = v.w;
      }
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t i = q * kGroup + 4 * lane + k;
          key[q][k] = n ? keys[i < n ? i : n - 1] : 0u;
        }
    }
    // the record before the wave's first (none: a segment that does not exist)
    uint32_t before = n && wbase > 0 ? *(keys - 1) >> ck : 0xFFFFFFFFu;
    uint32_t head[Q], hx[Q], px[Q];  // head bits of the lane's four records; heads and pairs before them in the wave
    uint32_t heads = 0, pairs = 0;   // of the wave
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t s3 = key[q][3] >> ck;
      uint32_t last = static_cast<uint32_t>(__shfl_up(static_cast<int>(s3), 1, kWave));
      if (lane == 0) last = before;
      before = wave_readlane(s3, kWave - 1);
      uint32_t h = 0, p = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t seg = key[q][k] >> ck;
        const bool in = q * kGroup + 4 * lane + k < n;
        h |= (in && seg != last ? 1u : 0u) << k;
        last = seg;
        p += in ? __umul24((key[q][k] & xmask) + 1u, ((key[q][k] >> wx) & ymask) + 1u) : 0u;
      }
      const uint32_t hc = static_cast<uint32_t>(__builtin_popcount(h));
      const uint32_t hi = wave_inclusive(hc, OpAdd{}), pi = wave_inclusive(p, OpAdd{});
      head[q] = h;
      hx[q] = heads + hi - hc;
      px[q] = pairs + pi - p;
      heads += wave_readlane(hi, kWave - 1);
      pairs += wave_readlane(pi, kWave - 1);
    }
    if (lane == 0) {
      s_heads[w] = heads;
      s_pairs[w] = pairs;
    }
    __syncthreads();
    uint32_t hw = 0, pw = 0, ht = 0, pt = 0;  // before this wave in the tile; the tile's totals
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const uint32_t h = s_heads[i], p = s_pairs[i];
      hw += static_cast<uint32_t>(i) < w ? h : 0u;
      pw += static_cast<uint32_t>(i) < w ? p : 0u;
      ht += h;
      pt += p;
    }
    if (w == 0) {
      const uint64_t total = (static_cast<uint64_t>(ht) << 33) + pt;
      const uint64_t p = lookback_wave(a.status, tile, total);
      if (lane == 0) {
        s_prefix = p;
        if (tile == ntiles - 1) {
          const uint64_t all = p + total;
          const uint32_t nheads = static_cast<uint32_t>(all >> 33);
          const uint64_t npairs = all & ((uint64_t{1} << 33) - 1);
          // the records must hold exactly the pairs the count added up
          if (npairs != a.ctl->npairs || nheads > a.list_cap) {
            atomicOr(&a.ctl->error, kErrInternal);
          } else {
            a.list[nheads] = {a.code.nsegs, static_cast<uint32_t>(nrec), static_cast<uint32_t>(npairs), 0u};
            a.ctl->nlist = nheads;
          }
        }
      }
    }
    __syncthreads();
    const uint32_t j0 = static_cast<uint32_t>(s_prefix >> 33) + hw, p0 = static_cast<uint32_t>(s_prefix) + pw;  // (pairs < 2^32)
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      uint32_t j = j0 + hx[q], pos = p0 + px[q];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if ((head[q] >> k) & 1u) {
          if (j < a.list_cap)
            a.list[j] = {key[q][k] >> ck, static_cast<uint32_t>(wbase) + q * kGroup + 4 * lane + k, pos, 0u};
          ++j;
        }
        pos += __umul24((key[q][k] & xmask) + 1u, ((key[q][k] >> wx) & ymask) + 1u);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// From a segment's records to its pairs and its cells' ranges.
// ---------------------------------------------------------------------------
struct FinishArgs {
  GridSet gs;
  const GridRun* run;
  const uint32_t* keys;     // [records] sorted by segment, in object order within one
  const uint32_t* vals;
  SegCode code;
  const SegEntry* list;     // [list_cap + 1]
  uint32_t list_cap;
  uint32_t* gaps;           // [3 * gap_cap] (first segment, end segment, pair): the longest stretches of empty segments
  uint32_t gap_cap;
  Control* ctl;
};
constexpr int kSegCells = 256;          // cells of the widest segment

// Who writes the ranges of a stretch of empty segments, by about its cells: the
// wave of the segment before it up to kGapWave, one workgroup up to kGapBlock,
// and all workgroups of the last kernel beyond.  (Only the last kind is listed
// with an atomic add on one counter: those cost 14 ns each, one after another.)
constexpr uint32_t kGapWave = 4096, kGapBlock = 65536;
GB_DEV uint32_t gap_segs(const SegCode& c, uint32_t cells) { return cells >> (c.wx + c.wy); }

// A segment's place: its grid's outputs, its first cell and its cell count.
struct SegPlace {
  uint32_t* cells;
  uint32_t* objs;
  uint32_t* ranges;
  uint64_t pair_base;
  uint32_t cell0, ncell;
  uint32_t width;           // cells of one of its rows
};

// Grid of segment seg (largest g with seg_base[g] <= seg among grids that have
// cells, and every grid has some): one whole wave, 64 probes per level.
GB_DEV uint32_t grid_of_seg_wave(const GridSet& s, uint32_t seg) {
  uint32_t lo = 0, end = s.ngrids;
  const uint32_t lane = lane_id();
  while (end - lo > 1) {
    const uint32_t step = (end - lo + kWave - 1) / kWave;
    const uint32_t g = lo + lane * step;
    const bool le = g < end && s.table[g].seg_base <= seg;
    const uint32_t c = static_cast<uint32_t>(__popcll(ballot(le)));
    lo += (c - 1) * step;
    end = lo + step < end ? lo + step : end;
  }
  return lo;
}

// First cell of local segment ls of a grid, which is its cell count when ls is
// the grid's segment count.
GB_DEV uint32_t seg_first_cell(const GridDev& G, uint32_t ls, uint32_t& xi, uint32_t& yi) {
  const uint32_t nsxy = G.nsx * G.nsy;
  const uint32_t z = ls / nsxy;
  const uint32_t r = ls - z * nsxy;
  yi = r / G.nsx;
  xi = r - yi * G.nsx;
  return xi * G.sx + G.res[0] * (yi * G.sy + G.res[1] * z);
}

template <bool Batched>
GB_DEV SegPlace seg_place(const FinishArgs& a, uint32_t seg) {
  const uint32_t g = Batched ? __builtin_amdgcn_readfirstlane(grid_of_seg_wave(a.gs, seg)) : 0u;
  const GridDev& G = grid_at<Batched>(a.gs, g);
  SegPlace p;
  p.cells = G.out_cells;
  p.objs = G.out_objs;
  p.ranges = G.out_ranges;
  p.pair_base = Batched ? a.run[g].pair_base : 0;
  uint32_t xi, yi;
  p.cell0 = seg_first_cell(G, seg - G.seg_base, xi, yi);
  const uint32_t w = G.res[0] - xi * G.sx, h = G.res[1] - yi * G.sy;
  p.width = w < G.sx ? w : G.sx;
  p.ncell = p.width * (h < G.sy ? h : G.sy);
  return p;
}

// The ranges of the empty segments [s0, s1): every cell begins and ends at pair
// p.  Written by `threads` threads of which this is thread `t`.
template <bool Batched>
GB_DEV void write_gap(const FinishArgs& a, uint32_t s0, uint32_t s1, uint32_t p, uint64_t t, uint64_t threads) {
  uint32_t g = Batched ? __builtin_amdgcn_readfirstlane(grid_of_seg_wave(a.gs, s0)) : 0u;
  while (true) {
    const GridDev& G = grid_at<Batched>(a.gs, g);
    const uint32_t gend = Batched && g + 1 < a.gs.ngrids ? a.gs.table[g + 1].seg_base : a.code.nsegs;
    const uint32_t e = s1 < gend ? s1 : gend;
    uint32_t xi, yi;
    const uint64_t c0 = seg_first_cell(G, s0 - G.seg_base, xi, yi);
    const uint64_t c1 = e == gend ? static_cast<uint64_t>(G.res[0]) * G.res[1] * G.res[2]
                                  : seg_first_cell(G, e - G.seg_base, xi, yi);
    const uint32_t v = p - static_cast<uint32_t>(Batched ? a.run[g].pair_base : 0);
    uint32_t* r = G.out_ranges;
    if ((reinterpret_cast<uintptr_t>(r) & 7u) == 0) {
      uint2* r2 = reinterpret_cast<uint2*>(r);
      for (uint64_t c = c0 + t; c < c1; c += threads) r2[c] = make_uint2(v, v);
    } else {
      for (uint64_t i = 2 * c0 + t; i < 2 * c1; i += threads) r[i] = v;
    }
    if (s1 <= gend) break;
    s0 = gend;
    ++g;
  }
}

// One wave: a stretch too long for one workgroup, listed for all of them.
GB_DEV void list_gap(const FinishArgs& a, uint32_t s0, uint32_t s1, uint32_t p) {
  if (lane_id() != 0) return;
  const uint32_t at = atomicAdd(&a.ctl->ngaps, 1u);
  if (at >= a.gap_cap) {
    atomicOr(&a.ctl->error, kErrInternal);
    return;
  }
  a.gaps[3 * at] = s0;
  a.gaps[3 * at + 1] = s1;
  a.gaps[3 * at + 2] = p;
}

// A record as a segment's pairs see it: its cells inside the segment.
struct Rect {
  uint32_t x0, y0, mx, my;
};
GB_DEV uint32_t rect_code(const SegCode& c, uint32_t key, uint32_t val) {
  return (key & ((1u << c.ck) - 1u)) | ((val >> c.objbits) << c.ck);
}
GB_DEV Rect unpack_rect(const SegCode& c, uint32_t code) {
  const uint32_t xm = (1u << c.wx) - 1u, ym = (1u << c.wy) - 1u;
  Rect r;
  r.mx = (code & xm) + 1u;
  r.my = ((code >> c.wx) & ym) + 1u;
  r.x0 = (code >> (c.wx + c.wy)) & xm;
  r.y0 = (code >> (2 * c.wx + c.wy)) & ym;
  return r;
}

// A run of records walked 64 at a time by one wave: the first kHeld batches are
// loaded at once and stay in registers, so that the two walks over a segment's
// records wait for memory once; a longer run loads the rest as it goes.
struct RecordRun {
  static constexpr int kHeld = 4;
  const uint32_t* keys;
  const uint32_t* vals;
  uint32_t n;
  uint32_t key[kHeld], val[kHeld];
  GB_DEV RecordRun() {}
  GB_DEV RecordRun(const FinishArgs& a, uint32_t r0, uint32_t r1) : keys(a.keys + r0), vals(a.vals + r0), n(r1 - r0) {
    const uint32_t lane = lane_id();
#pragma unroll
    for (int b = 0; b < kHeld; ++b) {
      const uint32_t i = b * kWave + lane;
      key[b] = i < n ? keys[i] : 0u;
      val[b] = i < n ? vals[i] : 0u;
    }
  }
  GB_DEV void batch(uint32_t b, uint32_t& k, uint32_t& v) const {
    if (b < static_cast<uint32_t>(kHeld)) {  // (b is uniform: scalar branches)
      k = key[0];
      v = val[0];
#pragma unroll
      for (int h = 1; h < kHeld; ++h)
        if (b == static_cast<uint32_t>(h)) {
          k = key[h];
          v = val[h];
        }
    } else {
      const uint32_t i = b * kWave + lane_id();
      k = i < n ? keys[i] : 0u;
      v = i < n ? vals[i] : 0u;
    }
  }
};

// Coverage counts of a run of records, one wave: s_diff[c] gains one where a
// row of a record starts and loses one past its end.
template <bool Rows>
GB_DEV void count_records(const FinishArgs& a, const RecordRun& run, uint32_t width, uint32_t* s_diff) {
  for (uint32_t b = 0; b * kWave < run.n; ++b) {
    uint32_t key, val;
    run.batch(b, key, val);
    if (b * kWave + lane_id() < run.n) {
      const Rect q = unpack_rect(a.code, rect_code(a.code, key, val));
      uint32_t c = q.x0 + (Rows ? __umul24(q.y0, width) : 0u);
      for (uint32_t y = 0; y < (Rows ? q.my : 1u); ++y) {
        atomicAdd(&s_diff[c], 1u);
        atomicSub(&s_diff[c + q.mx], 1u);
        c += width;
      }
    }
  }
}

// A wave's LDS for placing pairs.
constexpr uint32_t kPlaceSlots = 1024;        // pairs of a window
template <int Cells>
struct PlaceLds {
  uint64_t cover[Cells + 1];                  // each cell's records of the batch, as bits
  uint2 rec[kWave];                           // the batch's records: first slot << 16 | code, object
  uint32_t cur[Cells];                        // each cell's pairs before the batch
  uint32_t bits[kPlaceSlots / 32];            // slots where a record starts
};

// Places the pairs of a run of records in record order, one wave, 64 records at
// a time.  A record flips its bit where a row of its cells starts and past its
// end; the running exclusive-or over the cells is then each cell's set of
// records.  The batch's pairs are slots, 64 of them at a time: a record sets the
// bit of its first slot, a slot's owner is the number of bits up to it, and a
// pair's rank in its cell is the cell's pairs before the batch plus the records
// of its set before its owner.  So LDS sees two atomics a record, none a pair.
// cur[k]: pairs before the run in cell C * lane + k (C = Cells / 64).
// put(in, pos, d, obj): pair at position pos, cell d; nothing unless `in`.
template <bool Rows, int Cells, class Put>
GB_DEV void place_records(const FinishArgs& a, const RecordRun& run, uint32_t width, uint32_t (&cur)[Cells / kWave],
                          PlaceLds<Cells>& s, Put put) {
  constexpr int C = Cells / kWave;
  const uint32_t lane = lane_id();
  const uint32_t omask = a.code.objbits < 32 ? (1u << a.code.objbits) - 1u : 0xFFFFFFFFu;
  const uint64_t bit = uint64_t{1} << lane;
  for (uint32_t bt = 0; bt * kWave < run.n; ++bt) {
    uint32_t key, val;
    run.batch(bt, key, val);
    const bool live = bt * kWave + lane < run.n;
    const uint32_t code = rect_code(a.code, key, val);
    const Rect q0 = unpack_rect(a.code, code);
    const uint32_t cnt = live ? (Rows ? __umul24(q0.mx, q0.my) : q0.mx) : 0u;
    const uint32_t incl = wave_inclusive(cnt, OpAdd{});
    const uint32_t excl = incl - cnt;
    const uint32_t total = wave_readlane(incl, kWave - 1);
    s.rec[lane] = make_uint2((excl << 16) | code, val & omask);  // excl < 64 * 256
#pragma unroll
    for (int k = 0; k < C; ++k) s.cover[k * kWave + lane] = 0;
    if (lane < kPlaceSlots / 32) s.bits[lane] = 0;
    wave_sync();
    if (live) {
      uint32_t c = q0.x0 + (Rows ? __umul24(q0.y0, width) : 0u);
      for (uint32_t y = 0; y < (Rows ? q0.my : 1u); ++y) {
        atomicXor(reinterpret_cast<unsigned long long*>(&s.cover[c]), static_cast<unsigned long long>(bit));
        atomicXor(reinterpret_cast<unsigned long long*>(&s.cover[c + q0.mx]), static_cast<unsigned long long>(bit));
        c += width;
      }
      if (excl < kPlaceSlots) atomicOr(&s.bits[excl >> 5], 1u << (excl & 31u));
    }
    wave_sync();
    {
      uint64_t t[C];
#pragma unroll
      for (int k = 0; k < C; ++k) t[k] = s.cover[C * lane + k] ^ (k ? t[k > 0 ? k - 1 : 0] : 0u);
      const uint32_t lo = static_cast<uint32_t>(t[C - 1]), hi = static_cast<uint32_t>(t[C - 1] >> 32);
      const uint64_t before = (static_cast<uint64_t>(wave_inclusive(hi, OpXor{}) ^ hi) << 32) | (wave_inclusive(lo, OpXor{}) ^ lo);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        t[k] ^= before;
        s.cover[C * lane + k] = t[k];
        s.cur[C * lane + k] = cur[k];
        cur[k] += static_cast<uint32_t>(__builtin_popcountll(t[k]));
      }
    }
    wave_sync();
    for (uint32_t wb = 0; wb < total; wb += kPlaceSlots) {
      const uint32_t n = total - wb < kPlaceSlots ? total - wb : kPlaceSlots;
      uint32_t first = 0;  // records that start before the chunk
      if (wb) {            // a batch of more than kPlaceSlots pairs: the next window's bits
        if (lane < kPlaceSlots / 32) s.bits[lane] = 0;
        wave_sync();
        const uint32_t o = excl - wb;
        if (live && o < kPlaceSlots) atomicOr(&s.bits[o >> 5], 1u << (o & 31u));
        first = static_cast<uint32_t>(__builtin_popcountll(ballot(live && excl < wb)));
        wave_sync();
      }
      for (uint32_t c = 0; c < n; c += kWave) {
        const uint32_t hlo = __builtin_amdgcn_readfirstlane(s.bits[c / 32]);
        const uint32_t hhi = __builtin_amdgcn_readfirstlane(s.bits[c / 32 + 1]);
        const uint64_t heads = (static_cast<uint64_t>(hhi) << 32) | hlo;
        const uint32_t owner = first - 1u + (hlo & 1u) + mbcnt(heads >> 1);  // bits at or below the lane's
        first += static_cast<uint32_t>(__builtin_popcountll(heads));
        const uint2 rec = s.rec[owner & 63u];
        const uint32_t slot = c + lane;
        const uint32_t rid = wb + slot - (rec.x >> 16);
        const Rect q = unpack_rect(a.code, rec.x & 0xFFFFu);
        uint32_t d;
        if constexpr (Rows) {
          // rid / mx by a reciprocal: rid + 0.5 is at least 0.5 / mx >= 1/512 away
          // from a multiple of mx, far more than the product's rounding
          const uint32_t ry = static_cast<uint32_t>((static_cast<float>(rid) + 0.5f) *
                                                    __builtin_amdgcn_rcpf(static_cast<float>(q.mx)));
          d = __umul24(q.y0 + ry, width) + q.x0 + (rid - __umul24(ry, q.mx));
        } else {
          d = q.x0 + rid;
        }
        const bool in = slot < n;
        d = in ? d : 0u;
        const uint64_t m = s.cover[d] & ((uint64_t{1} << (owner & 63u)) - 1u);
        put(in, s.cur[d] + static_cast<uint32_t>(__builtin_popcountll(m)), d, rec.y);
      }
    }
    wave_sync();
  }
}

// Four words at an address that need only be aligned to one.
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
GB_DEV void store4(uint32_t* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  u32x4_a4 v = {a, b, c, d};
  *reinterpret_cast<u32x4_a4*>(p) = v;
}

// Staged pairs [0, n) stored in order by `threads` threads, four per thread and turn.
GB_DEV void store_staged(uint32_t* cells, uint32_t* objs, const uint32_t* s_obj, const uint8_t* s_d, uint32_t cell0,
                         uint32_t n, uint32_t t, uint32_t threads) {
  for (uint32_t i = 4 * t; i < n; i += 4 * threads) {
    const uint4 o = *reinterpret_cast<const uint4*>(s_obj + i);
    const uint32_t d = *reinterpret_cast<const uint32_t*>(s_d + i);
    const uint32_t c[4] = {cell0 + (d & 255u), cell0 + ((d >> 8) & 255u), cell0 + ((d >> 16) & 255u), cell0 + (d >> 24)};
    if (i + 4 <= n) {
      store4(cells + i, c[0], c[1], c[2], c[3]);
      store4(objs + i, o.x, o.y, o.z, o.w);
    } else {
      const uint32_t m = n - i;
      cells[i] = c[0];
      objs[i] = o.x;
      if (m > 1) {
        cells[i + 1] = c[1];
        objs[i + 1] = o.y;
      }
      if (m > 2) {
        cells[i + 2] = c[2];
        objs[i + 2] = o.z;
      }
    }
  }
}

// One wave per listed segment of at most Cap pairs: counts, ranges, pairs.  The
// pairs are staged in LDS, so that cells and objects are stored in order
// (stored where their ranks put them, 64 scattered words at a time, the kernel
// took three times as long).  A short stretch of empty segments after the
// segment is its wave's too.

// A wave's LDS for one segment.
template <uint32_t Cap, int Cells>
struct FinishLds {
  PlaceLds<Cells> place;
  alignas(16) uint32_t obj[Cap + 4];    // the coverage differences first, then the staged pairs
  alignas(16) uint8_t d[Cap + 4];
};

// One list entry, one wave.
template <uint32_t Cap, int Cells, bool Batched, bool Rows>
GB_DEV void finish_segment(const FinishArgs& a, const SegEntry& e0, const SegEntry& e1, const RecordRun& run,
                           FinishLds<Cap, Cells>& lds) {
  constexpr int C = Cells / kWave;  // cells per lane
  static_assert(Cap % 4 == 0 && Cap > static_cast<uint32_t>(Cells), "differences fit the staging");
  const uint32_t lane = lane_id();
  const uint32_t seg = e0.seg, p0 = e0.pair, seg1 = e1.seg, p1 = e1.pair;
  if (seg1 - seg - 1 != 0 && seg1 - seg - 1 <= gap_segs(a.code, kGapWave)) write_gap<Batched>(a, seg + 1, seg1, p1, lane, kWave);
  const uint32_t n = p1 - p0;
  if (n > Cap) return;  // a workgroup's
  const SegPlace pl = seg_place<Batched>(a, seg);
  uint32_t* diff = lds.obj;
#pragma unroll
  for (int k = 0; k < C; ++k) diff[k * kWave + lane] = 0;
  if (lane == 0) diff[Cells] = 0;
  wave_sync();
  count_records<Rows>(a, run, pl.width, diff);
  wave_sync();
  // coverage -> counts -> first pairs, C consecutive cells per lane
  uint32_t cur[C];
  {
    uint32_t v[C];
#pragma unroll
    for (int k = 0; k < C; ++k) v[k] = diff[C * lane + k] + (k ? v[k > 0 ? k - 1 : 0] : 0u);
    const uint32_t ci = wave_inclusive(v[C - 1], OpAdd{}) - v[C - 1];  // (differences wrap; the sums do not)
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
      v[k] += ci;
      s += v[k];
    }
    uint32_t e = wave_inclusive(s, OpAdd{}) - s;
    uint32_t rg[2 * C];
    const uint32_t lp32 = p0 - static_cast<uint32_t>(pl.pair_base);  // the segment's first pair in its grid's lists
#pragma unroll
    for (int k = 0; k < C; ++k) {
      cur[k] = e;
      rg[2 * k] = lp32 + e;
      e += v[k];
      rg[2 * k + 1] = lp32 + e;
    }
    uint32_t* out = pl.ranges + 2 * (static_cast<uint64_t>(pl.cell0) + C * lane);
    if (C * lane + C <= pl.ncell) {
      if constexpr (C == 1) {
        out[0] = rg[0];
        out[1] = rg[1];
      } else {
#pragma unroll
        for (int k = 0; k < C; k += 2) store4(out + 2 * k, rg[2 * k], rg[2 * k + 1], rg[2 * k + 2], rg[2 * k + 3]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < C; ++k)
        if (C * lane + k < pl.ncell) {
          out[2 * k] = rg[2 * k];
          out[2 * k + 1] = rg[2 * k + 1];
        }
    }
  }
  wave_sync();
  const uint64_t lp = p0 - pl.pair_base;
  uint32_t* so = lds.obj;
  uint8_t* sd = lds.d;
  place_records<Rows>(a, run, pl.width, cur, lds.place, [&](bool in, uint32_t pos, uint32_t d, uint32_t obj) {
    const uint32_t p = in ? pos : Cap;
    so[p] = obj;
    sd[p] = static_cast<uint8_t>(d);
  });
  store_staged(pl.cells + lp, pl.objs + lp, so, sd, pl.cell0, n, lane, kWave);
}

// One-wave workgroups: a long segment holds up one wave's LDS and nothing else.
// (A persistent grid with a fixed stride took a third longer: the dense segments
// of a scene lie together.  Claims from a counter would cost 14 ns each.)  A
// wave takes kFinishRun consecutive list entries and loads the next one's
// records while it works on one.
constexpr uint32_t kFinishRun = 2;
template <uint32_t Cap, int Cells, bool Batched, bool Rows>
__global__ __launch_bounds__(kWave, 4) void finish_kernel(FinishArgs a) {
  __shared__ FinishLds<Cap, Cells> s_lds;
  const uint32_t j0 = blockIdx.x * kFinishRun, lane = lane_id();
  // entries j0 .. j0 + kFinishRun, one per lane (what lies past the list's end is not used)
  const SegEntry mine = a.list[j0 + lane < a.list_cap ? j0 + lane : a.list_cap];
  if (build_failed(a.ctl)) return;
  const uint32_t nlist = a.ctl->nlist;
  auto entry = [&](uint32_t i) {
    SegEntry e;
    e.seg = wave_readlane(mine.seg, static_cast<int>(i));
    e.rec = wave_readlane(mine.rec, static_cast<int>(i));
    e.pair = wave_readlane(mine.pair, static_cast<int>(i));
    e.pad = 0;
    return e;
  };
  if (j0 == 0) {
    // the empty segments before the first listed one
    const uint32_t s1 = nlist ? entry(0).seg : a.code.nsegs;
    if (s1 > 0 && s1 <= gap_segs(a.code, kGapWave)) write_gap<Batched>(a, 0, s1, 0, lane, kWave);
    else if (s1 > gap_segs(a.code, kGapBlock)) list_gap(a, 0, s1, 0);
  }
  if (j0 >= nlist) return;
  const uint32_t m = nlist - j0 < kFinishRun ? nlist - j0 : kFinishRun;
  SegEntry e0 = entry(0), e1 = entry(1);
  RecordRun run(a, e0.rec, e1.rec);
  for (uint32_t i = 0;; ++i) {
    const bool more = i + 1 < m;
    const SegEntry e2 = entry(more ? i + 2 : i + 1);
    const RecordRun next(a, e1.rec, e2.rec);  // (none when there is no next entry)
    if (e1.seg - e0.seg - 1 > gap_segs(a.code, kGapBlock)) list_gap(a, e0.seg + 1, e1.seg, e1.pair);
    finish_segment<Cap, Cells, Batched, Rows>(a, e0, e1, run, s_lds);
    if (!more) break;
    e0 = e1;
    e1 = e2;
    run = next;
    wave_sync();
  }
}

// What finish_kernel leaves: segments with more than `least` and at most `most`
// pairs, one workgroup each, and longer stretches of empty segments.  Workgroup
// b looks at every gridDim-th list entry from b, 64 at a time.  The records of
// a segment are split into one run per wave; each wave counts its own run, the
// counts are scanned over (cell, wave), and each wave places its run from its
// own cursors.  Mid: this launch takes the stretches of up to kGapBlock cells;
// Last: it takes the listed ones.
template <int Block, uint32_t Cap, bool Mid, bool Last, bool Batched, bool Rows>
__global__ __launch_bounds__(Block) void finish_big_kernel(FinishArgs a, uint32_t least, uint32_t most) {
  constexpr int W = Block / kWave;
  constexpr int kDiff = kSegCells + 4;
  static_assert(Cap % 4 == 0 && Cap >= static_cast<uint32_t>(W * kDiff), "the waves' differences fit the staging");
  __shared__ PlaceLds<kSegCells> s_place[W];
  __shared__ __align__(16) uint32_t s_obj[Cap + 4];   // the waves' coverage differences first, then the staged pairs
  __shared__ __align__(16) uint8_t s_d[Cap + 4];
  __shared__ uint32_t s_wtot[W];
  if (build_failed(a.ctl)) return;
  const uint32_t nlist = a.ctl->nlist;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(tid / kWave);
  uint32_t* const diff = s_obj + w * kDiff;
  if constexpr (Last) {
    const uint32_t ngaps = a.ctl->ngaps;
    for (uint32_t i = 0; i < ngaps; ++i)
      write_gap<Batched>(a, a.gaps[3 * i], a.gaps[3 * i + 1], a.gaps[3 * i + 2],
                         static_cast<uint64_t>(blockIdx.x) * Block + tid, static_cast<uint64_t>(gridDim.x) * Block);
  }
  if (Mid && blockIdx.x == 0) {
    const uint32_t s1 = nlist ? a.list[0].seg : a.code.nsegs;
    if (s1 > gap_segs(a.code, kGapWave) && s1 <= gap_segs(a.code, kGapBlock)) write_gap<Batched>(a, 0, s1, 0, tid, Block);
  }
  for (uint64_t j0 = blockIdx.x; j0 < nlist; j0 += static_cast<uint64_t>(gridDim.x) * kWave) {
   // every wave finds the same entries
   const uint64_t jl = j0 + static_cast<uint64_t>(lane) * gridDim.x;
   bool mine = false;
   if (jl < nlist) {
     const SegEntry e0 = a.list[jl], e1 = a.list[jl + 1];
     const uint32_t n = e1.pair - e0.pair, gap = e1.seg - e0.seg - 1;
     mine = (n > least && n <= most) ||
            (Mid && gap > gap_segs(a.code, kGapWave) && gap <= gap_segs(a.code, kGapBlock));
   }
   uint64_t todo = ballot(mine);
   while (todo) {
    const uint32_t j = static_cast<uint32_t>(j0 + static_cast<uint64_t>(__builtin_ctzll(todo)) * gridDim.x);
    todo &= todo - 1;
    const SegEntry e0 = a.list[j], e1 = a.list[j + 1];
    const uint32_t r0 = e0.rec, r1 = e1.rec, p0 = e0.pair, n = e1.pair - p0;
    if constexpr (Mid) {
      const uint32_t gap = e1.seg - e0.seg - 1;
      if (gap > gap_segs(a.code, kGapWave) && gap <= gap_segs(a.code, kGapBlock))
        write_gap<Batched>(a, e0.seg + 1, e1.seg, e1.pair, tid, Block);
    }
    if (n <= least || n > most) continue;
    const SegPlace pl = seg_place<Batched>(a, e0.seg);
    const uint64_t nr = r1 - r0;
    const uint64_t per = (nr + W * kWave - 1) / (W * kWave) * kWave;
    const uint32_t off0 = static_cast<uint32_t>(w * per < nr ? w * per : nr);
    const uint32_t off1 = static_cast<uint32_t>(off0 + per < nr ? off0 + per : nr);
    for (uint32_t c = lane; c < kDiff; c += kWave) diff[c] = 0;
    wave_sync();
    const RecordRun run(a, r0 + off0, r0 + off1);
    count_records<Rows>(a, run, pl.width, diff);
    wave_sync();
    {
      // the wave's coverage, four consecutive cells per lane
      uint32_t* cur = diff + 4 * lane;
      const uint32_t x0 = cur[0], x1 = x0 + cur[1], x2 = x1 + cur[2], x3 = x2 + cur[3];
      const uint32_t ci = wave_inclusive(x3, OpAdd{}) - x3;
      cur[0] = ci + x0;
      cur[1] = ci + x1;
      cur[2] = ci + x2;
      cur[3] = ci + x3;
    }
    __syncthreads();
    uint32_t cnt = 0;
    if (tid < kSegCells) {
      for (int v = 0; v < W; ++v) cnt += s_obj[v * kDiff + tid];
    }
    uint32_t tot;
    const uint32_t begin = block_exclusive_sum<Block>(cnt, s_wtot, tot);
    const uint64_t lp = p0 - pl.pair_base;
    if (tid < kSegCells) {
      uint32_t c = begin;
      for (int v = 0; v < W; ++v) {
        const uint32_t x = s_obj[v * kDiff + tid];
        s_obj[v * kDiff + tid] = c;
        c += x;
      }
      if (tid < pl.ncell) {
        uint32_t* rg = pl.ranges + 2 * (static_cast<uint64_t>(pl.cell0) + tid);
        rg[0] = static_cast<uint32_t>(lp) + begin;
        rg[1] = static_cast<uint32_t>(lp) + begin + cnt;
      }
    }
    __syncthreads();
    uint32_t cur[kSegCells / kWave];
#pragma unroll
    for (int k = 0; k < kSegCells / kWave; ++k) cur[k] = diff[kSegCells / kWave * lane + k];
    __syncthreads();
    uint32_t* oc = pl.cells + lp;
    uint32_t* oo = pl.objs + lp;
    if (n <= Cap) {
      place_records<Rows>(a, run, pl.width, cur, s_place[w], [&](bool in, uint32_t pos, uint32_t d, uint32_t obj) {
        const uint32_t p = in ? pos : Cap;
        s_obj[p] = obj;
        s_d[p] = static_cast<uint8_t>(d);
      });
      __syncthreads();
      store_staged(oc, oo, s_obj, s_d, pl.cell0, n, tid, Block);
    } else {
      place_records<Rows>(a, run, pl.width, cur, s_place[w], [&](bool in, uint32_t pos, uint32_t d, uint32_t obj) {
        if (in) {
          oc[pos] = pl.cell0 + d;
          oo[pos] = obj;
        }
      });
    }
    __syncthreads();
   }
  }
}

}  // namespace gb
