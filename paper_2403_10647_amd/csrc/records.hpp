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
// are never read again.  Segments of many pairs are cut into chunks of records,
// which workgroups take in turn, so that the work stays even where a scene crowds.
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
  const GridRun* run;       // batches resumed from their count: each grid's pair count, to check its outputs by (else null)
};

// A batch resumed from its count learns its outputs only then: whether some grid's
// are too small.  Every wave looks at all grids, so all of them come to the same
// answer by themselves: a flag that one workgroup raises while others read it would
// stop some waves of a workgroup and leave the rest to scan totals never written.
GB_DEV bool outputs_too_small(const GridSet& s, const GridRun* run) {
  bool over = false;
  for (uint32_t g = lane_id(); g < s.ngrids; g += kWave) over = over || run[g].npairs > s.table[g].cap_pairs;
  return ballot(over) != 0;
}

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
  if constexpr (Batched) {
    if (a.run && outputs_too_small(a.o.ex.gs, a.run)) {
      if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&a.o.ctl->cap_flag, 1u);  // for the kernels that follow
      return;
    }
  }
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

// Pairs above which a segment is left to workgroups: the kernel of the waves lasts
// as long as its longest, so four times the mean of the listed segments and a
// thousandth of the build's pairs (a wave each on most of the GPU), but no fewer
// than are worth a workgroup; a wave's staging is the other limit.  Builds, us, at
// 64 / 256 / 512 / 1000 pairs: 246K pairs in a corner 115 115 115 123; mesh of 4.3M,
// mean 150, 312 239 226 236; arch-like 54M, mean 260, 1487 1286 999 821.
constexpr uint32_t kCrowdLeast = 256;
GB_DEV uint32_t crowded_above(uint64_t npairs, uint32_t nlist) {
  const uint64_t a = 4 * npairs / nlist, b = npairs / 1024, c = a < b ? a : b;
  return static_cast<uint32_t>(c > kCrowdLeast ? c : kCrowdLeast);
}

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
            a.ctl->crowd = crowded_above(npairs, nheads);
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
constexpr int kSegCells = 256;          // cells of the widest segment

// What a segment's wave leaves is listed as tasks of about equal size, which the
// workgroups of the last kernels take in turn however the scene crowds them:
//  - a segment of more pairs than its wave stages, as chunks of its records (one
//    workgroup a segment took 3.4 ms for 3.6M pairs in 8 segments; by pairs, whose
//    work is equal by construction, that whole build is 204 us);
//  - a stretch of empty segments of more than kGapWave cells, in pieces of about
//    kGapTask (shorter ones are the wave's of the segment before).
// kChunkPairs: a chunk's least; a segment below twice as many is one chunk, whose
// pairs a workgroup stages.  At most kMaxChunks a segment (each reads the counts of
// those before it), so that chunks grow beyond 4M pairs in one segment.
constexpr uint32_t kGapWave = 4096, kGapTask = 16384;
constexpr uint32_t kChunkPairs = 2048, kMaxChunks = 2048;
constexpr uint32_t kGroupChunks = 32;   // chunks whose counts are also added up together
constexpr uint32_t kTaskLists = 64;     // most lists (adds to one counter cost 14 ns each, one after another)
constexpr uint32_t kTaskStride = 16;    // counters of the lists, one a 128-byte line
constexpr uint32_t kTaskGap = 1u << 31;     // a task entry's stretch of empty segments ...
constexpr uint32_t kTaskFirst = 0x7FFFFFFFu;  // ... after this list entry (kTaskFirst: before the first one)
GB_DEV uint32_t gap_segs(const SegCode& c, uint32_t cells) { return cells >> (c.wx + c.wy); }
GB_DEV uint32_t chunks_of(uint32_t pairs) {
  const uint32_t c = pairs / kChunkPairs;
  return c < 2 ? 1u : c < kMaxChunks ? c : kMaxChunks;
}
// Chunks take rows of per-cell counts by their segment's pairs: those of [p, p + n)
// are rows ceil(p / kChunkPairs) on, at most n / kChunkPairs of them, so no two
// segments share one.  The same holds for groups of kGroupChunks chunks, whose
// last one is the longer (a segment of fewer than two groups has none).
GB_DEV uint32_t row_of(uint32_t pair) { return pair / kChunkPairs + (pair % kChunkPairs ? 1u : 0u); }
GB_DEV uint32_t group_row_of(uint32_t pair) {
  constexpr uint32_t n = kChunkPairs * kGroupChunks;
  return pair / n + (pair % n ? 1u : 0u);
}
GB_DEV uint32_t row_cells(const SegCode& c) { return 1u << (c.wx + c.wy); }
GB_DEV uint32_t groups_of(uint32_t chunks) { return chunks < 2 * kGroupChunks ? 0u : chunks / kGroupChunks; }

// Tasks of one kind: entries of what they are of, in lists of so many entries each.
struct TaskLists {
  uint2* entry;             // [lists][cap] (list entry | kTaskGap, its first task in this list)
  uint64_t* n;              // [lists * kTaskStride] (zeroed) entries << 32 | tasks
  uint32_t cap;
};

struct FinishArgs {
  GridSet gs;
  const GridRun* run;
  const uint32_t* keys;     // [records] sorted by segment, in object order within one
  const uint32_t* vals;
  SegCode code;
  const SegEntry* list;     // [list_cap + 1]
  uint32_t list_cap;
  uint32_t task_lists;      // lists of each kind of tasks (a power of two)
  TaskLists once;           // segments of one chunk and empty stretches
  TaskLists several;        // segments of several chunks
  uint32_t* rows;           // [ceil(pairs / kChunkPairs)][row_cells] a chunk's pairs per cell (null: not counted beforehand)
  uint32_t* groups;         // [ceil(pairs / (kChunkPairs * kGroupChunks))][row_cells] the same of whole groups
  Control* ctl;
};

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

// One wave: what it leaves, listed as n tasks.
GB_DEV void list_tasks(const FinishArgs& a, const TaskLists& to, uint32_t what, uint32_t n) {
  if (lane_id() != 0) return;
  const uint32_t l = blockIdx.x & (a.task_lists - 1);
  const uint64_t at = atomicAdd(reinterpret_cast<unsigned long long*>(to.n + l * kTaskStride), (1ull << 32) | n);
  const uint32_t e = static_cast<uint32_t>(at >> 32);
  if (e < to.cap) to.entry[static_cast<uint64_t>(l) * to.cap + e] = make_uint2(what, static_cast<uint32_t>(at));
  else atomicOr(&a.ctl->error, kErrInternal);
}

// A stretch of `segs` empty segments: nothing, or listed when it is more than its wave's.
GB_DEV void list_gap(const FinishArgs& a, uint32_t what, uint32_t segs) {
  const uint32_t per = gap_segs(a.code, kGapTask);
  if (segs > gap_segs(a.code, kGapWave)) list_tasks(a, a.once, kTaskGap | what, segs / per + (segs % per ? 1u : 0u));
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

// List entry j, one wave.
template <uint32_t Cap, int Cells, bool Batched, bool Rows>
GB_DEV void finish_segment(const FinishArgs& a, uint32_t j, const SegEntry& e0, const SegEntry& e1, const RecordRun& run,
                           uint32_t crowd, FinishLds<Cap, Cells>& lds) {
  constexpr int C = Cells / kWave;  // cells per lane
  static_assert(Cap % 4 == 0 && Cap > static_cast<uint32_t>(Cells), "differences fit the staging");
  const uint32_t lane = lane_id();
  const uint32_t seg = e0.seg, p0 = e0.pair, seg1 = e1.seg, p1 = e1.pair;
  if (seg1 - seg - 1 != 0 && seg1 - seg - 1 <= gap_segs(a.code, kGapWave)) write_gap<Batched>(a, seg + 1, seg1, p1, lane, kWave);
  const uint32_t n = p1 - p0;
  if (n > crowd) {  // workgroups': listed, and its groups' counts cleared for them
    const uint32_t chunks = chunks_of(n);
    uint32_t* g = a.groups + static_cast<uint64_t>(group_row_of(p0)) * row_cells(a.code);
    for (uint32_t i = lane; i < groups_of(chunks) * row_cells(a.code); i += kWave) g[i] = 0;
    list_tasks(a, chunks > 1 ? a.several : a.once, j, chunks);
    return;
  }
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
  const uint32_t nlist = a.ctl->nlist, crowd = a.ctl->crowd < Cap ? a.ctl->crowd : Cap;
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
    else list_gap(a, kTaskFirst, s1);
  }
  if (j0 >= nlist) return;
  const uint32_t m = nlist - j0 < kFinishRun ? nlist - j0 : kFinishRun;
  SegEntry e0 = entry(0), e1 = entry(1);
  RecordRun run(a, e0.rec, e1.rec);
  for (uint32_t i = 0;; ++i) {
    const bool more = i + 1 < m;
    const SegEntry e2 = entry(more ? i + 2 : i + 1);
    const RecordRun next(a, e1.rec, e2.rec);  // (none when there is no next entry)
    list_gap(a, j0 + i, e1.seg - e0.seg - 1);
    finish_segment<Cap, Cells, Batched, Rows>(a, j0 + i, e0, e1, run, crowd, s_lds);
    if (!more) break;
    e0 = e1;
    e1 = e2;
    run = next;
    wave_sync();
  }
}

// The tasks of one kind, found by number: lane l holds list l's.
struct TaskMap {
  uint32_t entries, upto;   // the list's entries; tasks of this list and those before it
  uint32_t total;
};
GB_DEV TaskMap task_map(const FinishArgs& a, const TaskLists& of) {
  const uint32_t lane = lane_id();
  const uint64_t n = lane < a.task_lists ? of.n[lane * kTaskStride] : 0;
  TaskMap m;
  m.entries = static_cast<uint32_t>(n >> 32);
  m.upto = wave_inclusive(static_cast<uint32_t>(n), OpAdd{});
  m.total = wave_readlane(m.upto, kWave - 1);
  return m;
}

// Task t (below total): what it is of, and which of its tasks.  One whole wave;
// a list's entries are in the order of their first tasks (one add gave both).
GB_DEV uint32_t find_task(const TaskLists& of, const TaskMap& m, uint32_t t, uint32_t& part) {
  const uint32_t lane = lane_id();
  const uint32_t l = static_cast<uint32_t>(__popcll(ballot(m.upto <= t)));  // (below total: some list's upto exceeds t)
  if (l) t -= wave_readlane(m.upto, static_cast<int>(l - 1));
  uint32_t lo = 0, end = wave_readlane(m.entries, static_cast<int>(l));
  const uint2* e = of.entry + static_cast<uint64_t>(l) * of.cap;
  while (end - lo > 1) {
    const uint32_t step = (end - lo + kWave - 1) / kWave;
    const uint32_t g = lo + lane * step;
    const uint32_t c = static_cast<uint32_t>(__popcll(ballot(g < end && e[g].y <= t)));
    lo += (c - 1) * step;
    end = lo + step < end ? lo + step : end;
  }
  part = t - __builtin_amdgcn_readfirstlane(e[lo].y);
  return __builtin_amdgcn_readfirstlane(e[lo].x);
}

constexpr int kTaskBlock = 256;
constexpr int kTaskWaves = kTaskBlock / kWave;
constexpr uint32_t kTaskDiff = kSegCells + 4;   // a wave's coverage differences
constexpr uint32_t kTaskCap = 2 * kChunkPairs;  // pairs a workgroup stages
static_assert(kTaskBlock == kSegCells, "a thread per cell");

// A wave's run of records [r0, r1) (whole sixteens) of which there is one a wave.
GB_DEV RecordRun wave_run(const FinishArgs& a, uint32_t r0, uint32_t r1, uint32_t w) {
  const uint64_t nr = r1 - r0;
  const uint64_t per = (nr + kTaskWaves * 16 - 1) / (kTaskWaves * 16) * 16;
  const uint32_t off0 = static_cast<uint32_t>(w * per < nr ? w * per : nr);
  const uint32_t off1 = static_cast<uint32_t>(off0 + per < nr ? off0 + per : nr);
  return RecordRun(a, r0 + off0, r0 + off1);
}
GB_DEV void clear_diff(uint32_t* diff) {
  for (uint32_t c = lane_id(); c < kTaskDiff; c += kWave) diff[c] = 0;
  wave_sync();
}
// A wave's coverage differences made counts: diff[c] = its pairs in cell c.
GB_DEV void sum_diff(uint32_t* diff) {
  wave_sync();
  uint32_t* cur = diff + 4 * lane_id();  // four consecutive cells per lane
  const uint32_t x0 = cur[0], x1 = x0 + cur[1], x2 = x1 + cur[2], x3 = x2 + cur[3];
  const uint32_t ci = wave_inclusive(x3, OpAdd{}) - x3;
  cur[0] = ci + x0;
  cur[1] = ci + x1;
  cur[2] = ci + x2;
  cur[3] = ci + x3;
}

// Records [r0, r1) of a chunk, one run per wave, counted into the wave's diff.
// The caller's barrier follows before other waves' counts are read.
template <bool Rows>
GB_DEV RecordRun count_chunk(const FinishArgs& a, uint32_t r0, uint32_t r1, uint32_t width, uint32_t w, uint32_t* diff) {
  clear_diff(diff);
  const RecordRun run = wave_run(a, r0, r1, w);
  count_records<Rows>(a, run, width, diff);
  sum_diff(diff);
  return run;
}

// Any number of records, by the workgroup: pairs of this thread's cell.
template <bool Rows>
GB_DEV uint32_t count_cell(const FinishArgs& a, uint32_t r0, uint32_t r1, uint32_t width, uint32_t w, uint32_t* diffs) {
  constexpr uint32_t kStep = kTaskWaves * RecordRun::kHeld * kWave;  // loaded at once
  uint32_t* const diff = diffs + w * kTaskDiff;
  clear_diff(diff);
  for (uint32_t r = r0; r < r1; r += kStep) count_records<Rows>(a, wave_run(a, r, r1 - r < kStep ? r1 : r + kStep, w), width, diff);
  sum_diff(diff);
  __syncthreads();
  uint32_t n = 0;
#pragma unroll
  for (int v = 0; v < kTaskWaves; ++v) n += diffs[v * kTaskDiff + threadIdx.x];
  __syncthreads();
  return n;
}

// First record of chunk c of a segment's `chunks`, of records [r0, r1).
GB_DEV uint32_t chunk_first(uint32_t r0, uint32_t r1, uint32_t chunks, uint32_t c) {
  const uint64_t nr = r1 - r0, per = (nr + chunks - 1) / chunks, off = per * c;
  return r0 + static_cast<uint32_t>(off < nr ? off : nr);
}

// The pairs per cell of every chunk of the segments that have several, and of their
// groups.  (A kernel of its own: counted by the workgroups that place them, with a
// wait between, each row's release fence wrote back its XCD's L2, and 100k
// hairball-like triangles in a corner took 278 us against 144.)
template <bool Batched, bool Rows>
__global__ __launch_bounds__(kTaskBlock) void finish_count_kernel(FinishArgs a) {
  __shared__ uint32_t s_diff[kTaskWaves * kTaskDiff];
  if (build_failed(a.ctl)) return;
  const TaskMap map = task_map(a, a.several);
  const uint32_t tid = threadIdx.x;
  const uint32_t w = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (uint32_t t = blockIdx.x; t < map.total; t += gridDim.x) {
    uint32_t chunk;
    const uint32_t j = find_task(a.several, map, t, chunk);
    const SegEntry e0 = a.list[j], e1 = a.list[j + 1];
    const uint32_t chunks = chunks_of(e1.pair - e0.pair);
    const SegPlace pl = seg_place<Batched>(a, e0.seg);
    count_chunk<Rows>(a, chunk_first(e0.rec, e1.rec, chunks, chunk), chunk_first(e0.rec, e1.rec, chunks, chunk + 1), pl.width, w,
                      s_diff + w * kTaskDiff);
    __syncthreads();
    uint32_t n = 0;
#pragma unroll
    for (int v = 0; v < kTaskWaves; ++v) n += s_diff[v * kTaskDiff + tid];
    const uint32_t cells = row_cells(a.code);
    if (tid < cells) {
      a.rows[static_cast<uint64_t>(row_of(e0.pair) + chunk) * cells + tid] = n;
      const uint32_t groups = groups_of(chunks);
      if (groups && n) {
        const uint32_t g = chunk / kGroupChunks < groups ? chunk / kGroupChunks : groups - 1;
        atomicAdd(a.groups + static_cast<uint64_t>(group_row_of(e0.pair) + g) * cells + tid, n);
      }
    }
    __syncthreads();
  }
}

// The tasks: pieces of long stretches of empty segments, and the chunks of crowded
// segments, each placed from where the chunks before it end in every cell.  A chunk
// whose pairs exceed the staging (long records, or a segment of kMaxChunks) goes in
// rounds of its records.  256 threads, so that four workgroups, at different phases,
// share a CU's LDS.  Bound by the latency of those phases and, where thousands of
// objects share a cell, by LDS atomics on the same words: 45M pairs crowded into an
// eighth of their box 303 us (1024-thread workgroups, one a segment: 358), into a
// millionth 347 (10883); mesh of 4.3M pairs 32 (57 and 34 for its larger segments).
template <bool Batched, bool Rows>
__global__ __launch_bounds__(kTaskBlock) void finish_tasks_kernel(FinishArgs a) {
  __shared__ PlaceLds<kSegCells> s_place[kTaskWaves];
  __shared__ __align__(16) uint32_t s_obj[kTaskCap + 4];   // the waves' coverage first, then the staged pairs
  __shared__ __align__(16) uint8_t s_d[kTaskCap + 4];
  __shared__ uint32_t s_at[kSegCells];                     // a cell's first pair of the round less its first slot
  __shared__ uint32_t s_wtot[kTaskWaves];
  static_assert(kTaskCap % 4 == 0 && kTaskCap >= kTaskWaves * kTaskDiff, "the waves' coverage fits the staging");
  if (build_failed(a.ctl)) return;
  const TaskMap once = task_map(a, a.once), several = task_map(a, a.several);
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(tid / kWave);
  uint32_t* const diff = s_obj + w * kTaskDiff;
  for (uint32_t t = blockIdx.x; t < once.total + several.total; t += gridDim.x) {
    uint32_t part;
    const uint32_t what = t < once.total ? find_task(a.once, once, t, part) : find_task(a.several, several, t - once.total, part);
    if (what & kTaskGap) {
      const uint32_t j = what & ~kTaskGap, nlist = a.ctl->nlist;
      const uint32_t s0 = j == kTaskFirst ? 0u : a.list[j].seg + 1;
      const uint32_t next = j == kTaskFirst ? 0u : j + 1;
      const uint32_t s1 = nlist ? a.list[next].seg : a.code.nsegs;  // (entry nlist closes the list)
      const uint32_t p = j == kTaskFirst ? 0u : a.list[next].pair;
      const uint32_t per = gap_segs(a.code, kGapTask);
      const uint32_t b = s0 + part * per;
      write_gap<Batched>(a, b, s1 - b < per ? s1 : b + per, p, tid, kTaskBlock);
      continue;
    }
    const SegEntry e0 = a.list[what], e1 = a.list[what + 1];
    const uint32_t p0 = e0.pair, n = e1.pair - p0;
    const uint32_t chunks = chunks_of(n);
    const SegPlace pl = seg_place<Batched>(a, e0.seg);
    const uint64_t lp = p0 - pl.pair_base;
    uint32_t* const ranges = pl.ranges + 2 * (static_cast<uint64_t>(pl.cell0) + tid);
    uint32_t r0 = chunk_first(e0.rec, e1.rec, chunks, part);
    const uint32_t r1 = chunk_first(e0.rec, e1.rec, chunks, part + 1);
    uint32_t rounds = 1, at = 0;   // at: the cell's next pair in the segment
    if (chunks > 1) {
      // the cell's pairs in this chunk, in those before it, and in all of them
      const uint32_t cells = row_cells(a.code), groups = groups_of(chunks);
      const uint32_t mine = groups == 0 ? 0u : part / kGroupChunks < groups ? part / kGroupChunks : groups - 1;
      uint32_t before = 0, total = 0, own = 0;
      if (!a.rows) {  // a small build: no kernel has counted the chunks
        before = count_cell<Rows>(a, e0.rec, r0, pl.width, w, s_obj);
        own = count_cell<Rows>(a, r0, r1, pl.width, w, s_obj);
        total = before + own + count_cell<Rows>(a, r1, e1.rec, pl.width, w, s_obj);
      } else if (tid < cells) {
        const uint32_t* row = a.rows + static_cast<uint64_t>(row_of(p0)) * cells + tid;
        own = row[static_cast<uint64_t>(part) * cells];
        if (groups) {
          const uint32_t* g = a.groups + static_cast<uint64_t>(group_row_of(p0)) * cells + tid;
#pragma unroll 8
          for (uint32_t i = 0; i < groups; ++i) {
            const uint32_t x = g[static_cast<uint64_t>(i) * cells];
            total += x;
            before += i < mine ? x : 0u;
          }
#pragma unroll 8
          for (uint32_t i = mine * kGroupChunks; i < part; ++i) before += row[static_cast<uint64_t>(i) * cells];
        } else {
#pragma unroll 8
          for (uint32_t i = 0; i < chunks; ++i) {
            const uint32_t x = row[static_cast<uint64_t>(i) * cells];
            total += x;
            before += i < part ? x : 0u;
          }
        }
      }
      uint32_t sum;
      const uint32_t begin = block_exclusive_sum<kTaskBlock>(total, s_wtot, sum);
      if (part == 0 && tid < pl.ncell) {
        ranges[0] = static_cast<uint32_t>(lp) + begin;
        ranges[1] = static_cast<uint32_t>(lp) + begin + total;
      }
      at = begin + before;
      block_exclusive_sum<kTaskBlock>(own, s_wtot, sum);
      if (sum > kTaskCap) rounds = (sum + kChunkPairs - 1) / kChunkPairs;
    }
    const uint32_t per = static_cast<uint32_t>((static_cast<uint64_t>(r1 - r0) + rounds - 1) / rounds);
    uint32_t* const oc = pl.cells + lp;
    uint32_t* const oo = pl.objs + lp;
    do {  // (a chunk of no records is one empty round)
      const uint32_t re = r1 - r0 < per ? r1 : r0 + per;
      const RecordRun run = count_chunk<Rows>(a, r0, re, pl.width, w, diff);
      __syncthreads();
      uint32_t cnt = 0;
#pragma unroll
      for (int v = 0; v < kTaskWaves; ++v) cnt += s_obj[v * kTaskDiff + tid];
      uint32_t m;
      const uint32_t begin = block_exclusive_sum<kTaskBlock>(cnt, s_wtot, m);
      const bool staged = m <= kTaskCap;
      uint32_t c = staged ? begin : at;
#pragma unroll
      for (int v = 0; v < kTaskWaves; ++v) {
        const uint32_t x = s_obj[v * kTaskDiff + tid];
        s_obj[v * kTaskDiff + tid] = c;
        c += x;
      }
      if (chunks == 1 && tid < pl.ncell) {
        ranges[0] = static_cast<uint32_t>(lp) + begin;
        ranges[1] = static_cast<uint32_t>(lp) + begin + cnt;
      }
      s_at[tid] = at - begin;
      at += cnt;
      __syncthreads();
      uint32_t cur[kSegCells / kWave];
#pragma unroll
      for (int k = 0; k < kSegCells / kWave; ++k) cur[k] = diff[kSegCells / kWave * lane + k];
      __syncthreads();
      if (staged) {
        place_records<Rows>(a, run, pl.width, cur, s_place[w], [&](bool in, uint32_t pos, uint32_t d, uint32_t obj) {
          const uint32_t p = in ? pos : kTaskCap;
          s_obj[p] = obj;
          s_d[p] = static_cast<uint8_t>(d);
        });
        __syncthreads();
        if (chunks == 1) {
          store_staged(oc, oo, s_obj, s_d, pl.cell0, n, tid, kTaskBlock);
        } else {
          for (uint32_t i = tid; i < m; i += kTaskBlock) {
            const uint32_t d = s_d[i];
            const uint32_t p = s_at[d] + i;
            oc[p] = pl.cell0 + d;
            oo[p] = s_obj[i];
          }
        }
      } else {
        place_records<Rows>(a, run, pl.width, cur, s_place[w], [&](bool in, uint32_t pos, uint32_t d, uint32_t obj) {
          if (in) {
            oc[pos] = pl.cell0 + d;
            oo[pos] = obj;
          }
        });
      }
      __syncthreads();
      r0 = re;
    } while (r0 < r1);
  }
}

}  // namespace gb
