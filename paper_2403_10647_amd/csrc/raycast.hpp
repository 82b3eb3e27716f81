// Ray casting over a built grid, the use the grid is made for (Introduction;
// Related Work): each ray's closest triangle, found by walking the cells the
// ray crosses and testing the objects each cell lists (objs[ranges[2c] ..
// ranges[2c + 1])).
//
// Contract (the same result as testing every triangle):
//  * a ray is o + t d, t in [t0, t1]: [0, tmax] clipped to the grid box by
//    the slab test; only hits inside the box count;
//  * the hit test is Moller and Trumbore's in a fixed order of FP32
//    operations (no contraction, IEEE division); a grazing ray
//    (det^2 < 1e-8 |e1|^2 |e2|^2 |d|^2) or a degenerate triangle misses; edges
//    count;
//  * the result is the smallest hit t, then the smallest object id; no hit:
//    t = +inf, id 0xFFFFFFFF.
// The walk goes slab by slab along the ray's dominant axis; in each slab it
// visits every cell the ray can touch there, with the slab's t-interval and
// the cross-section widened by 1/32 of a cell, so rounding in the walk never
// skips a cell the ray passes through.  It stops after the slab in which the
// best hit lies (by the same margin) before the slab's far face: every later
// cell lies beyond that hit.  (Cells after the last one needed may be tested too:
// every hit counts wherever it is found.)
#pragma once

#include "grid.hpp"
#include "walk.hpp"

namespace gb {

constexpr float kGrazingRay = 1e-8f;
constexpr float kWalkPad = 1.0f / 32.0f;   // cells

GB_DEV float dot3r(const float a[3], const float b[3]) {
  float s = __fmul_rn(a[0], b[0]);
  s = __fadd_rn(s, __fmul_rn(a[1], b[1]));
  return __fadd_rn(s, __fmul_rn(a[2], b[2]));
}

GB_DEV void cross3r(const float a[3], const float b[3], float r[3]) {
  r[0] = __fsub_rn(__fmul_rn(a[1], b[2]), __fmul_rn(a[2], b[1]));
  r[1] = __fsub_rn(__fmul_rn(a[2], b[0]), __fmul_rn(a[0], b[2]));
  r[2] = __fsub_rn(__fmul_rn(a[0], b[1]), __fmul_rn(a[1], b[0]));
}

// Hit parameter of ray (o, d) with triangle (v0, v1, v2), or +inf.
GB_DEV float ray_tri(const float o[3], const float d[3], const float v0[3], const float v1[3], const float v2[3]) {
  float e1[3], e2[3], s[3], p[3], q[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    e1[a] = __fsub_rn(v1[a], v0[a]);
    e2[a] = __fsub_rn(v2[a], v0[a]);
    s[a] = __fsub_rn(o[a], v0[a]);
  }
  cross3r(d, e2, p);
  float det = dot3r(e1, p);
  const float lim = __fmul_rn(__fmul_rn(__fmul_rn(dot3r(e1, e1), dot3r(e2, e2)), dot3r(d, d)), kGrazingRay);
  if (!(__fmul_rn(det, det) >= lim) || det == 0.0f) return __builtin_inff();
  float u = dot3r(s, p);
  cross3r(s, e1, q);
  float v = dot3r(d, q);
  float tn = dot3r(e2, q);
  if (det < 0.0f) {
    det = -det;
    u = -u;
    v = -v;
    tn = -tn;
  }
  if (!(u >= 0.0f && v >= 0.0f && __fadd_rn(u, v) <= det)) return __builtin_inff();
  return __fdiv_rn(tn, det);
}

struct RaycastArgs {
  GridDev g;                // verts, tris, nverts, lo, inv, res
  float hi[3];
  const uint32_t* ranges;   // [2R]
  const uint32_t* objs;     // [NO]
  const float* rays;        // [6][nrays]
  uint32_t nrays;
  float tmax;
  float* hit_t;             // [nrays]
  uint32_t* hit_obj;        // [nrays]
};

// A wave casts 64 rays together.  A ray of its own per lane through walk, cells
// and objects kept 3 of 64 lanes at work (each loop waits for its longest lane),
// so only the walk is a lane's own: every turn each ray takes its next kRayCells
// cells, and the objects of all those cells, one after another, are tested one
// per lane.  What bounds it then: a turn is a chain of four dependent loads (a
// cell's range, an object's id, its vertex indices, its vertices), and nearly
// all of them miss L2, 71M lines of 128 bytes for the case below (4.3 TB/s); more waves
// per SIMD were no faster (5 and 6 waves 2075 and 2196 us, when the walk had no
// quotients: they are 3% of it now).  So the ranges of several cells are loaded
// together, past the cell that will turn out to hold the hit: 1, 2, 4, 6, 8 cells
// 2633, 2281, 2075, 2217, 2354 us (as above).  1M rays over the 10M-triangle arch
// grid: a ray per lane 4035 us, this 2132; 300k rays over a 1M mesh 5906 and 674;
// 2000 over 5k uniform triangles 244 and 85.  Taking new rays
// for lanes that are done gave nothing (2% slower at 140 rays a wave).
constexpr int kRayCells = 4;
constexpr uint32_t kRayTests = 4096;  // most tests of one cell in a turn (a turn's slots are 32 bits)

// A hit as a word ordered by t, then id; t >= 0, so its sign (of a zero) is kept
// in the last bit.
GB_DEV uint64_t hit_key(float t, uint32_t id) {
  const uint32_t tb = __float_as_uint(t);
  return (static_cast<uint64_t>(tb & 0x7FFFFFFFu) << 33) | (static_cast<uint64_t>(id) << 1) | (tb >> 31);
}

// x, y or z of a uniform triple by the lane's axis.
GB_DEV float axis_of(const float v[3], int m) { return m == 0 ? v[0] : (m == 1 ? v[1] : v[2]); }

// One wave per workgroup.
__global__ __launch_bounds__(kWave, 4) void raycast_kernel(RaycastArgs a) {
  __shared__ float s_ray[8][kWave];            // each lane's ray: o, d, t0, t1
  __shared__ uint64_t s_best[kWave];           // its closest hit (hit_key)
  __shared__ uint32_t s_mark[kWave];           // slot -> the cell of the turn that starts there
  __shared__ uint32_t s_off[kRayCells][kWave]; // a cell's first object less its first slot of the turn
  const uint32_t lane = threadIdx.x;
  const GridDev& G = a.g;
  const uint32_t rx = G.res[0], rxy = G.res[0] * G.res[1];
  const float fres[3] = {static_cast<float>(G.res[0]), static_cast<float>(G.res[1]), static_cast<float>(G.res[2])};
  const uint32_t r = blockIdx.x * kWave + lane;

  bool have = false;           // the lane's ray is being cast
  float t0 = 0.0f, t1 = a.tmax;
  int m = 0, k = 0, kend = 0;  // dominant axis, slab, last slab
  float om = 0, dm = 1, o1 = 0, d1 = 0, o2 = 0, d2 = 0, w = 0, wt = 0;
  float te = -__builtin_inff(), tdone = 0;         // far face of the slab, and of the one before
  int lo1 = 0, hi1 = 0, j1 = 0, hi2 = -1, j2 = 0;  // the slab's cells still to visit: j2 > hi2 when none are left
  if (r < a.nrays) {
    float o[3], d[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      o[q] = a.rays[static_cast<uint64_t>(q) * a.nrays + r];
      d[q] = a.rays[static_cast<uint64_t>(3 + q) * a.nrays + r];
    }
    // [t0, t1]: [0, tmax] clipped to the box (the contract's slab test)
    bool live = true;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      if (d[q] != 0.0f) {
        const float ta = __fdiv_rn(__fsub_rn(G.lo[q], o[q]), d[q]);
        const float tb = __fdiv_rn(__fsub_rn(a.hi[q], o[q]), d[q]);
        t0 = fmaxf(t0, fminf(ta, tb));
        t1 = fminf(t1, fmaxf(ta, tb));
      } else if (!(o[q] >= G.lo[q] && o[q] <= a.hi[q])) {
        live = false;
      }
    }
    live = live && t0 <= t1;
    // the dominant axis m and the two others
    const float ad0 = fabsf(d[0]), ad1 = fabsf(d[1]), ad2 = fabsf(d[2]);
    m = (ad0 >= ad1 && ad0 >= ad2) ? 0 : (ad1 >= ad2 ? 1 : 2);
    om = axis_of(o, m);
    dm = axis_of(d, m);
    o1 = m == 0 ? o[1] : o[0];
    d1 = m == 0 ? d[1] : d[0];
    o2 = m == 2 ? o[1] : o[2];
    d2 = m == 2 ? d[1] : d[2];
    have = live && dm != 0.0f;
    if (have) {
      const float lom = axis_of(G.lo, m), inv = axis_of(G.inv, m), rm = axis_of(fres, m) - 1.0f;
      w = __fdiv_rn(__fsub_rn(axis_of(a.hi, m), lom), axis_of(fres, m));  // slab width
      wt = fabsf(w / dm);                                                  // in t
      const float step = dm > 0.0f ? 1.0f : -1.0f;
      const float k0 = fminf(fmaxf(floorf((om + t0 * dm - lom) * inv), 0.0f), rm);
      const float k1 = fminf(fmaxf(floorf((om + t1 * dm - lom) * inv), 0.0f), rm);
      // one slab early and late (rounding may misplace the ends), and one more
      // early: the walk steps first
      k = static_cast<int>(fminf(fmaxf(k0 - step, 0.0f), rm) - step);
      kend = static_cast<int>(fminf(fmaxf(k1 + step, 0.0f), rm));
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        s_ray[q][lane] = o[q];
        s_ray[3 + q][lane] = d[q];
      }
      s_ray[6][lane] = t0;
      s_ray[7][lane] = t1;
      s_best[lane] = hit_key(__builtin_inff(), 0xFFFFFFFFu);
    } else {
      a.hit_t[r] = __builtin_inff();
      a.hit_obj[r] = 0xFFFFFFFFu;
    }
  }
  const bool up = dm > 0.0f;
  while (ballot(have) != 0) {
    uint32_t b[kRayCells], cnt[kRayCells];
    if (have) {
      // a hit before the far face of the last slab visited (by the walk's margin) ends the walk
      const uint64_t key = s_best[lane];
      const float best = __uint_as_float(static_cast<uint32_t>(key >> 33));
      if (best <= (j2 > hi2 ? te : tdone) - kWalkPad * wt || (j2 > hi2 && (up ? k >= kend : k <= kend))) {
        a.hit_t[r] = (key & 1u) ? -best : best;
        a.hit_obj[r] = static_cast<uint32_t>(key >> 1);
        have = false;
      }
    }
    // the next cells of the walk, their ranges loaded together
    uint64_t cell[kRayCells];
    bool in[kRayCells];
#pragma unroll
    for (int c = 0; c < kRayCells; ++c) {
      in[c] = false;
      cell[c] = 0;
      if (have) {
        if (j2 > hi2 && (up ? k < kend : k > kend)) {
          k += up ? 1 : -1;
          // faces are numbered as the slabs below them: the far face of one slab is the near one of the next
          const float lom = axis_of(G.lo, m);
          const float near = te > -__builtin_inff() ? te : plane_t(lom + static_cast<float>(up ? k : k + 1) * w, om, dm);
          tdone = te;
          te = plane_t(lom + static_cast<float>(up ? k + 1 : k) * w, om, dm);
          const float ps = fmaxf(t0, near - kWalkPad * wt);
          const float pe = fminf(t1, te + kWalkPad * wt);
          if (ps <= pe) {
            {
              const float lo = m == 0 ? G.lo[1] : G.lo[0], inv = m == 0 ? G.inv[1] : G.inv[0];
              const float c0 = o1 + ps * d1, c1 = o1 + pe * d1;
              const float f0 = floorf((fminf(c0, c1) - lo) * inv - kWalkPad);
              const float f1 = floorf((fmaxf(c0, c1) - lo) * inv + kWalkPad);
              const float rr = (m == 0 ? fres[1] : fres[0]) - 1.0f;
              lo1 = static_cast<int>(fminf(fmaxf(f0, 0.0f), rr));
              hi1 = static_cast<int>(fminf(fmaxf(f1, 0.0f), rr));
            }
            {
              const float lo = m == 2 ? G.lo[1] : G.lo[2], inv = m == 2 ? G.inv[1] : G.inv[2];
              const float c0 = o2 + ps * d2, c1 = o2 + pe * d2;
              const float f0 = floorf((fminf(c0, c1) - lo) * inv - kWalkPad);
              const float f1 = floorf((fmaxf(c0, c1) - lo) * inv + kWalkPad);
              const float rr = (m == 2 ? fres[1] : fres[2]) - 1.0f;
              j2 = static_cast<int>(fminf(fmaxf(f0, 0.0f), rr));
              hi2 = static_cast<int>(fminf(fmaxf(f1, 0.0f), rr));
            }
            j1 = lo1;
          }
        }
        if (j2 <= hi2) {
          const uint32_t kk = static_cast<uint32_t>(k), u1 = static_cast<uint32_t>(j1), u2 = static_cast<uint32_t>(j2);
          const uint32_t x = m == 0 ? kk : u1, y = m == 1 ? kk : (m == 0 ? u1 : u2), z = m == 2 ? kk : u2;
          cell[c] = x + rx * y + static_cast<uint64_t>(rxy) * z;
          in[c] = true;
          const bool row = j1 == hi1;
          j1 = row ? lo1 : j1 + 1;
          j2 += row ? 1 : 0;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < kRayCells; ++c) {
      b[c] = in[c] ? a.ranges[2 * cell[c]] : 0u;
      const uint32_t e = in[c] ? a.ranges[2 * cell[c] + 1] : 0u;
      cnt[c] = e > b[c] ? e - b[c] : 0u;
    }
    // the tests: the cells' objects one after another, a test per lane
    while (true) {
      uint32_t n[kRayCells], mine = 0;
#pragma unroll
      for (int c = 0; c < kRayCells; ++c) mine += n[c] = cnt[c] < kRayTests ? cnt[c] : kRayTests;
      if (ballot(mine != 0) == 0) break;
      const uint32_t incl = wave_inclusive(mine, OpAdd{});
      const uint32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
      {
        uint32_t at = incl - mine;
#pragma unroll
        for (int c = 0; c < kRayCells; ++c) {
          s_off[c][lane] = b[c] - at;
          at += n[c];
        }
      }
      for (uint32_t base = 0; base < total; base += kWave) {
        s_mark[lane] = 0;
        wave_sync();
        uint32_t at = incl - mine;
#pragma unroll
        for (int c = 0; c < kRayCells; ++c) {
          if (n[c] != 0 && at < base + kWave && at + n[c] > base) s_mark[at > base ? at - base : 0u] = lane * kRayCells + c;
          at += n[c];
        }
        wave_sync();
        const uint32_t own = wave_inclusive(s_mark[lane], OpMax{}), ray = own / kRayCells;
        const uint32_t slot = base + lane;
        bool ok = slot < total;
        const uint32_t t = ok ? a.objs[s_off[own % kRayCells][ray] + slot] : 0u;
        ok = ok && t < G.ntris;  // an object id this scene does not have: never hit
        const uint32_t* tri = G.tris + 3 * static_cast<uint64_t>(ok ? t : 0u);
        uint32_t vi[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) vi[q] = ok ? tri[q] : 0u;
        ok = ok && vi[0] < G.nverts && vi[1] < G.nverts && vi[2] < G.nverts;
        if (ok) {
          float v[3][3], o[3], d[3];
#pragma unroll
          for (int jj = 0; jj < 3; ++jj)
#pragma unroll
            for (int q = 0; q < 3; ++q) v[jj][q] = G.verts[static_cast<uint64_t>(q) * G.nverts + vi[jj]];
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            o[q] = s_ray[q][ray];
            d[q] = s_ray[3 + q][ray];
          }
          const float th = ray_tri(o, d, v[0], v[1], v[2]);
          if (th >= s_ray[6][ray] && th <= s_ray[7][ray])
            atomicMin(reinterpret_cast<unsigned long long*>(&s_best[ray]), static_cast<unsigned long long>(hit_key(th, t)));
        }
        wave_sync();
      }
#pragma unroll
      for (int c = 0; c < kRayCells; ++c) {
        b[c] += n[c];
        cnt[c] -= n[c];
      }
    }
  }
}

}  // namespace gb
