// Tile scatter on the matrix cores, shared by P2G and the reverse of G2P.
//
// Both add, for every particle p of a cell tile and every stencil offset
// o = (ox, oy, oz) in {0,1,2}^3, the value w_o(f_p) (q_p + A_p o) into node
// base_p + o of the tile's 6^3 node region, with f_p the particle's position
// in its base cell (in cells), w_o the quadratic B-spline weight, q_p a
// 3-vector and A_p a 3x3 matrix (P2G also adds w_o m_p as a fourth value).
// A workgroup stages its particles in LDS in cell order (m, q, A row-major as
// 13 feature rows; the weights as 3 rows w_x and 9 rows w_y w_z), cuts each
// cell into units of at most SC_UNIT particles, and per unit forms Feat (13 x
// n) W (n x 27) with fp32 MFMA 16x16x4 (four particles per step, offsets in
// two 16-column tiles), the rows ordered so that the four result rows a lane
// holds give one node value: (1, ox, oy, oz) . rows.  Every wave adds its
// units' 27 x 4 values into its own 6^3 node block in LDS (a unit's 27 offsets
// reach 27 distinct nodes: plain adds); the node owners then add the wave
// blocks.
// What bounds a scatter is no one unit: of 4M particles' P2G the matrix phase is
// 70 us, its read-modify-writes of the node blocks 20 of them, the stresses 9,
// and the rest the particle loads and the phases between barriers.  Three
// things were worth their while: the staging thread evaluates its particle's
// weights once (every lane of a step evaluated the polynomials of its column
// anew: 22 % of all vector instructions), both tiles' old node values are
// read together, and the units are ordered by steps instead of lengths.  P2G
// of 4M / 500k / 20k particles 246 / 44.7 / 12.7 -> 234 / 42.6 / 12.0 us, reverse G2P of
// 256k 45 -> 41.
#pragma once

#include "dw_internal.h"

namespace dw {

constexpr int SC_L = 6;           // local node extent of a cell tile's stencils
constexpr int SC_NODES = 216;     // 6^3
constexpr int SC_DAT = 13;        // staged feature rows per particle: m (P2G only), q(3), A(9)
constexpr int SC_WGT = 12;        // staged weight rows: w_x(3), w_y w_z(9)
constexpr int SC_UNIT = 16;       // particles per unit (4 MFMA steps): a dense cell spreads over waves
constexpr int SC_MAX_UNITS = 64 + WORK_CHUNK / SC_UNIT;  // bounds the sum over cells of ceil(count / unit)
constexpr int SC_THREADS = WORK_CHUNK;
constexpr int SC_WAVES = SC_THREADS / 64;
constexpr int SC_PITCH = WORK_CHUNK + 4;  // staged rows padded: the rows one read touches hit distinct banks
constexpr int SC_TAIL = SC_UNIT;  // floats after the last row: a step reads (and drops) up to these past a unit's end

typedef float floatx4_t __attribute__((ext_vector_type(4)));

// Per-lane constants of the MFMA 16x16x4 roles: r16 = row of the feature
// operand / column (offset within a 16-wide tile) of the weight operand,
// kq = particle slot of the step.  MASS: the features have a mass row.
struct ScLane {
  int kq;
  int at_f;                // element of the lane's feature row, slot kq
  int at_x[2], at_yz[2];   // elements of its columns' weight rows, slot kq
  int oo[2], onode[2];
  float fo[2][3];
};

template <bool MASS>
__device__ __forceinline__ ScLane sc_lane(int lane) {
  ScLane L;
  const int r16 = lane & 15;
  L.kq = lane >> 4;
  // staged feature of operand row r16, grouped so that result rows 4 kq ..
  // 4 kq + 3 (held by lane group kq) all feed node value kq:
  //   rows 0-3: m, -, -, -;  rows 4 + 4d .. 7 + 4d: q_d, A_d0, A_d1, A_d2
  // (rows without a feature repeat the first one; group 0 drops them below)
  const int feat = r16 < 4 ? 0 : ((r16 & 3) == 0 ? (r16 >> 2) : 4 + 3 * ((r16 >> 2) - 1) + (r16 & 3) - 1);
  L.at_f = (MASS || feat == 0 ? feat : feat - 1) * SC_PITCH + L.kq;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int o = t * 16 + r16;
    L.oo[t] = o;
    const int oc = o < 27 ? o : 0;
    const int ox = oc % 3, oy = (oc / 3) % 3, oz = oc / 9;
    L.onode[t] = ox + SC_L * (oy + SC_L * oz);
    L.at_x[t] = ox * SC_PITCH + L.kq;
    L.at_yz[t] = (3 + oc / 3) * SC_PITCH + L.kq;
    L.fo[t][0] = L.kq ? (float)ox : 0.f;
    L.fo[t][1] = L.kq ? (float)oy : 0.f;
    L.fo[t][2] = L.kq ? (float)oz : 0.f;
  }
  return L;
}

// DPP source v shifted by CTRL within the enabled rows (ROWS mask), zero
// where the source lane lies outside the row or the row is not enabled
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int sc_dpp(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}

// Inclusive scan over the 64 lanes of a fully active wave without LDS round
// trips: Hillis-Steele inside each 16-lane row (row shifts by 1, 2, 4, 8),
// then row 0's total broadcast into row 1 and row 2's into row 3 (row
// broadcast of lane 15), then the total of rows 0-1 into rows 2 and 3 (row
// broadcast of lane 31).
__device__ __forceinline__ int sc_wave_scan(int v) {
  v += sc_dpp<0x111>(v);
  v += sc_dpp<0x112>(v);
  v += sc_dpp<0x114>(v);
  v += sc_dpp<0x118>(v);
  v += sc_dpp<0x142, 0xA>(v);
  v += sc_dpp<0x143, 0xC>(v);
  return v;
}

// Wave 0: exclusive scan of the 64 cell counts into s_off / s_cur and the
// unit descriptors (first slot | count << 10 | node base << 17).  The units
// are listed whole ones first, then the partial ones (each cell's last) by
// decreasing number of four-particle steps, so that the two units a wave takes
// at a time mostly have as many.
// The order depends only on the counts.
__device__ __forceinline__ void sc_scan_units(int lane, const int *s_cnt, int *s_off, int *s_cur, int *s_udesc,
                                              int *s_nunits) {
  const int v = s_cnt[lane];
  const int inc = sc_wave_scan(v);
  s_off[lane] = inc - v;
  s_cur[lane] = inc - v;
  const int nbase = (lane & 3) + SC_L * (((lane >> 2) & 3) + SC_L * (lane >> 4));
  const int nf = v / SC_UNIT, pl = v % SC_UNIT;  // whole units, length of the partial one
  const int finc = sc_wave_scan(nf);
  const int nfull = __shfl(finc, 63, 64);
  for (int q = 0; q < nf; ++q) s_udesc[finc - nf + q] = (inc - v + q * SC_UNIT) | (SC_UNIT << 10) | (nbase << 17);
  const uint64_t below = (1ull << lane) - 1ull;
  int pos = nfull;
#pragma unroll
  for (int steps = SC_UNIT / 4; steps > 0; --steps) {
    const uint64_t m = __ballot((pl + 3) / 4 == steps);
    if ((pl + 3) / 4 == steps)
      s_udesc[pos + __popcll(m & below)] = (inc - v + nf * SC_UNIT) | (pl << 10) | (nbase << 17);
    pos += __popcll(m);
  }
  if (lane == 63) *s_nunits = pos;
}

// Stage one particle at `slot`: its weights and features (A row-major).
template <bool MASS>
__device__ __forceinline__ void sc_stage(float *s_dat, float *s_wgt, int slot, const float f[3], float m,
                                         const float q[3], const float A[9]) {
  float w[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a) bspline_w(f[a], w[a]);
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    s_wgt[o * SC_PITCH + slot] = w[0][o];
#pragma unroll
    for (int oy = 0; oy < 3; ++oy) s_wgt[(3 + oy + 3 * o) * SC_PITCH + slot] = w[1][oy] * w[2][o];
  }
  float *d = s_dat + slot;
  if (MASS) {
    *d = m;
    d += SC_PITCH;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) d[k * SC_PITCH] = q[k];
#pragma unroll
  for (int k = 0; k < 9; ++k) d[(3 + k) * SC_PITCH] = A[k];
}

// Pass over the units on the matrix cores; wave `wid` adds into wnode.
// Two adjacent units of the list (nearly equal lengths) per wave at a time.
__device__ __forceinline__ void sc_units_mfma(const ScLane &L, int wid, const float *s_dat, const float *s_wgt,
                                              const int *s_udesc, int nunits, float (*wnode)[4]) {
  for (int u = 2 * wid; u < nunits; u += 2 * SC_WAVES) {
    int kn[2], cb[2];
    const float *pf[2], *px[2][2], *py[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int ue = u + e;
      const int d = __builtin_amdgcn_readfirstlane(ue < nunits ? s_udesc[ue] : 0);
      const int k0 = d & 1023;
      kn[e] = (d >> 10) & 127;
      cb[e] = d >> 17;
      pf[e] = s_dat + L.at_f + k0;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        px[e][t] = s_wgt + L.at_x[t] + k0;
        py[e][t] = s_wgt + L.at_yz[t] + k0;
      }
    }
    floatx4_t acc[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[e][t] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    const int len = max(kn[0], kn[1]);
#pragma unroll
    for (int kk = 0; kk < SC_UNIT; kk += 4) {
      if (kk >= len) break;
      float av[2], w[2][2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        av[e] = pf[e][kk];
#pragma unroll
        for (int t = 0; t < 2; ++t) w[e][t] = px[e][t][kk] * py[e][t][kk];
      }
      // slots past a unit's end hold other particles or nothing: both
      // operands zero there
#pragma unroll
      for (int e = 0; e < 2; ++e)
        if (kn[e] < kk + 4) {
          const bool live = L.kq < kn[e] - kk;
          av[e] = live ? av[e] : 0.f;
          w[e][0] = live ? w[e][0] : 0.f;
          w[e][1] = live ? w[e][1] : 0.f;
        }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          acc[e][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], w[e][t], acc[e][t], 0, 0, 0);
    }
    // lane (kq, r16) holds rows 4 kq + i of column r16 (offset o) of each
    // tile: node value kq of node cell + o is row 4 kq + (1, ox, oy, oz).  A
    // unit's nodes are distinct, so both tiles' old values are read before
    // either is written.
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (kn[e] == 0) continue;
      float *p[2], old[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        p[t] = &wnode[cb[e] + L.onode[t]][L.kq];
        old[t] = *p[t];
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const floatx4_t a4 = acc[e][t];
        const float v = a4[0] + L.fo[t][0] * a4[1] + L.fo[t][1] * a4[2] + L.fo[t][2] * a4[3];
        if (L.oo[t] < 27) *p[t] = old[t] + v;
      }
    }
  }
}

// Deterministic mode, second pass of the tile scatter: every node of an
// active node tile sums, in a fixed order (cell tile z, y, x, then work
// item), the partial node blocks (item_part, 6^3 x 4 values per work item)
// of the work items whose 6^3 region covers it.  ADJ = false (P2G):
// overwrites gm with value 0 and gmv with values 1-3.  ADJ = true (reverse
// G2P): adds values 1-3 into gmv, the grid-velocity adjoint.
// Bit-reproducible given a deterministic particle order.
template <bool ADJ>
static __global__ __launch_bounds__(256) void k_det_gather(GridDev g, const int32_t *__restrict__ node_tiles,
                                                        const int32_t *__restrict__ n_tiles,
                                                        const int32_t *__restrict__ tile_count,
                                                        const int32_t *__restrict__ item_first,
                                                        const float *__restrict__ item_part, float *__restrict__ gm,
                                                        float *__restrict__ gmv, int64_t N,
                                                        int32_t *__restrict__ ticket) {
  int nt = *n_tiles;
  if (!ADJ && blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;  // for the next P2G
  int sub = threadIdx.x >> 6, l = threadIdx.x & 63;
  for (int it = blockIdx.x * 4 + sub; it < nt; it += gridDim.x * 4) {
    int t = node_tiles[it];
    int tx = t % g.tx, ty = (t / g.tx) % g.ty, tz = t / (g.tx * g.ty);
    int lx = l & 3, ly = (l >> 2) & 3, lz = l >> 4;
    int i = tx * 4 + lx, j = ty * 4 + ly, k = tz * 4 + lz;
    if (i >= g.nx || j >= g.ny || k >= g.nz) continue;
    float sm = 0.f, s0 = 0.f, s1 = 0.f, s2 = 0.f;
    for (int dz = 1; dz >= 0; --dz) {
      int cz = tz - dz, oz = lz + 4 * dz;
      if (cz < 0 || oz > 5) continue;
      for (int dy = 1; dy >= 0; --dy) {
        int cy = ty - dy, oy = ly + 4 * dy;
        if (cy < 0 || oy > 5) continue;
        for (int dxx = 1; dxx >= 0; --dxx) {
          int cx = tx - dxx, ox = lx + 4 * dxx;
          if (cx < 0 || ox > 5) continue;
          int ct = cx + g.tx * (cy + g.ty * cz);
          int nitem = (tile_count[ct] + WORK_CHUNK - 1) / WORK_CHUNK;
          int li = ox + SC_L * (oy + SC_L * oz);
          for (int q = 0; q < nitem; ++q) {
            const float *src = item_part + ((int64_t)(item_first[ct] + q) * SC_NODES + li) * 4;
            sm += src[0];
            s0 += src[1];
            s1 += src[2];
            s2 += src[3];
          }
        }
      }
    }
    int64_t node = i + (int64_t)g.nx * (j + (int64_t)g.ny * k);
    if (ADJ) {
      gmv[node] += s0;
      gmv[N + node] += s1;
      gmv[2 * N + node] += s2;
    } else {
      gm[node] = sm;
      gmv[node] = s0;
      gmv[N + node] = s1;
      gmv[2 * N + node] = s2;
    }
  }
}

}  // namespace dw
