// Differentiable rendering of the 3D Gaussian kernels and the photometric
// loss L_render (Sec. 3.3, Eq. rendering and L_render; appendix "3D Gaussian
// Representation").
//
// Forward (gs_render), every stage a kernel of this file:
//   1. k_gs_project: per kernel, camera point p = R mu + t, projected centre,
//      2-D covariance J R Sigma R^T J^T and its inverse (the conic), the
//      pixel box where alpha can reach alpha_min, and the 16 x 16 pixel
//      tiles that box covers.  Kernels behind the near plane, with a
//      degenerate 2-D covariance or with no pixel in reach are not drawn.
//   2. stable LSD radix sort of (depth bits, kernel) -- 4 passes of 8 bits;
//      kernels that are not drawn carry the largest key and no tiles.
//   3. exclusive scan of the tile counts in depth order; every drawn kernel
//      writes one (tile, kernel) pair per covered tile, in depth order.
//   4. stable radix sort of the pairs by tile (depth order kept inside a
//      tile), then each tile's range in the sorted list.
//   5. k_gs_classify: tiles whose lists are long and hold small kernels are
//      rasterised by four workgroups, the others by one.
//   6. k_gs_raster: batches of list entries staged in LDS, each wave keeps
//      those whose pixel box meets its pixels and blends them front to back.
//      A pixel stops once its transmittance falls below t_min; the list
//      position it stopped at is kept for the reverse pass.
// Reverse (gs_render_adj): front to back again, recomputing alpha and T, 16
// entries x 4 pixels at a time.  With s_i = G . c_i (G the image gradient at
// the pixel), dL/dalpha_i = T_i s_i - (G . C - P_i) / (1 - alpha_i) where
// P_i = sum_{j <= i} T_j alpha_j s_j and C includes the background term.  The
// sums over pixels are taken in registers; k_gs_project_adj takes the centre
// and conic adjoints back to mu and Sigma through the projection.
// Loss (render_loss): L1 and SSIM with an 11 x 11 Gaussian window
// (sigma 1.5, zero padding) per channel; the five window sums are separable
// convolutions staged in LDS; the gradient of the SSIM mean is the window
// correlation of the per-pixel partial derivatives (the window is
// symmetric).  Loss partial sums are reduced in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <utility>

#include "dw_internal.h"

namespace dw {

constexpr int GS_TILE = 16;
constexpr int GS_THREADS = 256;
// per-kernel sums of the reverse pass, e = dL/dalpha exp(-q/2) summed over
// pixels with the weights: [0..2] colour, [3] e, [4] e dx, [5] e dx^2,
// [6] e dx dy, [7] e dy^2, [8] e dy
constexpr int GS_NB = 9;
constexpr int RS_THREADS = 256;
constexpr int RS_ROUNDS = 16;                     // keys per thread of large inputs (small ones: 4 or 8)
constexpr int RS_CHUNK = RS_THREADS * RS_ROUNDS;  // keys per radix-sort block (at most)
constexpr int RS_DIRECT = 64;                     // blocks whose histograms a block adds up by itself
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER = 8;
constexpr int SCAN_CHUNK = SCAN_THREADS * SCAN_PER;
constexpr int SCAN_TOP_MAX = 16384;  // blocks of the tile-count scan at most

// workspace header: [0] status, [1] pair count, [2] tiles of one raster
// workgroup, [3] tiles of four, [4] and [5] raster and reverse tickets, [6] a drawn kernel has a non-finite
// colour, [GS_CNT0 ...] 64 partial
// 64-bit pair totals (one per block residue, to spread the atomics)
constexpr int GS_HDR_INTS = 256;
constexpr int GS_CNT0 = 64;
constexpr int GS_NCNT = 64;

struct CamDev {
  int W, H, tw, th;
  float fx, fy, cx, cy;
  float R[9], t[3];
  float near_, amin, tmin;
  float bg[3];
};

// Workspace of gs_render / gs_render_adj (all sections 256-aligned):
//   header [256] int32: status, pair count, 64 partial pair totals (u64)
//   rec [n] 3 float4: (mx, my, A, B), (C, o, c0, c1), (c2, pixel box, -),
//   the box as two words of two 16-bit numbers: first | last << 16 in x, y
//   rect [n] tile box, two words of two 16-bit numbers: first | last << 16 in
//   x, y; cnt [n] int32
//   key_a, key_b [n] u32, id_a, id_b [n] int32   (depth sort)
//   off [n + 1] int32 (tile-count scan in depth order)
//   pk_a, pk_b [P] u32, pv_a, pv_b [P] int32      (pair sort)
//   hist [nblk(max(n, P))][256] int32 (radix sort), bsum [SCAN_TOP_MAX] int32
//   (digit totals of a radix pass, block sums of the tile-count scan)
//   range [T] int2, whole, split [T] int32 (tiles of one raster workgroup and
//   of four), last [W * H] int32
//   gbar [n][9] float (per-kernel sums of the reverse pass, GS_NB)
struct GsWs {
  int32_t *hdr;
  float4 *rec;
  uint2 *rect;
  int32_t *cnt;
  uint32_t *key_a, *key_b;
  int32_t *id_a, *id_b;
  int32_t *off;
  uint32_t *pk_a, *pk_b;
  int32_t *pv_a, *pv_b;
  int32_t *hist, *bsum;
  int2 *range;
  int32_t *whole, *split;
  int32_t *last;
  float *gbar;
  size_t bytes;
};

static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

static int64_t rs_blocks(int64_t m) { return (m + RS_CHUNK - 1) / RS_CHUNK; }

// rows of 256 counters that radix_sort has: the histograms of RS_CHUNK blocks,
// and bsum behind them, which only passes of more than RS_DIRECT blocks use
static int64_t rs_rows(int64_t n, int64_t P) { return rs_blocks(n > P ? n : P) + SCAN_TOP_MAX / 256; }

static GsWs gs_layout(char *base, int64_t n, int64_t P, int W, int H) {
  GsWs w;
  const int64_t T = (int64_t)((W + GS_TILE - 1) / GS_TILE) * ((H + GS_TILE - 1) / GS_TILE);
  const int64_t nb = rs_blocks(n > P ? n : P);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char *p = base ? base + o : nullptr;
    o += al256(bytes);
    return p;
  };
  w.hdr = (int32_t *)take(GS_HDR_INTS * 4);
  w.rec = (float4 *)take((size_t)n * 3 * sizeof(float4));
  w.rect = (uint2 *)take((size_t)n * sizeof(uint2));
  w.cnt = (int32_t *)take((size_t)n * 4);
  w.key_a = (uint32_t *)take((size_t)n * 4);
  w.key_b = (uint32_t *)take((size_t)n * 4);
  w.id_a = (int32_t *)take((size_t)n * 4);
  w.id_b = (int32_t *)take((size_t)n * 4);
  w.off = (int32_t *)take((size_t)(n + 1) * 4);
  w.pk_a = (uint32_t *)take((size_t)P * 4);
  w.pk_b = (uint32_t *)take((size_t)P * 4);
  w.pv_a = (int32_t *)take((size_t)P * 4);
  w.pv_b = (int32_t *)take((size_t)P * 4);
  w.hist = (int32_t *)take((size_t)256 * nb * 4);
  w.bsum = (int32_t *)take((size_t)SCAN_TOP_MAX * 4);
  w.range = (int2 *)take((size_t)T * sizeof(int2));
  w.whole = (int32_t *)take((size_t)T * 4);
  w.split = (int32_t *)take((size_t)T * 4);
  w.last = (int32_t *)take((size_t)W * H * 4);
  w.gbar = (float *)take((size_t)GS_NB * n * 4);
  w.bytes = o;
  return w;
}

// ------------------------------------------------------------- projection

// Everything of one kernel that the raster and its reverse need.
struct Proj {
  bool drawn;
  float px, py, pz;      // camera point
  float mx, my;          // projected centre (pixels)
  float a, b, c;         // 2-D covariance [[a, b], [b, c]]
  float A, B, C;         // its inverse
  float T0[3], T1[3];    // rows of J R
  int i0, i1, j0, j1;    // pixels where alpha can reach alpha_min
  int tx0, tx1, ty0, ty1;
};

__device__ __forceinline__ Proj gs_proj(const CamDev &K, float mux, float muy, float muz, const float S[6],
                                        float o) {
  Proj r;
  r.drawn = false;
  r.tx0 = r.ty0 = 0;
  r.tx1 = r.ty1 = -1;
  r.px = K.R[0] * mux + K.R[1] * muy + K.R[2] * muz + K.t[0];
  r.py = K.R[3] * mux + K.R[4] * muy + K.R[5] * muz + K.t[1];
  r.pz = K.R[6] * mux + K.R[7] * muy + K.R[8] * muz + K.t[2];
  if (!(r.pz > K.near_)) return r;
  const float iz = 1.0f / r.pz;
  r.mx = K.fx * r.px * iz + K.cx;
  r.my = K.fy * r.py * iz + K.cy;
  // J = [[fx/z, 0, -fx px/z^2], [0, fy/z, -fy py/z^2]]; T = J R
  const float j00 = K.fx * iz, j02 = -K.fx * r.px * iz * iz;
  const float j11 = K.fy * iz, j12 = -K.fy * r.py * iz * iz;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    r.T0[c] = j00 * K.R[c] + j02 * K.R[6 + c];
    r.T1[c] = j11 * K.R[3 + c] + j12 * K.R[6 + c];
  }
  // Sigma T^T columns
  const float Sm[9] = {S[0], S[3], S[4], S[3], S[1], S[5], S[4], S[5], S[2]};
  float u0[3], u1[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u0[a] = Sm[3 * a] * r.T0[0] + Sm[3 * a + 1] * r.T0[1] + Sm[3 * a + 2] * r.T0[2];
    u1[a] = Sm[3 * a] * r.T1[0] + Sm[3 * a + 1] * r.T1[1] + Sm[3 * a + 2] * r.T1[2];
  }
  r.a = r.T0[0] * u0[0] + r.T0[1] * u0[1] + r.T0[2] * u0[2];
  r.b = r.T0[0] * u1[0] + r.T0[1] * u1[1] + r.T0[2] * u1[2];
  r.c = r.T1[0] * u1[0] + r.T1[1] * u1[1] + r.T1[2] * u1[2];
  const float det = r.a * r.c - r.b * r.b;
  if (!(det > 0.f) || !(r.a > 0.f)) return r;
  const float id = 1.0f / det;
  r.A = r.c * id;
  r.B = -r.b * id;
  r.C = r.a * id;
  // pixel box: alpha = o exp(-q/2) >= amin  <=>  q <= Q = 2 ln(o / amin);
  // the ellipse q <= Q reaches sqrt(Q a) in x and sqrt(Q c) in y (padded by a
  // relative 1e-4 and 1e-3 pixel against rounding at the rim)
  int i0 = 0, i1 = K.W - 1, j0 = 0, j1 = K.H - 1;
  if (K.amin > 0.f) {
    if (!(o >= K.amin)) return r;
    const float Q = 2.0f * logf(o / K.amin);
    const float ex = sqrtf(Q * r.a) * 1.0001f + 1e-3f, ey = sqrtf(Q * r.c) * 1.0001f + 1e-3f;
    const float fx0 = ceilf(r.mx - ex - 0.5f), fx1 = floorf(r.mx + ex - 0.5f);
    const float fy0 = ceilf(r.my - ey - 0.5f), fy1 = floorf(r.my + ey - 0.5f);
    if (!(fx1 >= 0.f && fx0 <= (float)(K.W - 1) && fy1 >= 0.f && fy0 <= (float)(K.H - 1))) return r;
    i0 = (int)fmaxf(fx0, 0.f);
    i1 = (int)fminf(fx1, (float)(K.W - 1));
    j0 = (int)fmaxf(fy0, 0.f);
    j1 = (int)fminf(fy1, (float)(K.H - 1));
    if (i0 > i1 || j0 > j1) return r;
  }
  r.i0 = i0;
  r.i1 = i1;
  r.j0 = j0;
  r.j1 = j1;
  r.tx0 = i0 / GS_TILE;
  r.tx1 = i1 / GS_TILE;
  r.ty0 = j0 / GS_TILE;
  r.ty1 = j1 / GS_TILE;
  r.drawn = true;
  return r;
}

__global__ __launch_bounds__(256) void k_gs_project(CamDev K, int n, const float *__restrict__ mu,
                                                    const float *__restrict__ sigma, const float *__restrict__ col,
                                                    const float *__restrict__ op, GsWs w) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  const bool has = g < n;
  float S[6] = {1.f, 1.f, 1.f, 0.f, 0.f, 0.f};
  float o = 0.f, m0 = 0.f, m1 = 0.f, m2 = 0.f;
  if (has) {
#pragma unroll
    for (int e = 0; e < 6; ++e) S[e] = sigma[(int64_t)e * n + g];
    o = op[g];
    m0 = mu[g];
    m1 = mu[(int64_t)n + g];
    m2 = mu[2 * (int64_t)n + g];
  }
  Proj r = gs_proj(K, m0, m1, m2, S, o);
  r.drawn = r.drawn && has;
  int c = 0;
  uint32_t key = 0xffffffffu;
  if (r.drawn) {
    c = (r.tx1 - r.tx0 + 1) * (r.ty1 - r.ty0 + 1);
    key = __float_as_uint(r.pz);  // pz > near >= 0: the bits order like the values
    if (!(isfinite(col[g]) && isfinite(col[(int64_t)n + g]) && isfinite(col[2 * (int64_t)n + g]))) atomicOr(&w.hdr[6], 1);
    w.rec[3 * (int64_t)g] = make_float4(r.mx, r.my, r.A, r.B);
    w.rec[3 * (int64_t)g + 1] = make_float4(r.C, o, col[g], col[(int64_t)n + g]);
    w.rec[3 * (int64_t)g + 2] = make_float4(col[2 * (int64_t)n + g], __uint_as_float((uint32_t)r.i0 | (uint32_t)r.i1 << 16),
                                            __uint_as_float((uint32_t)r.j0 | (uint32_t)r.j1 << 16), 0.f);
  }
  if (has) {
    w.rect[g] = make_uint2((uint32_t)r.tx0 | (uint32_t)r.tx1 << 16, (uint32_t)r.ty0 | (uint32_t)r.ty1 << 16);
    w.cnt[g] = c;
    w.key_a[g] = key;
    w.id_a[g] = g;
  }
  // 64-bit pair total (the int32 scan below is only trusted when it fits):
  // a block sum added to one of 64 partial counters
  __shared__ unsigned long long s_c[256 / 64];
  unsigned long long sw = (unsigned long long)c;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) sw += __shfl_xor(sw, m, 64);
  if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = sw;
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long b = s_c[0] + s_c[1] + s_c[2] + s_c[3];
    if (b) atomicAdd(reinterpret_cast<unsigned long long *>(w.hdr + GS_CNT0) + (blockIdx.x % GS_NCNT), b);
  }
}

// ------------------------------------------------------------ scan (int32)

__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) {
    const int t = __shfl_up(v, sh, 64);
    if (lane >= sh) v += t;
  }
  return v;
}

// exclusive scan of the per-thread values of a 256-thread block; returns the
// thread's offset, *total the block sum
__device__ __forceinline__ int block_excl_scan(int v, int *s_w, int *total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int inc = wave_incl_scan(v, lane);
  if (lane == 63) s_w[wid] = inc;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int q = 0; q < SCAN_THREADS / 64; ++q) {
    base += q < wid ? s_w[q] : 0;
    tot += s_w[q];
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// Length m may live on the device (m_dev, not NULL) with m_cap as bound.
__device__ __forceinline__ int64_t dev_len(const int32_t *m_dev, int64_t m_cap) {
  if (!m_dev) return m_cap;
  const int64_t m = *m_dev;
  return m <= m_cap ? m : 0;
}

// Tile counts in depth order and their exclusive scan: the first kernel
// gathers the counts and leaves a sum per block of SCAN_CHUNK, the second
// adds up the sums before its own (a block-wide reduction of at most
// SCAN_TOP_MAX values) and scans its counts.  Its last block has the total:
// a 64-bit pair total (the partial counters of k_gs_project; the int32 scan is
// only trusted when it fits) above the capacity sets status bit
// DW_STATUS_RENDER_OVERFLOW and the pair count hdr[1] to 0: nothing is
// emitted, sorted or drawn.
__global__ __launch_bounds__(SCAN_THREADS) void k_gs_cnt_sums(int n, const int32_t *__restrict__ id,
                                                              const int32_t *__restrict__ cnt,
                                                              int32_t *__restrict__ off, int32_t *__restrict__ bsum) {
  __shared__ int s_w[SCAN_THREADS / 64];
  const int64_t b0 = (int64_t)blockIdx.x * SCAN_CHUNK;
  int c[SCAN_PER], v = 0;
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    const int64_t r = b0 + q * SCAN_THREADS + threadIdx.x;
    c[q] = r < n ? cnt[id[r]] : 0;
  }
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    const int64_t r = b0 + q * SCAN_THREADS + threadIdx.x;
    if (r < n) off[r] = c[q];
    v += c[q];
  }
  int tot;
  block_excl_scan(v, s_w, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_gs_cnt_scan(int n, const int32_t *__restrict__ bsum, int64_t cap,
                                                              int32_t *__restrict__ off, int32_t *hdr) {
  __shared__ int s_w[SCAN_THREADS / 64];
  int before = 0;
  for (int q = threadIdx.x; q < (int)blockIdx.x; q += SCAN_THREADS) before += bsum[q];
  const int64_t b0 = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_PER;
  int v[SCAN_PER], s = 0;
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    v[q] = b0 + q < n ? off[b0 + q] : 0;
    s += v[q];
  }
  int base, tot;
  block_excl_scan(before, s_w, &base);
  int run = base + block_excl_scan(s, s_w, &tot);
#pragma unroll
  for (int q = 0; q < SCAN_PER; ++q) {
    if (b0 + q < n) off[b0 + q] = run;
    run += v[q];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x < 64) {
    unsigned long long t = reinterpret_cast<const unsigned long long *>(hdr + GS_CNT0)[threadIdx.x];
    static_assert(GS_NCNT == 64, "one counter per lane");
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) t += __shfl_xor(t, m, 64);
    if (threadIdx.x == 0) {
      const bool over = t > (unsigned long long)cap;
      if (over) hdr[0] |= DW_STATUS_RENDER_OVERFLOW;
      hdr[1] = over ? 0 : base + tot;
    }
  }
}

// -------------------------------------------------- stable LSD radix sort
//
// One pass sorts by a digit of at most 8 bits: a digit histogram per block of
// RS_CHUNK keys (hist[block][256]), its exclusive scan over the blocks
// (k_rs_scan; up to RS_DIRECT blocks the scatter adds the histograms up by
// itself, which saves the launch), then k_rs_scatter.  There a wave ranks
// 1024 consecutive keys in 16 rounds of 64 against counters of its own (a
// key's rank is its digit's count in the wave so far plus the same-digit
// lanes below it, from a 64-bit peer mask of ballots), so the rounds need no
// barrier; the block's keys are put in order in LDS and stored in runs of
// equal digits.  Keys of equal digit keep their input order, so the passes
// compose to a stable sort.
// Bound by latency for small inputs and by the 16 bytes moved per key and
// pass for large ones; the histograms are therefore added up 32 loads at a
// time.  A pass over 20k keys 31 -> 8.5 us, over 256k 16, over 1M 39 -> 22 us;
// the two tile passes of 5.7M pairs 190 -> 76 us (before: three barriers per
// round of 256 keys, stores scattered key by key, three scan kernels).

template <int ROUNDS>
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const uint32_t *__restrict__ key, int64_t m_cap,
                                                        const int32_t *m_dev, int shift, uint32_t mask,
                                                        int32_t *__restrict__ hist) {
  __shared__ int s_h[RS_THREADS / 64][256];
  const int64_t m = dev_len(m_dev, m_cap);
  const int64_t b0 = (int64_t)blockIdx.x * (RS_THREADS * ROUNDS);
  if (b0 >= m) return;  // block-uniform; no reader looks at this block's row
  const int wid = threadIdx.x >> 6;
#pragma unroll
  for (int w = 0; w < RS_THREADS / 64; ++w) s_h[w][threadIdx.x] = 0;
  uint32_t k[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t i = b0 + r * RS_THREADS + threadIdx.x;
    k[r] = i < m ? key[i] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (b0 + r * RS_THREADS + threadIdx.x < m) atomicAdd(&s_h[wid][(k[r] >> shift) & mask], 1);
  __syncthreads();
  int c = 0;
#pragma unroll
  for (int w = 0; w < RS_THREADS / 64; ++w) c += s_h[w][threadIdx.x];
  hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = c;
}

// exclusive scan of every digit over the blocks, in place, and the digit
// totals: 16 digits (64 bytes of a row) x 64 groups of blocks per workgroup
__global__ __launch_bounds__(1024) void k_rs_scan(int64_t m_cap, const int32_t *m_dev, int32_t *__restrict__ hist,
                                                  int32_t *__restrict__ total) {
  __shared__ int s_g[64][17];
  const int nblk = (int)((dev_len(m_dev, m_cap) + RS_CHUNK - 1) / RS_CHUNK);
  if (nblk <= RS_DIRECT) return;
  const int d = blockIdx.x * 16 + (threadIdx.x & 15), g = threadIdx.x >> 4;
  const int per = (nblk + 63) / 64, r0 = g * per, r1 = min(nblk, r0 + per);
  int s = 0;
#pragma unroll 8
  for (int r = r0; r < r1; ++r) s += hist[(int64_t)r * 256 + d];
  s_g[g][threadIdx.x & 15] = s;
  __syncthreads();
  int run = 0;
  for (int q = 0; q < g; ++q) run += s_g[q][threadIdx.x & 15];
  if (g == 63) total[d] = run + s;
#pragma unroll 8
  for (int r = r0; r < r1; ++r) {
    const int c = hist[(int64_t)r * 256 + d];
    hist[(int64_t)r * 256 + d] = run;
    run += c;
  }
}

template <int ROUNDS, int BITS>
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(const uint32_t *__restrict__ kin,
                                                           const int32_t *__restrict__ vin, int64_t m_cap,
                                                           const int32_t *m_dev, int shift,
                                                           const int32_t *__restrict__ hist,
                                                           const int32_t *__restrict__ total,
                                                           uint32_t *__restrict__ kout, int32_t *__restrict__ vout) {
  constexpr int CHUNK = RS_THREADS * ROUNDS;
  constexpr uint32_t mask = (1u << BITS) - 1u;
  __shared__ int s_cnt[RS_THREADS / 64][256];  // per wave: keys of the digit, then their first slot in the block
  __shared__ int s_delta[256];                 // slot in the block -> place in the output
  __shared__ uint32_t s_k[CHUNK];
  __shared__ int32_t s_v[CHUNK];
  __shared__ int s_w[SCAN_THREADS / 64];
  const int64_t m = dev_len(m_dev, m_cap);
  const int64_t b0 = (int64_t)blockIdx.x * CHUNK;
  if (b0 >= m) return;  // block-uniform
  const int nvalid = (int)min((int64_t)CHUNK, m - b0);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int w0 = wid * (CHUNK / (RS_THREADS / 64)) + lane;  // this lane's key of round 0
  uint32_t k[ROUNDS];
  int32_t v[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = w0 + r * 64;
    k[r] = i < nvalid ? kin[b0 + i] : 0u;
    v[r] = i < nvalid ? vin[b0 + i] : 0;
  }
#pragma unroll
  for (int w = 0; w < RS_THREADS / 64; ++w) s_cnt[w][threadIdx.x] = 0;
  // thread d: keys of digit d in the blocks before this one, and in all
  const int nblk = (int)((m + CHUNK - 1) / CHUNK);
  int before = 0, all = 0;
  if (nblk <= RS_DIRECT) {
    for (int q0 = 0; q0 < nblk; q0 += 32) {
      int c[32];
#pragma unroll
      for (int e = 0; e < 32; ++e) c[e] = hist[(int64_t)min(q0 + e, nblk - 1) * 256 + threadIdx.x];
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        all += q0 + e < nblk ? c[e] : 0;
        before += q0 + e < (int)blockIdx.x ? c[e] : 0;
      }
    }
  } else {
    before = hist[(int64_t)blockIdx.x * 256 + threadIdx.x];
    all = threadIdx.x <= mask ? total[threadIdx.x] : 0;
  }
  __syncthreads();
  const uint64_t lt = (1ull << lane) - 1ull;
  int rank[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const bool valid = w0 + r * 64 < nvalid;
    const uint32_t d = (k[r] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < BITS; ++bit) {
      const bool one = (d >> bit) & 1u;
      const uint64_t bal = __ballot(one);
      peers &= one ? bal : ~bal;
    }
    rank[r] = s_cnt[wid][d] + __popcll(peers & lt);
    // LDS operations of a wave are in order: every lane has read its count
    __builtin_amdgcn_wave_barrier();
    if (valid && (peers >> lane) == 1ull) s_cnt[wid][d] = rank[r] + 1;  // the highest lane of its digit
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // thread d: first slot of the digit in the block, then of each wave's keys
  int c[RS_THREADS / 64], sum = 0, tot;
#pragma unroll
  for (int w = 0; w < RS_THREADS / 64; ++w) {
    c[w] = s_cnt[w][threadIdx.x];
    sum += c[w];
  }
  int slot = block_excl_scan(sum, s_w, &tot);
  s_delta[threadIdx.x] = block_excl_scan(all, s_w, &tot) + before - slot;
#pragma unroll
  for (int w = 0; w < RS_THREADS / 64; ++w) {
    s_cnt[w][threadIdx.x] = slot;
    slot += c[w];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (w0 + r * 64 < nvalid) {
      const int at = s_cnt[wid][(k[r] >> shift) & mask] + rank[r];
      s_k[at] = k[r];
      s_v[at] = v[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int i = r * RS_THREADS + threadIdx.x;
    if (i < nvalid) {
      const uint32_t key = s_k[i];
      const int at = s_delta[(key >> shift) & mask] + i;
      kout[at] = key;
      vout[at] = s_v[i];
    }
  }
}

// bits of the digit when `bits` key bits are sorted in passes of at most 8: as
// even as possible (fewer digits, longer runs to store)
static int rs_passes(int bits) { return (bits + 7) / 8; }
static int rs_digit(int bits) { return (bits + rs_passes(bits) - 1) / rs_passes(bits); }

template <int ROUNDS, int BITS = 8>
static void rs_scatter(int w, unsigned g, hipStream_t s, const uint32_t *kin, const int32_t *vin, int64_t m_cap,
                       const int32_t *m_dev, int shift, const int32_t *hist, const int32_t *total, uint32_t *kout,
                       int32_t *vout) {
  if constexpr (BITS > 4) {
    if (w < BITS)
      return rs_scatter<ROUNDS, BITS - 1>(w, g, s, kin, vin, m_cap, m_dev, shift, hist, total, kout, vout);
  }
  hipLaunchKernelGGL((k_rs_scatter<ROUNDS, BITS>), dim3(g), dim3(RS_THREADS), 0, s, kin, vin, m_cap, m_dev, shift, hist,
                     total, kout, vout);
}

template <int ROUNDS>
static void radix_passes(uint32_t **ka, int32_t **va, uint32_t **kb, int32_t **vb, int64_t m_cap, const int32_t *m_dev,
                         int bits, bool have_hist, int32_t *hist, int32_t *total, hipStream_t s) {
  const int w = rs_digit(bits) < 4 ? 4 : rs_digit(bits);  // digits below 4 bits: the key bits above are zero
  const unsigned g = grid_blocks(m_cap, RS_THREADS * ROUNDS);
  for (int p = 0; p < rs_passes(bits); ++p) {
    const int shift = p * w;
    if (p > 0 || !have_hist)
      hipLaunchKernelGGL(k_rs_hist<ROUNDS>, dim3(g), dim3(RS_THREADS), 0, s, *ka, m_cap, m_dev, shift, (1u << w) - 1u,
                         hist);
    if (g > RS_DIRECT)
      hipLaunchKernelGGL(k_rs_scan, dim3((1u << w) / 16), dim3(1024), 0, s, m_cap, m_dev, hist, total);
    rs_scatter<ROUNDS>(w, g, s, *ka, *va, m_cap, m_dev, shift, hist, total, *kb, *vb);
    std::swap(*ka, *kb);
    std::swap(*va, *vb);
  }
}

// Sorts (key, value) pairs by key bits [0, bits) stably; the result ends in
// *ka / *va (the pointers are swapped when it lands in the second buffer).
// have_hist: hist already holds the first pass's histograms (blocks of
// RS_CHUNK keys).  Inputs are cut into blocks of the fewest rounds (4, 8) that
// make at most RS_DIRECT blocks and fit the rows: their passes are a chain of
// latencies that few rounds make shorter and more blocks spread over the chip
// (a depth pass of 20k keys 13 -> 8 us; at 256k keys 125 blocks of eight rounds
// gain 1 of 16 us).
static void radix_sort(uint32_t **ka, int32_t **va, uint32_t **kb, int32_t **vb, int64_t m_cap, const int32_t *m_dev,
                       int bits, bool have_hist, int32_t *hist, int64_t rows, int32_t *total, hipStream_t s) {
  const int64_t most = have_hist ? 0 : std::min<int64_t>(RS_DIRECT, rows);
  if (grid_blocks(m_cap, RS_THREADS * 4) <= most)
    radix_passes<4>(ka, va, kb, vb, m_cap, m_dev, bits, have_hist, hist, total, s);
  else if (grid_blocks(m_cap, RS_THREADS * 8) <= most)
    radix_passes<8>(ka, va, kb, vb, m_cap, m_dev, bits, have_hist, hist, total, s);
  else
    radix_passes<RS_ROUNDS>(ka, va, kb, vb, m_cap, m_dev, bits, have_hist, hist, total, s);
}

// ---------------------------------------------------------- tile binning

// header, and the tile ranges (empty)
__global__ __launch_bounds__(256) void k_gs_begin(GsWs w, int64_t T) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < GS_HDR_INTS) w.hdr[i] = 0;
  if (i < T) w.range[i] = make_int2(0, 0);
}

__global__ void k_gs_status(const int32_t *hdr, int32_t *out) {
  if (threadIdx.x < 2) out[threadIdx.x] = hdr[threadIdx.x];
}

__device__ __forceinline__ bool gs_failed(const int32_t *hdr) { return (hdr[0] & DW_STATUS_RENDER_OVERFLOW) != 0; }

// Pairs in depth order.  Block b writes pairs [b E, (b + 1) E) of the list
// (E = GS_EMIT): two waves find the depth ranks that own its first and last
// pair (off is the exclusive scan of the tile counts in depth order; every
// drawn kernel owns at least one pair and the kernels that are not drawn sort
// last, so at most E ranks are involved); their offsets, ids and tile boxes
// are staged in LDS, each marks its first pair, and a running maximum over
// the marks gives every pair its owner.  The work per block is fixed whatever
// the kernels' sizes, so a kernel covering thousands of tiles does not hold
// up a wave, and no load waits for another pair's.  A block's slice is a
// block of the radix sort: its digit histogram for the first pass is taken
// here.
constexpr int GS_EMIT = RS_CHUNK;
constexpr int GS_EMIT_PER = GS_EMIT / 256;

// last rank whose first pair is at or before tgt, by a whole wave: 64 probes
// at a time, log64 n dependent loads instead of log2 n
__device__ __forceinline__ int rank_of_pair(const int32_t *__restrict__ off, int n, int64_t tgt, int lane) {
  int lo = 0, hi = n;  // off[lo] <= tgt (off[0] = 0), off[hi] > tgt or hi = n
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) / 64;
    const int64_t q = lo + (int64_t)step * (lane + 1);
    const int below = __popcll(__ballot(q < hi && off[q] <= tgt));  // off ascends: the first lanes
    lo += step * below;
    hi = min(hi, lo + step);
  }
  return lo;
}

__global__ __launch_bounds__(256) void k_gs_emit(int n, CamDev K, const int32_t *__restrict__ id,
                                                 const int32_t *__restrict__ off, const uint2 *__restrict__ rect,
                                                 const int32_t *hdr, uint32_t mask, uint32_t *__restrict__ pk,
                                                 int32_t *__restrict__ pv, int32_t *__restrict__ hist) {
  __shared__ int s_off[GS_EMIT], s_g[GS_EMIT];
  __shared__ uint2 s_rect[GS_EMIT];
  __shared__ __attribute__((aligned(16))) uint16_t s_own[GS_EMIT];
  __shared__ int s_h[256];
  __shared__ int s_r[2], s_w[4];
  if (gs_failed(hdr)) return;  // grid-uniform
  const int64_t total = hdr[1];
  const int64_t P0 = (int64_t)blockIdx.x * GS_EMIT;
  if (P0 >= total) return;  // block-uniform
  const int m_pairs = (int)min((int64_t)GS_EMIT, total - P0);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  s_h[threadIdx.x] = 0;
  for (int q = threadIdx.x; q < GS_EMIT / 2; q += 256) reinterpret_cast<uint32_t *>(s_own)[q] = 0u;
  if (wid < 2) {
    const int r = rank_of_pair(off, n, wid == 0 ? P0 : P0 + m_pairs - 1, lane);
    if (lane == 0) s_r[wid] = r;
  }
  __syncthreads();
  const int r_lo = s_r[0], m_ranks = s_r[1] - s_r[0] + 1;  // <= GS_EMIT
#pragma unroll 4
  for (int k = threadIdx.x; k < m_ranks; k += 256) {
    const int o = (int)(off[r_lo + k] - P0), g = id[r_lo + k];
    s_off[k] = o;
    s_g[k] = g;
    s_rect[k] = rect[g];
    if (k > 0) s_own[o] = (uint16_t)k;  // rank r_lo owns the slice's first pair
  }
  __syncthreads();
  // running maximum: 16 consecutive pairs per thread, then over the threads
  const int j0 = threadIdx.x * GS_EMIT_PER;
  int own[GS_EMIT_PER], top = 0;
#pragma unroll
  for (int q = 0; q < GS_EMIT_PER; ++q) {
    top = max(top, (int)s_own[j0 + q]);
    own[q] = top;
  }
#pragma unroll
  for (int sh = 1; sh < 64; sh <<= 1) {
    const int t = __shfl_up(top, sh, 64);
    if (lane >= sh) top = max(top, t);
  }
  if (lane == 63) s_w[wid] = top;
  int before = __shfl_up(top, 1, 64);
  if (lane == 0) before = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) before = max(before, w < wid ? s_w[w] : 0);
#pragma unroll
  for (int q = 0; q < GS_EMIT_PER; ++q) s_own[j0 + q] = (uint16_t)max(own[q], before);
  __syncthreads();
#pragma unroll 4
  for (int j = threadIdx.x; j < m_pairs; j += 256) {
    const int k = s_own[j];
    const uint2 b = s_rect[k];
    const uint32_t x0 = b.x & 0xffffu, w = (b.x >> 16) - x0 + 1u, q = (uint32_t)(j - s_off[k]);
    const uint32_t ty = q / w, t = x0 + (q - ty * w) + (uint32_t)K.tw * ((b.y & 0xffffu) + ty);
    pk[P0 + j] = t;
    pv[P0 + j] = s_g[k];
    atomicAdd(&s_h[t & mask], 1);
  }
  __syncthreads();
  hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = s_h[threadIdx.x];
}

// grid-stride over the pairs actually present (the grid is sized for a
// typical count, not for the capacity), four per thread: a pair whose tile
// differs from its predecessor's ends that tile's range and starts its own
__global__ __launch_bounds__(256) void k_gs_ranges(const uint32_t *__restrict__ pk, const int32_t *__restrict__ hdr,
                                                   int2 *__restrict__ range) {
  const int64_t m = hdr[1];
  for (int64_t i = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x); i < m; i += 1024 * (int64_t)gridDim.x) {
    uint4 q = i + 4 <= m ? *reinterpret_cast<const uint4 *>(pk + i)
                         : make_uint4(pk[i], i + 1 < m ? pk[i + 1] : 0u, i + 2 < m ? pk[i + 2] : 0u, 0u);
    const uint32_t t[4] = {q.x, q.y, q.z, q.w};
    uint32_t prev = i > 0 ? pk[i - 1] : 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k >= m) break;
      if (i + k == 0 || t[k] != prev) {
        range[t[k]].x = (int)(i + k);
        if (i + k > 0) range[prev].y = (int)(i + k);
      }
      if (i + k == m - 1) range[t[k]].y = (int)m;
      prev = t[k];
    }
  }
}

// ------------------------------------------------------------- raster

struct GsRec {
  float mx, my, A, B, C, o, c0, c1, c2;
};

// alpha of kernel r at pixel centre (x, y); the same expression in the
// forward and reverse passes, so both take the same alpha_min decisions
__device__ __forceinline__ float gs_alpha(const GsRec &r, float x, float y, float &e) {
  const float dx = x - r.mx;
  const float dy = y - r.my;
  const float q = r.A * dx * dx + 2.0f * r.B * dx * dy + r.C * dy * dy;
  e = __expf(-0.5f * q);
  return r.o * e;
}

typedef float gs_floatx4 __attribute__((ext_vector_type(4)));

template <int N>
struct GsBatch {
  float4 a[N];  // mx, my, A, B
  float2 b[N];  // C, o
  float4 rgb[N];
  uint2 box[N];
  // per wave: entries of the batch that meet its pixels
  __attribute__((aligned(16))) uint8_t list[GS_THREADS / 64][N];
};

// The list of one tile, a batch of N at a time; with AHEAD the records of the
// next batch and the ids of the one after are requested while a batch is
// blended.  Without, the first batch is half a batch long and nothing but ids
// is requested early: where large kernels cover a tile its pixels are opaque
// after some hundred entries of a list of thousands.
template <int N, bool AHEAD>
struct GsFeed {
  const int32_t *pv;
  const float4 *rec;
  int pos, len, end;  // list position and length of the batch to stage
  int id, id_next;
  gs_floatx4 r0, r1, r2;

  __device__ __forceinline__ int entry(int p) { return (int)threadIdx.x < N && p < end ? pv[p] : 0; }
  __device__ __forceinline__ void load_rec() {
    // threads past the batch read kernel 0's record and do not store it
    const gs_floatx4 *p = reinterpret_cast<const gs_floatx4 *>(rec + 3 * (int64_t)((int)threadIdx.x < len ? id : 0));
    r0 = p[0];
    r1 = p[1];
    r2 = p[2];
  }
  __device__ __forceinline__ GsFeed(const int32_t *pv_, const float4 *rec_, int first, int end_)
      : pv(pv_), rec(rec_), pos(first), end(end_) {
    len = min(AHEAD ? N : N / 2, end - pos);
    id = entry(pos + threadIdx.x);
    id_next = entry(pos + len + threadIdx.x);
    if (AHEAD) load_rec();
  }
  __device__ __forceinline__ bool more() const { return pos < end; }
  // puts the batch into LDS
  __device__ __forceinline__ void stage(GsBatch<N> &s, int *s_id) {
    const int t = threadIdx.x;
    if (!AHEAD) load_rec();
    if (t < len) {
      s.a[t] = make_float4(r0.x, r0.y, r0.z, r0.w);
      s.b[t] = make_float2(r1.x, r1.y);
      s.rgb[t] = make_float4(r1.z, r1.w, r2.x, 0.f);
      s.box[t] = make_uint2(__float_as_uint(r2.y), __float_as_uint(r2.z));
      if (s_id) s_id[t] = id;
    }
  }
  // moves on to the next batch and requests what belongs to it
  __device__ __forceinline__ void advance() {
    pos += len;
    len = min(N, end - pos);
    id = id_next;
    if (AHEAD) load_rec();
    id_next = entry(pos + len + threadIdx.x);
  }
};

// entries of the batch whose pixel box meets pixels [wx, wx + ext] x [wy, wy + ext],
// in order, into the wave's list; returns their number.  hits (optional): the
// mask of the entries taken, 64 to a word
template <int N>
__device__ __forceinline__ int gs_pick(GsBatch<N> &s, int wid, int lane, int n, int wx, int wy, int ext,
                                       uint64_t *hits = nullptr) {
  int cnt = 0;
  for (int c = 0; c < n; c += 64) {
    const int j = c + lane;
    bool hit = false;
    if (j < n) {
      const uint2 b = s.box[j];
      hit = (int)(b.x & 0xffffu) <= wx + ext && (int)(b.x >> 16) >= wx && (int)(b.y & 0xffffu) <= wy + ext &&
            (int)(b.y >> 16) >= wy;
    }
    const uint64_t m = __ballot(hit);
    if (hit) s.list[wid][cnt + __popcll(m & ((1ull << lane) - 1ull))] = (uint8_t)j;
    if (hits && lane == 0) hits[c >> 6] = m;
    cnt += __popcll(m);
  }
  __builtin_amdgcn_wave_barrier();  // other lanes of this wave read the list back (LDS is in order)
  return cnt;
}

template <int N>
__device__ __forceinline__ GsRec gs_entry(const GsBatch<N> &s, int j) {
  const float4 a = s.a[j], c = s.rgb[j];
  const float2 b = s.b[j];
  return GsRec{a.x, a.y, a.z, a.w, b.x, b.y, c.x, c.y, c.z};
}

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float old, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sorts the tiles into those that one workgroup rasterises and those that
// four do (k_gs_raster says how): long lists of small kernels, judged by the
// 4 x 4 pixel blocks of the tile that 16 entries from the list's first 1024
// meet.  Four lanes per tile, one atomic per class and 64 tiles (an atomic
// per tile took 53 us at 4096 tiles).  The order inside the lists does not
// matter.
constexpr int GS_SPLIT_LEN = 192, GS_SPLIT_BLOCKS = 6;

__global__ __launch_bounds__(256) void k_gs_classify(CamDev K, GsWs w, const int32_t *__restrict__ pv) {
  __shared__ int s_n[2], s_at[2];
  if (gs_failed(w.hdr)) return;
  const int tile = blockIdx.x * 64 + (threadIdx.x >> 2), sub = threadIdx.x & 3;
  if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
  __syncthreads();
  const bool has = tile < K.tw * K.th;
  int len = 0, blocks = 0;
  if (has) {
    const int2 rg = w.range[tile];
    len = rg.y - rg.x;
    if (len > GS_SPLIT_LEN) {
      const int X0 = (tile % K.tw) * GS_TILE, Y0 = (tile / K.tw) * GS_TILE;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 r2 = w.rec[3 * (int64_t)pv[rg.x + (4 * k + sub) * min(len, 1024) / 16] + 2];
        const uint32_t bx = __float_as_uint(r2.y), by = __float_as_uint(r2.z);
        const int nx = (min((int)(bx >> 16) - X0, GS_TILE - 1) >> 2) - (max((int)(bx & 0xffffu) - X0, 0) >> 2) + 1;
        const int ny = (min((int)(by >> 16) - Y0, GS_TILE - 1) >> 2) - (max((int)(by & 0xffffu) - Y0, 0) >> 2) + 1;
        blocks += nx * ny;
      }
    }
  }
  blocks += __shfl_xor(blocks, 1, 64);
  blocks += __shfl_xor(blocks, 2, 64);
  const int split = len > GS_SPLIT_LEN && blocks < 16 * GS_SPLIT_BLOCKS ? 1 : 0;
  const int at = has && sub == 0 ? atomicAdd(&s_n[split], 1) : 0;
  __syncthreads();
  if (threadIdx.x < 2) s_at[threadIdx.x] = atomicAdd(&w.hdr[2 + threadIdx.x], s_n[threadIdx.x]);
  __syncthreads();
  if (has && sub == 0) (split ? w.split : w.whole)[s_at[split] + at] = tile;
}

// One workgroup per tile, a wave per 8 x 8 pixels, one pixel per lane.  The
// four alphas of a step are independent and hide each other's latency, only
// the blending is a chain.
__device__ __forceinline__ void gs_raster_whole(const CamDev &K, GsBatch<GS_THREADS> &s, int tile, int2 rg,
                                                const int32_t *__restrict__ pv, const float4 *__restrict__ rec,
                                                float *__restrict__ image, int32_t *__restrict__ last) {
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wx = (tile % K.tw) * GS_TILE + 8 * (wid & 1), wy = (tile / K.tw) * GS_TILE + 8 * (wid >> 1);
  const int i = wx + (lane & 7), j = wy + (lane >> 3);
  const bool inside = i < K.W && j < K.H;
  const float x = i + 0.5f, y = j + 0.5f;
  float T = 1.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
  bool live = inside;
  int used = rg.y - rg.x;
  GsFeed<GS_THREADS, false> feed(pv, rec, rg.x, rg.y);
  while (feed.more()) {
    const bool done = __ballot(live) == 0ull;
    if (__syncthreads_and(done)) break;
    feed.stage(s, nullptr);
    __syncthreads();
    const int first = feed.pos - rg.x;
    if (!done) {
      const int cnt = gs_pick(s, wid, lane, feed.len, wx, wy, 7);
      for (int q = 0; q < cnt; q += 4) {
        const uint32_t four = __builtin_amdgcn_readfirstlane(*reinterpret_cast<const uint32_t *>(&s.list[wid][q]));
        GsRec r[4];
        float al[4], e;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          r[u] = gs_entry(s, (four >> (8 * u)) & 255u);
          al[u] = gs_alpha(r[u], x, y, e);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (live && q + u < cnt && al[u] >= K.amin) {
            const float wgt = T * al[u];
            c0 += wgt * r[u].c0;
            c1 += wgt * r[u].c1;
            c2 += wgt * r[u].c2;
            T *= 1.0f - al[u];
            if (T < K.tmin) {
              live = false;
              used = first + (int)((four >> (8 * u)) & 255u) + 1;
            }
          }
        }
        if (__ballot(live) == 0ull) break;
      }
    }
    feed.advance();
  }
  if (!inside) return;
  const int64_t pix = i + (int64_t)K.W * j, HW = (int64_t)K.W * K.H;
  image[pix] = c0 + T * K.bg[0];
  image[HW + pix] = c1 + T * K.bg[1];
  image[2 * HW + pix] = c2 + T * K.bg[2];
  last[pix] = used;
}

// One workgroup per 8 x 8 pixels, a wave per 4 x 4: lane l holds pixel l / 4
// and entry l % 4 of a step, so four alphas of every pixel are one
// evaluation; the lanes of a pixel then take the four entries' alphas from
// each other in order, lane c < 3 blending channel c.
__device__ __forceinline__ void gs_raster_split(const CamDev &K, GsBatch<GS_THREADS> &s, int tile, int quarter, int2 rg, bool strict,
                                                const int32_t *__restrict__ pv, const float4 *__restrict__ rec,
                                                float *__restrict__ image, int32_t *__restrict__ last) {
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wx = (tile % K.tw) * GS_TILE + 8 * (quarter & 1) + 4 * (wid & 1);
  const int wy = (tile / K.tw) * GS_TILE + 8 * (quarter >> 1) + 4 * (wid >> 1);
  const int e = lane & 3, i = wx + ((lane >> 2) & 3), j = wy + (lane >> 4);
  const bool inside = i < K.W && j < K.H;
  const float x = i + 0.5f, y = j + 0.5f;
  // T: the transmittance while the pixel blends, then 0; Tend: what it was
  // when the pixel stopped (so T + Tend is the final one)
  float T = inside ? 1.f : 0.f, Tend = 0.f, c = 0.f;
  int used = 0;
  bool on = inside;
  GsFeed<GS_THREADS, true> feed(pv, rec, rg.x, rg.y);
  while (feed.more()) {
    const bool done = __ballot(on) == 0ull;
    if (__syncthreads_and(done)) break;
    feed.stage(s, nullptr);
    __syncthreads();
    const int first = feed.pos - rg.x + 1, n = feed.len;
    feed.advance();
    if (done) continue;
    const int cnt = gs_pick(s, wid, lane, n, wx, wy, 3);
    struct Step {
      uint32_t four;
      float4 ra;
      float2 rb;
      float col[4];
    };
    auto fetch = [&](int q) {
      Step f;
      f.four = __builtin_amdgcn_readfirstlane(*reinterpret_cast<const uint32_t *>(&s.list[wid][q]));
      const int m = (f.four >> (8 * e)) & 255u;
      f.ra = s.a[m];
      f.rb = s.b[m];
#pragma unroll
      for (int u = 0; u < 4; ++u) f.col[u] = reinterpret_cast<const float *>(&s.rgb[(f.four >> (8 * u)) & 255u])[e];
      return f;
    };
    Step nx = fetch(0);
    for (int q = 0; q < cnt; q += 4) {
      const Step f = nx;
      nx = fetch(min(q + 4, GS_THREADS - 4));
      const GsRec r{f.ra.x, f.ra.y, f.ra.z, f.ra.w, f.rb.x, f.rb.y, 0.f, 0.f, 0.f};
      float ex;
      const float al = gs_alpha(r, x, y, ex);
      const float a = q + e < cnt && al >= K.amin ? al : -1.f;
      // the four entries one after another, each alpha from its lane of the pixel
      const float a0 = dpp_mov<0x00>(a, a), a1 = dpp_mov<0x55>(a, a), a2 = dpp_mov<0xAA>(a, a), a3 = dpp_mov<0xFF>(a, a);
      const float v0 = fmaxf(a0, 0.f), v1 = fmaxf(a1, 0.f), v2 = fmaxf(a2, 0.f), v3 = fmaxf(a3, 0.f);
      const float T1 = T * (1.0f - v0), T2 = T1 * (1.0f - v1), T3 = T2 * (1.0f - v2), T4 = T3 * (1.0f - v3);
      if (!strict && __ballot(on && !(T4 >= K.tmin)) == 0ull) {
        // no pixel of the wave stops in this step (and an alpha of zero adds
        // nothing: the colours are finite)
        c += (T * v0) * f.col[0];
        c += (T1 * v1) * f.col[1];
        c += (T2 * v2) * f.col[2];
        c += (T3 * v3) * f.col[3];
        T = T4;
        used = on ? first + (int)((f.four >> (8 * min(3, cnt - 1 - q))) & 255u) : used;
        continue;
      }
      auto blend = [&](float au, float col, int u) {
        const bool hit = au >= 0.f;
        const float av = fmaxf(au, 0.f);
        const float cn = c + (T * av) * col, Tn = T * (1.0f - av);
        c = hit && on ? cn : c;
        used = on && q + u < cnt ? first + (int)((f.four >> (8 * u)) & 255u) : used;
        on = on && Tn >= K.tmin;
        T = on ? Tn : 0.f;
        Tend += on ? 0.f : Tn;
      };
      blend(a0, f.col[0], 0);
      blend(a1, f.col[1], 1);
      blend(a2, f.col[2], 2);
      blend(a3, f.col[3], 3);
      if (__ballot(on) == 0ull) break;
    }
  }
  if (!inside) return;
  T += Tend;
  const int64_t pix = i + (int64_t)K.W * j, HW = (int64_t)K.W * K.H;
  if (e < 3) image[e * HW + pix] = c + T * (e == 0 ? K.bg[0] : e == 1 ? K.bg[1] : K.bg[2]);
  else last[pix] = used;
}

// Work items of both raster passes: the quarters of the split tiles, then
// the whole tiles; a workgroup starts with the item of its index and draws
// further ones from a ticket.  One workgroup per tile costs the least work
// in all, but its waves walk the whole list: views whose lists hold
// thousands of small kernels on a few tiles leave the chip idle behind them.
// There a wave of 4 x 4 pixels skips four entries of five and takes the rest
// four at a time.  The forward pass blends a pixel's entries one after
// another in list order either way.  Forward, against one thread per pixel
// walking the list entry by entry: 256k kernels on 247 tiles of a 512^2 view
// (lists up to 7,500) 672 -> 97 us, 20k on 44 tiles 245 -> 44 us, 1M kernels
// on 4096 tiles of which a pixel sees some hundred 78 -> 87 us.
struct GsItem {
  int tile, quarter;  // quarter < 0: the whole tile
};

__device__ __forceinline__ GsItem gs_item(const GsWs &w, int it, int nsplit) {
  if (it >= 4 * nsplit) return GsItem{w.whole[it - 4 * nsplit], -1};
  // the quarters of a tile to one XCD (workgroups are handed out round-robin
  // over 8), where they share its list
  const int group = it >> 5, in = min(8, nsplit - 8 * group), r = it & 31;
  return GsItem{w.split[8 * group + r % in], r / in};
}

// workgroups of a raster launch: enough to fill the chip six times per CU
// with quarters, at least one per tile
static unsigned gs_raster_blocks(int64_t T) {
  const int64_t most = T > 1536 ? T : 1536;
  return (unsigned)(4 * T < most ? 4 * T : most);
}

__global__ __launch_bounds__(GS_THREADS) void k_gs_raster(CamDev K, GsWs w, const int32_t *__restrict__ pv,
                                                         float *__restrict__ image) {
  __shared__ GsBatch<GS_THREADS> s;
  __shared__ int s_item;
  if (gs_failed(w.hdr)) return;  // over capacity: the image is not written
  const int nsplit = w.hdr[3], items = 4 * nsplit + w.hdr[2];
  int it = blockIdx.x;
  while (it < items) {
    const GsItem t = gs_item(w, it, nsplit);
    const int2 rg = w.range[t.tile];
    if (t.quarter < 0) gs_raster_whole(K, s, t.tile, rg, pv, w.rec, image, w.last);
    else gs_raster_split(K, s, t.tile, t.quarter, rg, w.hdr[6] != 0, pv, w.rec, image, w.last);
    if (items <= (int)gridDim.x) return;
    __syncthreads();
    if (threadIdx.x == 0) s_item = (int)gridDim.x + atomicAdd(&w.hdr[4], 1);
    __syncthreads();
    it = s_item;
  }
}

// ------------------------------------------------------- raster reverse

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Inclusive scans over the 16 lanes of every DPP row, four values at a time:
// step s combines a lane with the lane s below it; lanes without one are not
// written.  A DPP operand must be two wait states old: the s_nop covers the
// inputs, the three other chains every later step.
#define GS_SCAN4(OP, S)                                         \
  OP " %0, %0, %0 row_shr:" S " row_mask:0xf bank_mask:0xf\n\t" \
  OP " %1, %1, %1 row_shr:" S " row_mask:0xf bank_mask:0xf\n\t" \
  OP " %2, %2, %2 row_shr:" S " row_mask:0xf bank_mask:0xf\n\t" \
  OP " %3, %3, %3 row_shr:" S " row_mask:0xf bank_mask:0xf\n\t"

__device__ __forceinline__ void row_scan_mul4(float (&v)[4]) {
  asm volatile("s_nop 1\n\t" GS_SCAN4("v_mul_f32_dpp", "1") GS_SCAN4("v_mul_f32_dpp", "2") GS_SCAN4("v_mul_f32_dpp", "4")
                   GS_SCAN4("v_mul_f32_dpp", "8")
               : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}
__device__ __forceinline__ void row_scan_add4(float (&v)[4]) {
  asm volatile("s_nop 1\n\t" GS_SCAN4("v_add_f32_dpp", "1") GS_SCAN4("v_add_f32_dpp", "2") GS_SCAN4("v_add_f32_dpp", "4")
                   GS_SCAN4("v_add_f32_dpp", "8")
               : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}
#undef GS_SCAN4

// value of the lane below in the row (old in the row's first lane), and of
// the row's last lane
__device__ __forceinline__ float row_below(float old, float v) { return dpp_mov<0x111>(old, v); }
__device__ __forceinline__ float row_last(float v) { return dpp_mov<0x15F>(v, v); }

// Sums of a, b, c, d over the four rows of 16 lanes: row 0 gets a's, row 1 c's,
// row 2 b's, row 3 d's.  A swap exchanges half of one register with half of
// another, so that one addition serves two values.
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float row_sums(float a, float b, float c, float d) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(swap32_add(a, b)), __float_as_uint(swap32_add(c, d)),
                                                  false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 1 / m to about one rounding: the hardware reciprocal and a Newton step
__device__ __forceinline__ float recip(float m) {
  const float r = __builtin_amdgcn_rcpf(m);
  return fmaf(r, fmaf(-m, r, 1.0f), r);
}

// A wave evaluates 16 entries x 4 x 4 pixels at a time: lane l holds entry
// l % 16 and pixel column l / 16, the four pixel rows are four registers.
// The transmittance in front of an entry and P are scans over the 16 lanes of
// a DPP row, so the chain that a pixel's list imposes advances 16 entries at
// a time, and a wave only takes the entries whose pixel box meets its pixels
// (for kernels of a few pixels about a fifth of the tile's list).  In a
// quarter a wave has 4 x 4 pixels, in a whole tile 8 x 8 as four blocks per
// group of entries; the pixels' state waits in LDS meanwhile.
// An entry's sums over the pixel rows (the column's dx is one number) and over
// a tile's four blocks are taken in its lanes, those over the four columns by
// eight half-register swaps and additions.  (Moments about a
// block's centre, moved to the kernel afterwards, need one sum less and lose
// digits to cancellation where a kernel is smaller than a pixel.)  Every wave
// leaves its sums in an LDS table of its own (an entry comes up once per wave
// and batch: plain stores); for a whole tile the workgroup adds the tables of
// the waves that met an entry.  One float atomic per value goes to memory,
// the nine of a kernel side by side in one request.  (Float atomics in LDS
// took 375 us at 1M kernels and 1024^2 pixels, one global atomic per wave and
// value 532 us.)
// Against one wave per tile walking the list entry by entry: 256k kernels,
// 512^2 3,016 -> 108 us, 20k 1,768 -> 48 us, 1M kernels, 1024^2 357 -> 175 us,
// where the vector units are busy 84 % of the time (220 with nine MFMAs with
// ones for the column sums of every block, 182 with nine per group).
constexpr int GS_ADJ_N = 128;  // list entries per batch
struct GsPixel {
  float T, P, G0, G1, G2, gC;
  int used;
  float pad;
};

__global__ __launch_bounds__(GS_THREADS, 4) void k_gs_raster_adj(CamDev K, GsWs w, const int32_t *__restrict__ pv,
                                                                const float *__restrict__ image,
                                                                const float *__restrict__ image_bar) {
  __shared__ GsBatch<GS_ADJ_N> s;
  __shared__ __attribute__((aligned(16))) GsPixel px[GS_THREADS];
  __shared__ float s_sum[GS_THREADS / 64][GS_ADJ_N * GS_NB];
  __shared__ uint64_t s_hits[GS_THREADS / 64][GS_ADJ_N / 64];
  __shared__ int s_id[GS_ADJ_N];
  __shared__ int s_most, s_item;
  if (gs_failed(w.hdr)) return;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e = lane & 15, g = lane >> 4;
  const int64_t HW = (int64_t)K.W * K.H;
  const int nsplit = w.hdr[3], items = 4 * nsplit + w.hdr[2];
  int it = blockIdx.x;
  while (it < items) {
    const GsItem t = gs_item(w, it, nsplit);
    const int2 rg = w.range[t.tile];
    const int X0 = (t.tile % K.tw) * GS_TILE, Y0 = (t.tile / K.tw) * GS_TILE;
    const bool whole = t.quarter < 0;
    if (threadIdx.x == 0) s_most = 0;
    __syncthreads();
    if (whole || threadIdx.x < 64) {
      // one pixel per thread (a quarter's 64 by the first wave)
      const int n = threadIdx.x;
      const int lx = whole ? n & 15 : 8 * (t.quarter & 1) + (n & 7);
      const int ly = whole ? n >> 4 : 8 * (t.quarter >> 1) + (n >> 3);
      const int i = X0 + lx, j = Y0 + ly;
      const bool inside = i < K.W && j < K.H;
      const int64_t pix = i + (int64_t)K.W * j;
      GsPixel q;
      q.T = 1.f;
      q.P = 0.f;
      q.G0 = inside ? image_bar[pix] : 0.f;
      q.G1 = inside ? image_bar[HW + pix] : 0.f;
      q.G2 = inside ? image_bar[2 * HW + pix] : 0.f;
      q.gC = inside ? q.G0 * image[pix] + q.G1 * image[HW + pix] + q.G2 * image[2 * HW + pix] : 0.f;
      q.used = inside ? w.last[pix] : 0;
      q.pad = 0.f;
      px[ly * GS_TILE + lx] = q;
      // the furthest pixel bounds the traversal
      int most = q.used;
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) most = max(most, __shfl_xor(most, m, 64));
      if (lane == 0) atomicMax(&s_most, most);
    }
    __syncthreads();
    GsFeed<GS_ADJ_N, true> feed(pv, w.rec, rg.x, rg.x + s_most);
    const int nblk = whole ? 4 : 1;
    const int lx = whole ? 8 * (wid & 1) : 8 * (t.quarter & 1) + 4 * (wid & 1);
    const int ly = whole ? 8 * (wid >> 1) : 8 * (t.quarter >> 1) + 4 * (wid >> 1);
    while (feed.more()) {
      const int first = feed.pos - rg.x, n = feed.len;
      feed.stage(s, s_id);
      __syncthreads();
      feed.advance();
      const int cnt = gs_pick(s, wid, lane, n, X0 + lx, Y0 + ly, whole ? 7 : 3, s_hits[wid]);
      for (int q = 0; q < cnt; q += 16) {
        const bool has = q + e < cnt;
        const int j = has ? (int)s.list[wid][q + e] : 0;
        const GsRec r = gs_entry(s, j);
        const int idx = has ? first + j : INT_MAX;
        float m[GS_NB];  // the lane's sums over its pixels of all blocks
#pragma unroll
        for (int k = 0; k < GS_NB; ++k) m[k] = 0.f;
        for (int b = 0; b < nblk; ++b) {
          const int bx = lx + 4 * (b & 1), by = ly + 4 * (b >> 1);
          const float x0 = (float)(X0 + bx), y0 = (float)(Y0 + by);
          const float x = x0 + (float)g + 0.5f, y = y0 + 0.5f;
          float ex[4], al[4], z[4], sc[4], v[4], wg[4], Tx[4], T[4], P[4], G[4][3], gC[4];
          bool on[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const gs_floatx4 *pq = reinterpret_cast<const gs_floatx4 *>(&px[(by + p) * GS_TILE + bx + g]);
            const gs_floatx4 u0 = pq[0], u1 = pq[1];
            T[p] = u0.x;
            P[p] = u0.y;
            gC[p] = u1.y;
            const float a = gs_alpha(r, x, y + (float)p, ex[p]);
            on[p] = idx < __float_as_int(u1.z) && a >= K.amin;
            al[p] = on[p] ? a : 0.f;
            z[p] = 1.0f - al[p];
            G[p][0] = u0.z;
            G[p][1] = u0.w;
            G[p][2] = u1.x;
            sc[p] = G[p][0] * r.c0 + G[p][1] * r.c1 + G[p][2] * r.c2;
          }
          if (__ballot(on[0] || on[1] || on[2] || on[3]) == 0ull) continue;
          row_scan_mul4(z);
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const float Ti = T[p] * z[p];
            Tx[p] = row_below(T[p], Ti);
            T[p] = row_last(Ti);
            wg[p] = Tx[p] * al[p];
            v[p] = on[p] ? wg[p] * sc[p] : 0.f;
          }
          row_scan_add4(v);
          const float dx = x - r.mx;
          float d0 = 0.f, d1 = 0.f;  // sums of e and e dy
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const float Pi = P[p] + v[p];
            P[p] = row_last(Pi);
            const float dal = Tx[p] * sc[p] - (gC[p] - Pi) * recip(1.0f - al[p]);
            const float de = on[p] ? dal * ex[p] : 0.f, dy = y + (float)p - r.my;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) m[ch] += wg[p] * G[p][ch];
            d0 += de;
            d1 += de * dy;
            m[7] += de * dy * dy;
          }
          m[3] += d0;
          m[4] += d0 * dx;
          m[5] += d0 * dx * dx;
          m[6] += d1 * dx;
          m[8] += d1;
          if (e == 0) {
#pragma unroll
            for (int p = 0; p < 4; ++p)
              *reinterpret_cast<float2 *>(&px[(by + p) * GS_TILE + bx + g]) = make_float2(T[p], P[p]);
          }
        }
        // sums over the four columns: value at[k] of the lane's entry
        const float low = row_sums(m[0], m[1], m[2], m[3]), high = row_sums(m[4], m[5], m[6], m[7]),
                    top = row_sums(m[8], 0.f, 0.f, 0.f);
        const int at = ((g & 1) << 1) | (g >> 1);
        float *dst = s_sum[wid] + (whole ? j : e) * GS_NB;
        if (has || !whole) {
          dst[at] = low;
          dst[4 + at] = high;
          if (g == 0) dst[8] = top;
        }
        if (!whole) {
          // few waves meet an entry: straight to memory, 64 consecutive of the
          // group's 16 x 9 values at a time
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const int i = k * 64 + lane, m = i / GS_NB;
            if (m < 16 && q + m < cnt) {
              const float v = s_sum[wid][i];
              if (v != 0.f) atomicAdd(w.gbar + (int64_t)s_id[s.list[wid][q + m]] * GS_NB + i % GS_NB, v);
            }
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
      if (!whole) {
        __syncthreads();  // the next batch replaces the ids and the records
        continue;
      }
      __syncthreads();
      // 16 lanes per entry, nine of them with a value
      for (int j = threadIdx.x >> 4; j < n; j += GS_THREADS / 16) {
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < GS_THREADS / 64; ++v)
          if (e < GS_NB && (s_hits[v][j >> 6] >> (j & 63) & 1u)) sum += s_sum[v][j * GS_NB + e];
        if (sum != 0.f) atomicAdd(w.gbar + (int64_t)s_id[j] * GS_NB + e, sum);
      }
      __syncthreads();  // the next batch replaces the ids and the records
    }
    if (items <= (int)gridDim.x) return;
    if (threadIdx.x == 0) s_item = (int)gridDim.x + atomicAdd(&w.hdr[5], 1);
    __syncthreads();
    it = s_item;
  }
}

__global__ __launch_bounds__(256) void k_gs_adj_begin(GsWs w, int64_t count) {
  if (blockIdx.x == 0 && threadIdx.x == 0) w.hdr[5] = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
    reinterpret_cast<float4 *>(w.gbar)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Centre and conic adjoints back to mu and Sigma through the projection.
// conic K = Sigma2^-1: Sigma2_bar = -K Kbar K (Kbar the symmetric matrix of
// the conic adjoint, off-diagonal B_bar / 2); Sigma2 = T Sigma T^T with T = J R:
// Sigma_bar = T^T Sigma2_bar T, T_bar = 2 Sigma2_bar T Sigma; J_bar = T_bar R^T
// and the centre adjoint go to the camera point p, and mu_bar = R^T p_bar.
__global__ __launch_bounds__(256) void k_gs_project_adj(CamDev K, int n, const float *__restrict__ mu,
                                                        const float *__restrict__ sigma, const float *__restrict__ op,
                                                        const float *__restrict__ gbar, float *__restrict__ mu_bar,
                                                        float *__restrict__ sigma_bar, float *__restrict__ color_bar,
                                                        float *__restrict__ opacity_bar) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  float b[GS_NB];
  bool any = false;
#pragma unroll
  for (int v = 0; v < GS_NB; ++v) {
    b[v] = gbar[(int64_t)g * GS_NB + v];
    any = any || b[v] != 0.f;
  }
  if (!any) return;
  if (color_bar) {
#pragma unroll
    for (int c = 0; c < 3; ++c) color_bar[c * (int64_t)n + g] += b[c];
  }
  if (opacity_bar) opacity_bar[g] += b[3];
  float S[6];
#pragma unroll
  for (int e = 0; e < 6; ++e) S[e] = sigma[(int64_t)e * n + g];
  const Proj r = gs_proj(K, mu[g], mu[(int64_t)n + g], mu[2 * (int64_t)n + g], S, op[g]);
  if (!r.drawn) return;
  // alpha = o exp(-q/2), q = A dx^2 + 2 B dx dy + C dy^2 with d = x - m:
  // q_bar = -o/2 e, A_bar = sum q_bar dx^2, m_bar = -2 K sum q_bar d
  const float h = -0.5f * op[g];
  const float mxb = -2.0f * h * (r.A * b[4] + r.B * b[8]), myb = -2.0f * h * (r.B * b[4] + r.C * b[8]);
  const float Ab = h * b[5], Bb = 2.0f * h * b[6], Cb = h * b[7];
  if (mxb == 0.f && myb == 0.f && Ab == 0.f && Bb == 0.f && Cb == 0.f) return;
  // Sigma2_bar = -K Kbar K, K = [[A, B], [B, C]], Kbar = [[Ab, Bb/2], [Bb/2, Cb]]
  const float kb01 = 0.5f * Bb;
  const float m00 = r.A * Ab + r.B * kb01, m01 = r.A * kb01 + r.B * Cb;  // K Kbar
  const float m10 = r.B * Ab + r.C * kb01, m11 = r.B * kb01 + r.C * Cb;
  const float s00 = -(m00 * r.A + m01 * r.B), s01 = -(m00 * r.B + m01 * r.C);
  const float s11 = -(m10 * r.B + m11 * r.C);
  // Sigma_bar = T^T Sigma2_bar T (symmetric); stored off-diagonals count twice
  float Sb[9];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      Sb[3 * a + c] = r.T0[a] * (s00 * r.T0[c] + s01 * r.T1[c]) + r.T1[a] * (s01 * r.T0[c] + s11 * r.T1[c]);
  if (sigma_bar) {
    sigma_bar[g] += Sb[0];
    sigma_bar[(int64_t)n + g] += Sb[4];
    sigma_bar[2 * (int64_t)n + g] += Sb[8];
    sigma_bar[3 * (int64_t)n + g] += Sb[1] + Sb[3];
    sigma_bar[4 * (int64_t)n + g] += Sb[2] + Sb[6];
    sigma_bar[5 * (int64_t)n + g] += Sb[5] + Sb[7];
  }
  if (!mu_bar) return;
  // T_bar = 2 Sigma2_bar T Sigma (rows 0, 1)
  const float Sm[9] = {S[0], S[3], S[4], S[3], S[1], S[5], S[4], S[5], S[2]};
  float TS0[3], TS1[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    TS0[c] = r.T0[0] * Sm[c] + r.T0[1] * Sm[3 + c] + r.T0[2] * Sm[6 + c];
    TS1[c] = r.T1[0] * Sm[c] + r.T1[1] * Sm[3 + c] + r.T1[2] * Sm[6 + c];
  }
  float Tb0[3], Tb1[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    Tb0[c] = 2.0f * (s00 * TS0[c] + s01 * TS1[c]);
    Tb1[c] = 2.0f * (s01 * TS0[c] + s11 * TS1[c]);
  }
  // J_bar = T_bar R^T; only J00, J02, J11, J12 are non-zero functions of p
  const float jb00 = Tb0[0] * K.R[0] + Tb0[1] * K.R[1] + Tb0[2] * K.R[2];
  const float jb02 = Tb0[0] * K.R[6] + Tb0[1] * K.R[7] + Tb0[2] * K.R[8];
  const float jb11 = Tb1[0] * K.R[3] + Tb1[1] * K.R[4] + Tb1[2] * K.R[5];
  const float jb12 = Tb1[0] * K.R[6] + Tb1[1] * K.R[7] + Tb1[2] * K.R[8];
  const float iz = 1.0f / r.pz, iz2 = iz * iz, iz3 = iz2 * iz;
  // J00 = fx/z, J02 = -fx px/z^2, J11 = fy/z, J12 = -fy py/z^2;
  // mx = fx px/z + cx, my = fy py/z + cy
  const float pxb = -K.fx * iz2 * jb02 + K.fx * iz * mxb;
  const float pyb = -K.fy * iz2 * jb12 + K.fy * iz * myb;
  const float pzb = -K.fx * iz2 * jb00 + 2.0f * K.fx * r.px * iz3 * jb02 - K.fy * iz2 * jb11 +
                    2.0f * K.fy * r.py * iz3 * jb12 - K.fx * r.px * iz2 * mxb - K.fy * r.py * iz2 * myb;
  // mu_bar = R^T p_bar
#pragma unroll
  for (int a = 0; a < 3; ++a)
    mu_bar[(int64_t)a * n + g] += K.R[a] * pxb + K.R[3 + a] * pyb + K.R[6 + a] * pzb;
}

// ------------------------------------------------------------- loss

constexpr int SS_T = 16;               // output tile of the SSIM kernels
constexpr int SS_R = 5;                // window radius (11 x 11)
constexpr int SS_E = SS_T + 2 * SS_R;  // staged extent
constexpr int SS_ROWS = SS_T * SS_T / 32;  // rows that pass 1 stages at a time, half a wave each
// Pitch of the staged rows: the four rows of 16 columns that a wave reads in
// the horizontal pass then lie in different banks (1M pixels: 48 -> 45 us and
// 43 -> 39 us against a pitch of 26).
constexpr int SS_P = 48;
constexpr float SS_C1 = 0.01f * 0.01f, SS_C2 = 0.03f * 0.03f;

// Normalised 1-D Gaussian of sigma 1.5, taps -5 .. 5 (the 2-D window is its
// outer product): exp(-k^2 / 4.5) over the sum of the eleven as 32-bit
// arithmetic on the device gives them (their sum is 1 + 4.5e-8).  Constants: no
// wave waits for their evaluation, no tap reads one from LDS (three channels of
// 1024^2: pass 1 53 -> 51 us, pass 2 46 -> 43).
constexpr float SS_W[2 * SS_R + 1] = {0x1.0d957p-10f, 0x1.f1fe04p-8f, 0x1.26eb18p-5f, 0x1.bff1p-4f,
                                      0x1.b43c4p-3f,  0x1.106562p-2f, 0x1.b43c4p-3f,  0x1.bff1p-4f,
                                      0x1.26eb18p-5f, 0x1.f1fe04p-8f, 0x1.0d957p-10f};

// Pass 1: per channel and 16 x 16 tile: the five window sums of a and b
// (zero outside the image), the SSIM map value m and its partial
// derivatives with respect to mu_a, E[a^2] and E[ab] (written to d3 [3][C][HW]
// for pass 2); per block: sum of m and of |a - b| (fixed order).  Bound by
// vector arithmetic (86 % of the cycles before), so: one division per pixel
// for the five quotients, and a staged row per half wave instead of a division
// per element (three channels of 1024^2, all together: 53 -> 43 us).
__global__ __launch_bounds__(SS_T *SS_T) void k_ssim_fwd(int C, int H, int W, const float *__restrict__ a,
                                                          const float *__restrict__ b, float *__restrict__ d3,
                                                          float *__restrict__ part) {
  __shared__ float s_a[SS_E][SS_P], s_b[SS_E][SS_P];
  __shared__ float s_h[5][SS_E][SS_T];
  __shared__ float s_red[2][SS_T * SS_T / 64];
  const int tw = (W + SS_T - 1) / SS_T;
  const int tile = blockIdx.x, ch = blockIdx.y;
  const int X0 = (tile % tw) * SS_T - SS_R, Y0 = (tile / tw) * SS_T - SS_R;
  const int64_t HW = (int64_t)H * W;
  const float *A = a + ch * HW, *B = b + ch * HW;
  const int sx = threadIdx.x % 32, sy = threadIdx.x / 32, xx = X0 + sx;
#pragma unroll
  for (int i = 0; i < SS_E; i += SS_ROWS) {
    const int row = i + sy, yy = Y0 + row;
    if (sx >= SS_E || row >= SS_E) continue;
    const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
    s_a[row][sx] = in ? A[(int64_t)yy * W + xx] : 0.f;
    s_b[row][sx] = in ? B[(int64_t)yy * W + xx] : 0.f;
  }
  __syncthreads();
  // horizontal pass over the staged rows
  for (int q = threadIdx.x; q < SS_E * SS_T; q += SS_T * SS_T) {
    const int row = q / SS_T, col = q % SS_T;
    float h0 = 0.f, h1 = 0.f, h2 = 0.f, h3 = 0.f, h4 = 0.f;
#pragma unroll
    for (int k = 0; k <= 2 * SS_R; ++k) {
      const float wk = SS_W[k], va = s_a[row][col + k], vb = s_b[row][col + k];
      h0 += wk * va;
      h1 += wk * vb;
      h2 += wk * va * va;
      h3 += wk * vb * vb;
      h4 += wk * va * vb;
    }
    s_h[0][row][col] = h0;
    s_h[1][row][col] = h1;
    s_h[2][row][col] = h2;
    s_h[3][row][col] = h3;
    s_h[4][row][col] = h4;
  }
  __syncthreads();
  const int tx = threadIdx.x % SS_T, ty = threadIdx.x / SS_T;
  const int x = X0 + SS_R + tx, y = Y0 + SS_R + ty;
  float m = 0.f, l1 = 0.f;
  if (x < W && y < H) {
    float S[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k <= 2 * SS_R; ++k) {
      const float wk = SS_W[k];
#pragma unroll
      for (int v = 0; v < 5; ++v) S[v] += wk * s_h[v][ty + k][tx];
    }
    const float mu_a = S[0], mu_b = S[1];
    const float va = S[2] - mu_a * mu_a, vb = S[3] - mu_b * mu_b, cab = S[4] - mu_a * mu_b;
    const float n1 = 2.f * mu_a * mu_b + SS_C1, n2 = 2.f * cab + SS_C2;
    const float e1 = mu_a * mu_a + mu_b * mu_b + SS_C1, e2 = va + vb + SS_C2;
    const float den = e1 * e2;
    const float r = 1.0f / den;  // 1 / e2 = e1 r
    m = n1 * n2 * r;
    // m as a function of (mu_a, E[a^2], E[ab]) with mu_b, E[b^2] fixed:
    // dn1/dmu_a = 2 mu_b; dn2/dmu_a = -2 mu_b, dn2/dE[ab] = 2;
    // de1/dmu_a = 2 mu_a; de2/dmu_a = -2 mu_a, de2/dE[a^2] = 1
    const float dmu = 2.f * r * (mu_b * (n2 - n1) - m * (mu_a * (e2 - e1)));
    const float dEaa = -m * (e1 * r);
    const float dEab = 2.f * n1 * r;
    const int64_t pix = (int64_t)y * W + x;
    d3[(int64_t)ch * HW + pix] = dmu;
    d3[((int64_t)C + ch) * HW + pix] = dEaa;
    d3[(2 * (int64_t)C + ch) * HW + pix] = dEab;
    l1 = fabsf(s_a[ty + SS_R][tx + SS_R] - s_b[ty + SS_R][tx + SS_R]);
  }
  // block sums, fixed order
  const float sm = wave_sum(m), sl = wave_sum(l1);
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = sm;
    s_red[1][threadIdx.x >> 6] = sl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float t0 = 0.f, t1 = 0.f;
#pragma unroll
    for (int w = 0; w < SS_T * SS_T / 64; ++w) {
      t0 += s_red[0][w];
      t1 += s_red[1][w];
    }
    const int64_t blk = (int64_t)ch * gridDim.x + tile;
    part[2 * blk] = t0;
    part[2 * blk + 1] = t1;
  }
}

// one block: loss = (1 - lam) mean|a - b| + lam (1 - mean SSIM), added to
// *loss in a fixed order over the block partials
__global__ __launch_bounds__(256) void k_loss_final(int nblk, int64_t count, float lam,
                                                    const float *__restrict__ part, float *__restrict__ loss) {
  __shared__ float s_m[256], s_l[256];
  float m = 0.f, l = 0.f;
#pragma unroll 8
  for (int q = threadIdx.x; q < nblk; q += 256) {
    const float2 p = reinterpret_cast<const float2 *>(part)[q];
    m += p.x;
    l += p.y;
  }
  s_m[threadIdx.x] = m;
  s_l[threadIdx.x] = l;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      s_m[threadIdx.x] += s_m[threadIdx.x + h];
      s_l[threadIdx.x] += s_l[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float inv = 1.0f / (float)count;
    *loss += (1.0f - lam) * s_l[0] * inv + lam * (1.0f - s_m[0] * inv);
  }
}

// Pass 2: dL/da = (1 - lam)/N sign(a - b) - lam/N (w * dmu + 2 a (w * dEaa)
// + b (w * dEab)), the window correlations over the staged partials (zero
// outside the image); ADDS to a_bar.
__global__ __launch_bounds__(SS_T *SS_T) void k_ssim_bwd(int C, int H, int W, float lam, const float *__restrict__ a,
                                                          const float *__restrict__ b, const float *__restrict__ d3,
                                                          float *__restrict__ a_bar) {
  __shared__ float s_d[3][SS_E][SS_P];
  __shared__ float s_h[3][SS_E][SS_T];
  const int tw = (W + SS_T - 1) / SS_T;
  const int tile = blockIdx.x, ch = blockIdx.y;
  const int X0 = (tile % tw) * SS_T - SS_R, Y0 = (tile / tw) * SS_T - SS_R;
  const int64_t HW = (int64_t)H * W;
  for (int q = threadIdx.x; q < SS_E * SS_E; q += SS_T * SS_T) {
    const int yy = Y0 + q / SS_E, xx = X0 + q % SS_E;
    const bool in = yy >= 0 && yy < H && xx >= 0 && xx < W;
    const int64_t pix = (int64_t)yy * W + xx;
#pragma unroll
    for (int v = 0; v < 3; ++v) s_d[v][q / SS_E][q % SS_E] = in ? d3[((int64_t)v * C + ch) * HW + pix] : 0.f;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < SS_E * SS_T; q += SS_T * SS_T) {
    const int row = q / SS_T, col = q % SS_T;
    float h[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k <= 2 * SS_R; ++k)
#pragma unroll
      for (int v = 0; v < 3; ++v) h[v] += SS_W[k] * s_d[v][row][col + k];
#pragma unroll
    for (int v = 0; v < 3; ++v) s_h[v][row][col] = h[v];
  }
  __syncthreads();
  const int tx = threadIdx.x % SS_T, ty = threadIdx.x / SS_T;
  const int x = X0 + SS_R + tx, y = Y0 + SS_R + ty;
  if (x >= W || y >= H) return;
  float S[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k <= 2 * SS_R; ++k)
#pragma unroll
    for (int v = 0; v < 3; ++v) S[v] += SS_W[k] * s_h[v][ty + k][tx];
  const int64_t pix = (int64_t)ch * HW + (int64_t)y * W + x;
  const float va = a[pix], vb = b[pix];
  const float inv = 1.0f / (float)(C * HW);
  const float sg = va > vb ? 1.f : (va < vb ? -1.f : 0.f);
  a_bar[pix] += (1.0f - lam) * inv * sg - lam * inv * (S[0] + 2.f * va * S[1] + vb * S[2]);
}

static int make_cam(const dw_camera *c, CamDev *K) {
  DW_REQUIRE(c, DW_EINVAL, "render: camera is NULL");
  DW_REQUIRE(c->width >= 1 && c->height >= 1 && c->width <= 16384 && c->height <= 16384, DW_ERANGE,
             "render: image size must be 1..16384 per axis");
  DW_REQUIRE(c->near_plane >= 0.f, DW_EINVAL, "render: near plane must be >= 0");
  DW_REQUIRE(c->alpha_min >= 0.f && c->alpha_min < 1.f, DW_EINVAL, "render: alpha_min must be in [0, 1)");
  DW_REQUIRE(c->t_min >= 0.f && c->t_min < 1.f, DW_EINVAL, "render: t_min must be in [0, 1)");
  K->W = c->width;
  K->H = c->height;
  K->tw = (c->width + GS_TILE - 1) / GS_TILE;
  K->th = (c->height + GS_TILE - 1) / GS_TILE;
  K->fx = c->fx;
  K->fy = c->fy;
  K->cx = c->cx;
  K->cy = c->cy;
  for (int q = 0; q < 9; ++q) K->R[q] = c->R[q];
  for (int q = 0; q < 3; ++q) {
    K->t[q] = c->t[q];
    K->bg[q] = c->bg[q];
  }
  K->near_ = c->near_plane;
  K->amin = c->alpha_min;
  K->tmin = c->t_min;
  return DW_OK;
}

static int bits_for(int64_t v) {
  int b = 0;
  while (((int64_t)1 << b) < v) ++b;
  return b;
}

// passes of the pair sort by tile; an odd count leaves the pairs in buffer b
static int pair_bits(int64_t T) { return bits_for(T) < 1 ? 1 : bits_for(T); }
static bool pairs_in_b(int64_t T) { return ((pair_bits(T) + 7) / 8) % 2 == 1; }

}  // namespace dw

using namespace dw;

extern "C" size_t gs_render_workspace_bytes(int n, const dw_camera *cam, int64_t max_pairs) {
  if (n < 0 || !cam || cam->width < 1 || cam->height < 1 || max_pairs < 0) return 0;
  return gs_layout(nullptr, n, max_pairs, cam->width, cam->height).bytes;
}

static int gs_common(const char *who, const dw_camera *cam, int n, const float *mu, const float *sigma,
                     const float *color, const float *opacity, int64_t max_pairs, void *ws, size_t ws_bytes,
                     CamDev *K, GsWs *w) {
  int rc = make_cam(cam, K);
  if (rc) return rc;
  DW_REQUIRE(n >= 0, DW_EINVAL, "%s: n must be >= 0", who);
  DW_REQUIRE(max_pairs >= 0 && max_pairs < ((int64_t)1 << 31), DW_ERANGE, "%s: max_pairs must be in [0, 2^31)", who);
  DW_REQUIRE(ws, DW_EINVAL, "%s: workspace is NULL", who);
  DW_REQUIRE(n == 0 || (mu && sigma && color && opacity), DW_EINVAL, "%s: kernel arrays are NULL", who);
  *w = gs_layout((char *)ws, n, max_pairs, cam->width, cam->height);
  DW_REQUIRE(ws_bytes >= w->bytes, DW_EWORKSPACE, "%s: workspace too small (%zu < %zu bytes)", who, ws_bytes,
             w->bytes);
  DW_REQUIRE(rs_blocks(n > max_pairs ? n : max_pairs) * 256 <= (int64_t)SCAN_CHUNK * SCAN_TOP_MAX &&
                 (n + (int64_t)SCAN_CHUNK - 1) / SCAN_CHUNK <= SCAN_TOP_MAX,
             DW_ERANGE, "%s: too many kernels or pairs for the scan", who);
  return DW_OK;
}

extern "C" int gs_render(const dw_camera *cam, int n, const float *mu, const float *sigma, const float *color,
                         const float *opacity, float *image, int64_t max_pairs, void *ws, size_t ws_bytes,
                         void *stream) {
  CamDev K;
  GsWs w;
  int rc = gs_common("gs_render", cam, n, mu, sigma, color, opacity, max_pairs, ws, ws_bytes, &K, &w);
  if (rc) return rc;
  DW_REQUIRE(image, DW_EINVAL, "gs_render: image is NULL");
  hipStream_t s = (hipStream_t)stream;
  const int64_t T = (int64_t)K.tw * K.th;
  hipLaunchKernelGGL(k_gs_begin, dim3(grid_blocks(T > GS_HDR_INTS ? T : GS_HDR_INTS, 256)), dim3(256), 0, s, w, T);
  if (n > 0) {
    hipLaunchKernelGGL(k_gs_project, dim3(grid_blocks(n, 256)), dim3(256), 0, s, K, n, mu, sigma, color, opacity, w);
    uint32_t *ka = w.key_a, *kb = w.key_b;
    int32_t *va = w.id_a, *vb = w.id_b;
    radix_sort(&ka, &va, &kb, &vb, n, nullptr, 32, false, w.hist, rs_rows(n, max_pairs), w.bsum, s);  // 4 passes: back in buffer a
    const unsigned nsc = grid_blocks(n, SCAN_CHUNK);
    hipLaunchKernelGGL(k_gs_cnt_sums, dim3(nsc), dim3(SCAN_THREADS), 0, s, n, va, w.cnt, w.off, w.bsum);
    hipLaunchKernelGGL(k_gs_cnt_scan, dim3(nsc), dim3(SCAN_THREADS), 0, s, n, w.bsum, max_pairs, w.off, w.hdr);
    if (max_pairs > 0) {
      const int bits = pair_bits(T), w0 = rs_digit(bits) < 4 ? 4 : rs_digit(bits);
      hipLaunchKernelGGL(k_gs_emit, dim3(grid_blocks(max_pairs, GS_EMIT)), dim3(256), 0, s, n, K, va, w.off, w.rect,
                         w.hdr, (1u << w0) - 1u, w.pk_a, w.pv_a, w.hist);
      uint32_t *pa = w.pk_a, *pb = w.pk_b;
      int32_t *qa = w.pv_a, *qb = w.pv_b;
      radix_sort(&pa, &qa, &pb, &qb, max_pairs, w.hdr + 1, bits, true, w.hist, rs_rows(n, max_pairs), w.bsum, s);
      hipLaunchKernelGGL(k_gs_ranges, dim3(grid_blocks(max_pairs < 8 * (int64_t)n ? max_pairs : 8 * (int64_t)n, 1024)),
                         dim3(256), 0, s, pa, w.hdr, w.range);
    }
  }
  const int32_t *ids = pairs_in_b(T) ? w.pv_b : w.pv_a;
  hipLaunchKernelGGL(k_gs_classify, dim3(grid_blocks(T, 64)), dim3(256), 0, s, K, w, ids);
  hipLaunchKernelGGL(k_gs_raster, dim3(gs_raster_blocks(T)), dim3(GS_THREADS), 0, s, K, w, ids, image);
  return check_launch("gs_render");
}

extern "C" int gs_render_adj(const dw_camera *cam, int n, const float *mu, const float *sigma, const float *color,
                             const float *opacity, const float *image, const float *image_bar, float *mu_bar,
                             float *sigma_bar, float *color_bar, float *opacity_bar, int64_t max_pairs, void *ws,
                             size_t ws_bytes, void *stream) {
  CamDev K;
  GsWs w;
  int rc = gs_common("gs_render_adj", cam, n, mu, sigma, color, opacity, max_pairs, ws, ws_bytes, &K, &w);
  if (rc) return rc;
  DW_REQUIRE(image && image_bar, DW_EINVAL, "gs_render_adj: image / image_bar is NULL");
  if (n == 0) return DW_OK;
  hipStream_t s = (hipStream_t)stream;
  const int64_t T = (int64_t)K.tw * K.th;
  const int64_t n4 = (GS_NB * (int64_t)n + 3) / 4;  // the section is padded to 256 bytes
  hipLaunchKernelGGL(k_gs_adj_begin, dim3(grid_blocks(n4, 256)), dim3(256), 0, s, w, n4);
  const int32_t *ids = pairs_in_b(T) ? w.pv_b : w.pv_a;
  hipLaunchKernelGGL(k_gs_raster_adj, dim3(gs_raster_blocks(T)), dim3(GS_THREADS), 0, s, K, w, ids, image, image_bar);
  hipLaunchKernelGGL(k_gs_project_adj, dim3(grid_blocks(n, 256)), dim3(256), 0, s, K, n, mu, sigma, opacity, w.gbar,
                     mu_bar, sigma_bar, color_bar, opacity_bar);
  return check_launch("gs_render_adj");
}

extern "C" int gs_render_status(const void *ws, int32_t *status_out, void *stream) {
  DW_REQUIRE(ws && status_out, DW_EINVAL, "gs_render_status: NULL argument");
  hipLaunchKernelGGL(k_gs_status, dim3(1), dim3(64), 0, (hipStream_t)stream, (const int32_t *)ws, status_out);
  return check_launch("gs_render_status");
}

static size_t loss_layout(int C, int H, int W, float **d3, float **part, char *base) {
  const int64_t HW = (int64_t)H * W;
  const int64_t nblk = (int64_t)C * ((W + SS_T - 1) / SS_T) * ((H + SS_T - 1) / SS_T);
  size_t o = 0;
  if (d3) *d3 = base ? (float *)(base + o) : nullptr;
  o += al256((size_t)3 * C * HW * 4);
  if (part) *part = base ? (float *)(base + o) : nullptr;
  o += al256((size_t)2 * nblk * 4);
  return o;
}

extern "C" size_t render_loss_workspace_bytes(int C, int H, int W) {
  if (C < 1 || H < 1 || W < 1) return 0;
  return loss_layout(C, H, W, nullptr, nullptr, nullptr);
}

extern "C" int render_loss(int C, int H, int W, const float *image, const float *target, float lambda, float *loss,
                           float *image_bar, void *ws, size_t ws_bytes, void *stream) {
  DW_REQUIRE(C >= 1 && H >= 1 && W >= 1, DW_EINVAL, "render_loss: sizes must be >= 1");
  DW_REQUIRE(image && target && ws, DW_EINVAL, "render_loss: image / target / workspace is NULL");
  DW_REQUIRE(lambda >= 0.f && lambda <= 1.f, DW_EINVAL, "render_loss: lambda must be in [0, 1]");
  DW_REQUIRE(C <= 65535, DW_ERANGE, "render_loss: too many channels");
  float *d3, *part;
  const size_t need = loss_layout(C, H, W, &d3, &part, (char *)ws);
  DW_REQUIRE(ws_bytes >= need, DW_EWORKSPACE, "render_loss: workspace too small (%zu < %zu bytes)", ws_bytes, need);
  hipStream_t s = (hipStream_t)stream;
  const unsigned tiles = (unsigned)(((W + SS_T - 1) / SS_T) * ((H + SS_T - 1) / SS_T));
  hipLaunchKernelGGL(k_ssim_fwd, dim3(tiles, (unsigned)C), dim3(SS_T * SS_T), 0, s, C, H, W, image, target, d3, part);
  if (loss)
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, (int)(tiles * C), (int64_t)C * H * W, lambda, part,
                       loss);
  if (image_bar)
    hipLaunchKernelGGL(k_ssim_bwd, dim3(tiles, (unsigned)C), dim3(SS_T * SS_T), 0, s, C, H, W, lambda, image, target,
                       d3, image_bar);
  return check_launch("render_loss");
}
