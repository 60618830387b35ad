// BF16 MFMA 3x3x3 convolutions of the wind surrogate (gfx950), FP32 accumulation.
//
// The surrogate advances a wind velocity field k LBM steps at once:
//   u_{t+k} = u_t + g s net(u_t / s),  net = conv(32->3) o silu o conv(32->32)
//   o silu o conv(32->32) o silu o conv(3->32),  3x3x3 kernels, zero padding,
// s the per-field inflow speed, g a fixed output gain (the caller's scale of
// the output layer's residual).  Its error is measured against the lattice
// Boltzmann step of Eq. lbe.
//
// Implicit GEMM per layer: M = output channels (tiles of 16), N = a row of 16
// voxels along x, K = (tap, input channel).  Activations are channels-last
// BF16 [B][nz][ny][nx][C] with C padded to 8 (3-channel fields) or 32.  One
// v_mfma_f32_16x16x32_bf16 consumes K = 32: one tap of 32 channels, or four
// taps of 8 (padded) channels.  A workgroup (4 waves) stages zero-padded
// input patches of its output tiles in LDS; for 32-channel inputs a wave's
// m-tile weight fragments stay in registers for the life of the persistent
// workgroup.  Lane layout of the 16x16x32 MFMA: lane l holds
// A[l % 16][8 (l / 16) .. +8], B[8 (l / 16) .. +8][l % 16] and
// D[4 (l / 16) .. +4][l % 16].
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <algorithm>
#include <climits>

#include "dw_internal.h"

namespace dw {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// float -> bf16, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// two floats -> packed bf16 pair (a in the low half), one instruction
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(float2v{a, b}, bf16x2));
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// logistic function with the hardware exponential and reciprocal (about
// 1 ulp each, far below the bf16 rounding of every value it feeds)
__device__ __forceinline__ float sigmoid(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float silu_grad(float z) {
  const float sg = sigmoid(z);
  return sg * (1.0f + z * (1.0f - sg));
}

struct ConvGeom {
  int B, nx, ny, nz;
  int64_t L;  // voxels per field
};

// ----------------------------------------------------------------- forward
//
// Forward / data-gradient layer.  A workgroup (4 waves, 2 resident per CU)
// copies zero-padded input patches into LDS with buffer_load ... lds
// (channels-last, 16-byte chunks of 8 channels), then:
//  * 32-channel inputs: tiles of FX x FY x CZ = 16 x 4 x 4 outputs; a
//    workgroup walks a column of tiles along z, the patch planes in a ring
//    of RING slots; each wave copies one of the next tile's CZ new planes
//    into a slot the current tile does not read while its MFMAs run.  The
//    copies are asynchronous (copy_to_lds) from per-lane offsets made once per
//    column, and what the epilogue reads (the gradient's gates, the output
//    layer's field) is requested ahead of the MFMAs too, so that one wait per
//    tile is all that memory costs; with copies that the compiler waited for
//    and gates read in the epilogue, 16 x 64^3 voxels took 220 (32 -> 32), 150
//    (32 -> 3) and 322 us (data gradient), then 200, 118 and 226.  The matrix
//    cores need 92 us of the first at 2.4 GHz, the memory 160 of the third.
//    Wave w computes a
//    4 (y) x RZ (z) block of output rows for one 16-channel m-tile, holding
//    that m-tile's 27 weight fragments in registers for the life of the
//    kernel.  For each x-shift it walks the (RZ+2) x 6 input rows; every
//    fragment read from LDS feeds up to 3 RZ MFMAs (all (dz, dy) taps that
//    map it onto an output row).
//    The 3-channel output layer would leave 13 of the 16 rows of a weight
//    fragment empty: its rows are 3 x taps x 4 (3 channels and a zero) instead,
//    so a (dz, dy) pair costs one MFMA per row, not three, and a row's
//    fragment is read once.  Lane row dx then holds the products of tap dx at
//    the row's own voxels; the epilogue shifts them by a voxel and adds the
//    lane rows, each of which ends up with one output row.  What the taps need
//    from the voxels beside the 16 is one more fragment, of the four output
//    rows' ends, per (dz, dy).  45 MFMAs and 27 reads instead of 108 and 54
//    for 64 voxels: 256 x 128 x 128 voxels 116 -> 94 us, of which the memory
//    needs 73.
//  * 8-channel inputs (3 channels padded): tiles of FX x FY x FZ = 16 x 4 x 8
//    outputs, one patch per tile; K = 32 spans 4 taps; each wave computes 8
//    whole rows, all m-tiles, two rows at a time, and stores whole voxels
//    (out_channel).  Bound by the 268 MB that the 16 x 64^3 voxels write: 110
//    -> 96 us (3 -> 32), and by as much again read by the data gradient, 195 ->
//    141 (with four workgroups per CU instead of two).
// The 4 chunks of a voxel's 32 channels are stored permuted by swz(x) so the
// fragment reads spread over the LDS banks.

constexpr int FX = 16, FY = 4, FZ = 8;                 // output tile
constexpr int QX = FX + 2, QY = FY + 2, QZ = FZ + 2;   // input patch
constexpr int QVOX = QX * QY * QZ;

// 32-channel inputs: tiles of FX x FY x CZ outputs, walked along z; the
// patch planes live in a ring of RING slots of CPLANE elements in LDS
constexpr int CZ = 4, CQZ = CZ + 2, RING = QZ;
constexpr int CPLANE = (QX * QY * 4 + 63) / 64 * 64 * 8;  // whole waves of chunks
static_assert(RING >= CQZ + CZ, "the next tile's new planes need slots of their own");

struct FwdTiles {
  int tx, ty, tz, n;  // tiles per axis, total over the batch
  // 32-channel inputs: work items are (column, z segment) pairs; a column is
  // the tzc tiles (CZ planes each) of one (x, y) tile position of one field
  int tzc, ncol, zlen, nitems;
};

struct TileOrigin {
  int b, x0, y0, z0;
};
__device__ __forceinline__ TileOrigin fwd_tile(const FwdTiles &T, int t) {
  TileOrigin o;
  o.x0 = (t % T.tx) * FX;
  int r = t / T.tx;
  o.y0 = (r % T.ty) * FY;
  r /= T.ty;
  o.z0 = (r % T.tz) * FZ;
  o.b = r / T.tz;
  return o;
}

// chunk c of a patch voxel with x index xx is stored at position c ^ swz(xx).
// The 64 lanes of a fragment read take 16 consecutive x and all four chunks.
// Of the 1,024 linear maps of x's bits to two bits this is one of those whose
// reads are free of bank conflicts at every x shift (6.4 cycles per read of
// two workgroups against 9.8 with bits 2 and 3 of x).
__device__ __forceinline__ int swz(int xx) { return (xx & 1) | ((xx >> 1) & 2); }

typedef __attribute__((address_space(3))) void *lds_ptr_t;

// Copy the zero-padded input patch of a tile into LDS.  Chunk q of the patch
// lands at s_in + 16 q (each wave fills 64 consecutive chunks per
// instruction); voxels outside the field, and chunks past the patch up to the
// wave's 64, get an offset beyond the buffer's size, which the hardware
// returns as zeros: s_in must hold the patch rounded up to 64 chunks.
template <int CINP>
__device__ __forceinline__ void stage_patch(const ConvGeom &G, const uint16_t *__restrict__ x,
                                            const TileOrigin &o, uint16_t *s_in) {
  constexpr int VEC = CINP / 8;
  constexpr int NV = QVOX * VEC;
  constexpr int ITER = (NV + 255) / 256;
  // each iteration moves a lane 256 chunks = D voxels on through the patch:
  // its coordinates and field index advance by constant steps with carries
  // (no divisions or 32-bit multiplies per chunk)
  constexpr int D = 256 / VEC;
  constexpr int DX = D % QX, DY = (D / QX) % QY, DZ = D / (QX * QY);
  static_assert(256 % VEC == 0, "a lane keeps its channel chunk across iterations");
  const uint16_t *field = x + (int64_t)o.b * G.L * CINP;
  __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc((void *)field, (short)0, (int)(G.L * CINP * 2), 0x00020000);
  const int wid = threadIdx.x >> 6;
  int lane = threadIdx.x & 63;
  // recompute the per-lane patch coordinates for every tile rather than
  // keeping them live across the tile loop
  asm volatile("" : "+v"(lane));
  const int ql = wid * 64 + lane;  // this lane's chunk in iteration 0
  const int p = ql % VEC;
  const int v = ql / VEC;
  int xx = v % QX, yy = (v / QX) % QY;
  int gx = o.x0 + xx - 1, gy = o.y0 + yy - 1, gz = o.z0 + v / (QX * QY) - 1;
  const int sy = G.nx, sz = G.nx * G.ny;
  int lin = gx + sy * gy + sz * gz;
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int q0 = it * 256 + wid * 64;  // first chunk of this wave (uniform)
    if (q0 >= NV) break;
    const int q = q0 + lane;
    const int c = VEC == 4 ? (p ^ swz(xx)) : p;  // channel chunk stored at position p
    const bool in = q < NV && (unsigned)gx < (unsigned)G.nx && (unsigned)gy < (unsigned)G.ny &&
                    (unsigned)gz < (unsigned)G.nz;
    const unsigned off = in ? (unsigned)((lin * CINP + c * 8) * 2) : 0x80000000u;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(s_in + q0 * 8), 16, off, 0, 0, 0);
    xx += DX; gx += DX; lin += DX;
    if (xx >= QX) { xx -= QX; gx -= QX; yy += 1; gy += 1; lin += sy - QX; }
    yy += DY; gy += DY; lin += DY * sy;
    if (yy >= QY) { yy -= QY; gy -= QY; gz += 1; lin += sz - QY * sy; }
    gz += DZ; lin += DZ * sz;
  }
}

// one 16-byte chunk per lane from `off` of the buffer into LDS at `lds` +
// 16 lane; completion is counted in vmcnt only.  Written in assembly because
// the compiler cannot tell which LDS bytes the copy writes and would wait
// for it (and for every store before it) ahead of the next LDS read.  The
// caller waits (s_waitcnt vmcnt) and passes a barrier before reading.  m0 is
// set here and used by nothing else in these kernels.
__device__ __forceinline__ void copy_to_lds(__amdgpu_buffer_rsrc_t rsrc, uint32_t lds, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(off), "s"(rsrc)
               : "memory");
}

typedef __attribute__((address_space(3))) char *lds_bytes_t;

// Byte offsets, within a z plane of the field, of the PCH chunks per lane that
// make a plane of the patch of a column (32 channels): chunk 64 j + lane of
// the plane; out of the buffer (zeros) outside the field and past the plane.
constexpr int PCH = (QX * QY * 4 + 63) / 64;
__device__ __forceinline__ void plane_offsets(const ConvGeom &G, int x0, int y0, uint32_t (&off)[PCH]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < PCH; ++j) {
    const int q = j * 64 + lane, vox = q / 4, xx = vox % QX, yy = vox / QX;
    const int gx = x0 + xx - 1, gy = y0 + yy - 1, c = (q % 4) ^ swz(xx);
    const bool in = yy < QY && (unsigned)gx < (unsigned)G.nx && (unsigned)gy < (unsigned)G.ny;
    off[j] = in ? (uint32_t)((gx + G.nx * gy) * 64 + c * 16) : 0x80000000u;
  }
}

// Issue the copies of plane gz of field `field` (32 channels) into LDS at
// `lds`; a plane outside the field is zeros.  All of it wave-uniform.
__device__ __forceinline__ void copy_plane(const ConvGeom &G, const uint16_t *field, int gz, uint32_t lds,
                                           const uint32_t (&off)[PCH]) {
  const bool in = gz >= 0 && gz < G.nz;
  const uint32_t plane = (uint32_t)(G.nx * G.ny) * 64u;
  const uint64_t base = (uint64_t)field + (in ? (uint64_t)gz * plane : 0ull);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base), hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)),
                 size = __builtin_amdgcn_readfirstlane(in ? plane : 0u), dst = __builtin_amdgcn_readfirstlane(lds);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), (short)0,
                                                                        (int)size, 0x00020000);
#pragma unroll
  for (int j = 0; j < PCH; ++j) copy_to_lds(rsrc, dst + j * 1024, off[j]);
}

// Work item v of the column plan: column v % ncol, z segment v / ncol.
struct ColItem {
  int b, x0, y0, zt0, zt1;  // field, tile origin in x and y, z tiles [zt0, zt1)
};
__device__ __forceinline__ ColItem col_item(const FwdTiles &T, int v) {
  ColItem c;
  const int col = v % T.ncol, seg = v / T.ncol;
  c.x0 = (col % T.tx) * FX;
  const int r = col / T.tx;
  c.y0 = (r % T.ty) * FY;
  c.b = r / T.ty;
  c.zt0 = seg * T.zlen;
  c.zt1 = min(T.tzc, c.zt0 + T.zlen);
  return c;
}

// Epilogue of one output row: lane holds channels co0 .. co0 + 3 of voxel
// vi of field o.b (acc = those 4 sums); live = the voxel is inside the field
// (ragged edge tiles).  Per-field bases plus 32-bit element offsets.
template <int COUTP, int EPI>
__device__ __forceinline__ void conv_epilogue(const ConvGeom &G, const TileOrigin &o, bool live, uint32_t vi,
                                              int co0, floatx4 acc, const float *s_bias,
                                              uint16_t *__restrict__ y, uint16_t *__restrict__ zpre, uint2 zg) {
  if (!live) return;
  const uint32_t ei = vi * COUTP + co0;  // element offset in the field's activations
  const size_t fb = (size_t)o.b * G.L * COUTP;
  if (EPI == DW_CONV_HIDDEN) {
    float zv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) zv[j] = acc[j] + s_bias[co0 + j];
    *reinterpret_cast<uint2 *>(y + fb + ei) = make_uint2(f2bf2(silu(zv[0]), silu(zv[1])), f2bf2(silu(zv[2]), silu(zv[3])));
    if (zpre) *reinterpret_cast<uint2 *>(zpre + fb + ei) = make_uint2(f2bf2(zv[0], zv[1]), f2bf2(zv[2], zv[3]));
  } else {  // DW_CONV_DGRAD: gradient through the previous layer's silu
    const float zf[4] = {bf2f((uint16_t)(zg.x & 0xffff)), bf2f((uint16_t)(zg.x >> 16)), bf2f((uint16_t)(zg.y & 0xffff)),
                         bf2f((uint16_t)(zg.y >> 16))};
    float ob[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) ob[j] = acc[j] * silu_grad(zf[j]);
    *reinterpret_cast<uint2 *>(y + fb + ei) = make_uint2(f2bf2(ob[0], ob[1]), f2bf2(ob[2], ob[3]));
  }
}

// 8-channel inputs: a wave computes both 16-channel m-tiles, so their rows are
// dealt to the output channels such that a lane's four rows of each make eight
// adjacent channels 8 g .. 8 g + 7, and a wave stores 16 whole voxels (1 KB)
// with one instruction.
template <int MT>
__device__ __forceinline__ int out_channel(int m, int row) {
  return MT == 2 ? 8 * (row >> 2) + 4 * m + (row & 3) : row;
}

template <int EPI>
__device__ __forceinline__ void wide_epilogue(uint32_t vi, int g, const floatx4 (&acc)[2], const float *s_bias,
                                              uint16_t *__restrict__ y, uint16_t *__restrict__ zpre,
                                              const uint16_t *__restrict__ zgate) {
  const uint32_t ei = vi * 32 + 8 * g;
  uint32_t out[4];
  if (EPI == DW_CONV_HIDDEN) {
    uint32_t z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float a = acc[q >> 1][(2 * q) & 3] + s_bias[8 * g + 2 * q],
                  b = acc[q >> 1][(2 * q + 1) & 3] + s_bias[8 * g + 2 * q + 1];
      out[q] = f2bf2(silu(a), silu(b));
      z[q] = f2bf2(a, b);
    }
    if (zpre) *reinterpret_cast<uint4 *>(zpre + ei) = make_uint4(z[0], z[1], z[2], z[3]);
  } else {  // DW_CONV_DGRAD: gradient through the previous layer's silu
    const uint4 zg = *reinterpret_cast<const uint4 *>(zgate + ei);
    const uint32_t z[4] = {zg.x, zg.y, zg.z, zg.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      out[q] = f2bf2(acc[q >> 1][(2 * q) & 3] * silu_grad(bf2f((uint16_t)(z[q] & 0xffff))),
                     acc[q >> 1][(2 * q + 1) & 3] * silu_grad(bf2f((uint16_t)(z[q] >> 16))));
  }
  *reinterpret_cast<uint4 *>(y + ei) = make_uint4(out[0], out[1], out[2], out[3]);
}

// `x` of the lane that DPP control `CTRL` names, in the rows of 16 lanes of
// `ROWS`; `old` in the others and where that lane is outside the row
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp(float old, float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL, ROWS, 0xf, false));
}
constexpr int DPP_SHL = 0x100, DPP_SHR = 0x110, DPP_SAME = 0xe4;

// a and b summed over the rows of 16 lanes: first over rows two apart (a in
// the lower half, b in the upper), then over adjacent ones (a in the even
// rows, b in the odd)
__device__ __forceinline__ float halves_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float quarters_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Output layer: the three x taps of output row YO, channel sums v (lane row dx
// = the products of tap dx at the row's own voxels) and e (the same at the two
// voxels beside the row: lane YO left of it, lane 12 + YO right of it), moved
// to the voxel they belong to.  Lane row 3 holds no tap.
template <int YO>
__device__ __forceinline__ float x_taps(int g, float v, float e) {
  float t = dpp<YO ? DPP_SHL + YO : DPP_SAME, 1>(v, e);
  t = dpp<YO < 3 ? DPP_SHR + 3 - YO : DPP_SAME, 4>(t, e);
  t = dpp<DPP_SHR + 1, 1>(t, v);
  t = dpp<DPP_SHL + 1, 4>(t, v);
  return g < 3 ? t : 0.f;
}

// Packed weights: [chunk][COUTP][32] bf16, see conv_pack_weights.
template <int CINP, int COUTP, int EPI>
__global__ __launch_bounds__(256, CINP == 32 ? 2 : 4) void k_conv(ConvGeom G, FwdTiles T, const uint16_t *__restrict__ x,
                                                 const uint16_t *__restrict__ wk, const float *__restrict__ bias,
                                                 int cout, uint16_t *__restrict__ y, uint16_t *__restrict__ zpre,
                                                 const uint16_t *__restrict__ zgate, const float *__restrict__ u,
                                                 const float *__restrict__ scale, float *__restrict__ u_out) {
  constexpr int MT = COUTP / 16;
  // bf16 elements, whole waves of chunks
  constexpr int PATCH = CINP == 32 ? RING * CPLANE : (QVOX * CINP / 8 + 63) / 64 * 64 * 8;
  __shared__ __attribute__((aligned(16))) uint16_t s_in[PATCH];
  __shared__ float s_bias[32];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int g = lane >> 4, r16 = lane & 15;
  if (threadIdx.x < 32) s_bias[threadIdx.x] = (bias && (int)threadIdx.x < cout) ? bias[threadIdx.x] : 0.f;

  if constexpr (CINP == 32) {
    constexpr bool OUT = EPI == DW_CONV_OUTPUT;
    static_assert(OUT ? MT == 1 : MT == 2, "32 or 3 output channels");
    // wave -> (m-tile, z rows of the 16 x 4 x 4 tile)
    constexpr int RZ = OUT ? 1 : 2;
    const int mt = OUT ? 0 : (wid & 1);
    const int zb = OUT ? wid : (wid >> 1) * 2;
    bf16x8 wf[OUT ? 9 : 27];
    if constexpr (OUT) {
      // row 4 dx + co of a fragment: x tap dx, output channel co
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
        wf[tap] = r16 < 12 ? *reinterpret_cast<const bf16x8 *>(
                                 wk + (((3 * tap + (r16 >> 2)) * COUTP + (r16 & 3)) * 32 + g * 8))
                           : bf16x8{};
    } else {
#pragma unroll
      for (int tap = 0; tap < 27; ++tap)
        wf[tap] = *reinterpret_cast<const bf16x8 *>(wk + ((tap * COUTP + mt * 16 + r16) * 32 + g * 8));
    }
    // Work items in an order that gives the workgroups of one XCD (dispatch
    // is round-robin over the 8 XCDs) neighbouring columns, so the x and y
    // halos of concurrent tiles meet in one L2.  A column is walked along z
    // with its patch planes in a ring of RING slots: a tile reads CQZ slots,
    // and the CZ new planes of the column's next tile are copied into the
    // other CZ slots while this tile's MFMAs run.
    const int nb = (int)gridDim.x;
    int v = (nb & 7) ? (int)blockIdx.x : ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    ColItem ci{};
    int zt = 0, rot = 0;
    bool fresh = true;
    if (v < T.nitems) {
      ci = col_item(T, v);
      zt = ci.zt0;
    }
    floatx4 acc[RZ][FY], edge;
    float uin[3];
    uint2 zin[RZ][FY];
    uint32_t off[PCH];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_bytes_t)s_in;
    TileOrigin op{};
    bool have_prev = false;
    auto epilogue = [&](const TileOrigin &oe) {
      const int gx = oe.x0 + r16;
      const uint32_t sy = (uint32_t)G.nx, sz = (uint32_t)G.nx * (uint32_t)G.ny;
      const uint32_t v00 = (uint32_t)gx + sy * (uint32_t)oe.y0 + sz * (uint32_t)(oe.z0 + zb);
      if constexpr (OUT) {
        // u_{t+k} = u_t + s (sum + bias): lane row yo gets output row yo
        const float sb = scale[oe.b];
        const bool live = gx < G.nx && oe.y0 + g < G.ny && oe.z0 + zb < G.nz;
        const size_t ub = (size_t)oe.b * 3 * G.L;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const float s02 = halves_add(x_taps<0>(g, acc[0][0][j], edge[j]), x_taps<2>(g, acc[0][2][j], edge[j])),
                      s13 = halves_add(x_taps<1>(g, acc[0][1][j], edge[j]), x_taps<3>(g, acc[0][3][j], edge[j]));
          const float sum = quarters_add(s02, s13);
          if (live) u_out[ub + (uint32_t)j * (uint32_t)G.L + v00 + g * sy] = uin[j] + sb * (sum + s_bias[j]);
        }
      } else {
#pragma unroll
        for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
          for (int yo = 0; yo < FY; ++yo) {
            const bool live = gx < G.nx && oe.y0 + yo < G.ny && oe.z0 + zb + zo < G.nz;
            conv_epilogue<COUTP, EPI>(G, oe, live, v00 + yo * sy + zo * sz, mt * 16 + 4 * g, acc[zo][yo], s_bias, y,
                                      zpre, zin[zo][yo]);
          }
      }
    };
    while (v < T.nitems) {
      const TileOrigin o{ci.b, ci.x0, ci.y0, zt * CZ};
      const uint16_t *field = x + (int64_t)o.b * G.L * CINP;
      if (fresh) {
        plane_offsets(G, o.x0, o.y0, off);
        __syncthreads();  // every wave is done with the previous tile's planes
        for (int zi = wid; zi < CQZ; zi += 4) copy_plane(G, field, o.z0 - 1 + zi, lds0 + zi * CPLANE * 2, off);
        rot = 0;
        fresh = false;
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's copies have landed
      __syncthreads();  // every wave's have, and every wave is done with the previous tile
      const bool more = zt + 1 < ci.zt1;
      if (more) {
        // one new plane per wave: planes 2 .. CQZ-1 of the next tile's patch
        const int sl = rot + CQZ + wid;
        copy_plane(G, field, o.z0 + CZ + 1 + wid, lds0 + (sl >= RING ? sl - RING : sl) * CPLANE * 2, off);
      }
      // epilogue of the previous tile: its stores are issued before this
      // tile's MFMAs and complete while they run, so the next barrier does
      // not wait for them
      if (have_prev) epilogue(op);
      // output layer: the input field's values at this wave's outputs are
      // requested now and arrive during the MFMAs
      // (data gradient: likewise the pre-activations that gate it)
      if constexpr (EPI == DW_CONV_DGRAD) {
        const int gx = o.x0 + r16;
        const uint32_t sy = (uint32_t)G.nx, sz = (uint32_t)G.nx * (uint32_t)G.ny;
        const uint32_t v00 = (uint32_t)gx + sy * (uint32_t)o.y0 + sz * (uint32_t)(o.z0 + zb);
        const uint16_t *zf = zgate + (size_t)o.b * G.L * COUTP + mt * 16 + 4 * g;
#pragma unroll
        for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
          for (int yo = 0; yo < FY; ++yo) {
            const bool live = gx < G.nx && o.y0 + yo < G.ny && o.z0 + zb + zo < G.nz;
            zin[zo][yo] = live ? *reinterpret_cast<const uint2 *>(zf + (v00 + yo * sy + zo * sz) * COUTP) : uint2{};
          }
      }
      if constexpr (OUT) {
        const int gx = o.x0 + r16;
        const uint32_t sy = (uint32_t)G.nx, sz = (uint32_t)G.nx * (uint32_t)G.ny;
        const uint32_t v00 = (uint32_t)gx + sy * (uint32_t)(o.y0 + g) + sz * (uint32_t)(o.z0 + zb);
        const bool live = gx < G.nx && o.y0 + g < G.ny && o.z0 + zb < G.nz;
#pragma unroll
        for (int j = 0; j < 3; ++j) uin[j] = live ? u[(size_t)o.b * 3 * G.L + (uint32_t)j * (uint32_t)G.L + v00] : 0.f;
      }
#pragma unroll
      for (int zo = 0; zo < RZ; ++zo)
#pragma unroll
        for (int yo = 0; yo < FY; ++yo) acc[zo][yo] = floatx4{0.f, 0.f, 0.f, 0.f};
      // lane's fragment offset per x-shift (output layer: at the row's own
      // voxels, and at the voxels beside rows 0 .. 3); every read below adds a
      // constant.  The empty asm keeps the compiler from hoisting 108
      // precomputed addresses out of the tile loop (which costs 108 registers).
      int base[OUT ? 2 : 3];
      if constexpr (OUT) {
        const int xe = r16 < 8 ? 0 : QX - 1;
        base[0] = (r16 + 1) * 32 + (g ^ swz(r16 + 1)) * 8;
        base[1] = (xe + QX * (r16 & 3)) * 32 + (g ^ swz(xe)) * 8;
        asm volatile("" : "+v"(base[0]), "+v"(base[1]));
      } else {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) base[dx] = (r16 + dx) * 32 + (g ^ swz(r16 + dx)) * 8;
        asm volatile("" : "+v"(base[0]), "+v"(base[1]), "+v"(base[2]));
      }
      // LDS offset of the slot that holds patch plane zb + zi
      int poff[RZ + 2];
#pragma unroll
      for (int zi = 0; zi < RZ + 2; ++zi) {
        const int sl = rot + zb + zi;
        poff[zi] = (sl >= RING ? sl - RING : sl) * CPLANE;
      }
      if constexpr (OUT) {
        edge = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int zi = 0; zi < 3; ++zi) {
          bf16x8 bfr[QY], efr[3];
#pragma unroll
          for (int yi = 0; yi < QY; ++yi)
            bfr[yi] = *reinterpret_cast<const bf16x8 *>(s_in + base[0] + poff[zi] + QX * yi * 32);
#pragma unroll
          for (int dy = 0; dy < 3; ++dy)
            efr[dy] = *reinterpret_cast<const bf16x8 *>(s_in + base[1] + poff[zi] + QX * dy * 32);
          __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the MFMAs
#pragma unroll
          for (int dy = 0; dy < 3; ++dy) {
#pragma unroll
            for (int yo = 0; yo < FY; ++yo)
              acc[0][yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[3 * zi + dy], bfr[yo + dy], acc[0][yo], 0, 0, 0);
            edge = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[3 * zi + dy], efr[dy], edge, 0, 0, 0);
          }
        }
      } else {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
#pragma unroll
          for (int zi = 0; zi < RZ + 2; ++zi) {
            // the row's six fragments are read together, so their LDS latency
            // overlaps instead of stalling the matrix core per fragment
            bf16x8 bfr[QY];
#pragma unroll
            for (int yi = 0; yi < QY; ++yi)
              bfr[yi] = *reinterpret_cast<const bf16x8 *>(s_in + base[dx] + poff[zi] + QX * yi * 32);
            __builtin_amdgcn_sched_barrier(0);  // keep the six reads ahead of the MFMAs
#pragma unroll
            for (int yi = 0; yi < QY; ++yi) {
#pragma unroll
              for (int dz = 0; dz < 3; ++dz) {
                const int zo = zi - dz;
                if (zo < 0 || zo >= RZ) continue;
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                  const int yo = yi - dy;
                  if (yo < 0 || yo >= FY) continue;
                  acc[zo][yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[9 * dz + 3 * dy + dx], bfr[yi],
                                                                        acc[zo][yo], 0, 0, 0);
                }
              }
            }
          }
        }
      }
      op = o;
      have_prev = true;
      if (more) {
        ++zt;
        rot = rot + CZ >= RING ? rot + CZ - RING : rot + CZ;
      } else {
        v += nb;
        if (v < T.nitems) {
          ci = col_item(T, v);
          zt = ci.zt0;
          fresh = true;
        }
      }
    }
    if (have_prev) epilogue(op);
  } else {
    // 8-channel input: chunk c covers taps 4c .. 4c + 3 (lane group g: tap 4c + g)
    bf16x8 wf[7][MT];
#pragma unroll
    for (int c = 0; c < 7; ++c)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        wf[c][m] = *reinterpret_cast<const bf16x8 *>(wk + ((c * COUTP + out_channel<MT>(m, r16)) * 32 + g * 8));
    for (int t = blockIdx.x; t < T.n; t += gridDim.x) {
      const TileOrigin o = fwd_tile(T, t);
      __syncthreads();
      stage_patch<CINP>(G, x, o, s_in);
      __builtin_amdgcn_s_waitcnt(0x0f70);
      __syncthreads();
#pragma unroll
      for (int pr = 0; pr < 4; ++pr) {
        floatx4 acc[2][MT];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int m = 0; m < MT; ++m) acc[i][m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 7; ++c) {
          const int tap = 4 * c + g;
          const bool live = tap < 27;
          const int tt = live ? tap : 0;
          const int dz = tt / 9, dy = (tt / 3) % 3, dxx = tt % 3;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int row = wid * 8 + pr * 2 + i;  // row = yo + FY * zo
            const int yo = row % FY, zo = row / FY;
            int v = (r16 + dxx) + QX * ((yo + dy) + QY * (zo + dz));
            bf16x8 bfr = *reinterpret_cast<const bf16x8 *>(s_in + v * 8);
            if (!live) bfr = bf16x8{};
#pragma unroll
            for (int m = 0; m < MT; ++m)
              acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[c][m], bfr, acc[i][m], 0, 0, 0);
          }
        }
        const int gx = o.x0 + r16;
        const uint32_t sy = (uint32_t)G.nx, sz = (uint32_t)G.nx * (uint32_t)G.ny;
        const size_t fb = (size_t)o.b * G.L * COUTP;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int row = wid * 8 + pr * 2 + i;
          const int gy = o.y0 + row % FY, gz = o.z0 + row / FY;
          const bool live = gx < G.nx && gy < G.ny && gz < G.nz;
          const uint32_t vi = (uint32_t)gx + sy * (uint32_t)gy + sz * (uint32_t)gz;
          if (live) wide_epilogue<EPI>(vi, g, acc[i], s_bias, y + fb, zpre ? zpre + fb : nullptr, zgate + fb);
        }
      }
    }
  }
}

// u [B][3][L] float -> BF16 channels-last [B][L][8], scaled by 1/scale[b], padded with zeros
__global__ void k_conv_prep_input(ConvGeom G, const float *__restrict__ u, const float *__restrict__ scale,
                                  uint16_t *__restrict__ x0) {
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (int64_t)G.B * G.L) return;
  int b = (int)(q / G.L);
  int64_t v = q - (int64_t)b * G.L;
  float is = 1.0f / scale[b];
  uint16_t h[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) h[c] = c < 3 ? f2bf(u[((int64_t)b * 3 + c) * G.L + v] * is) : (uint16_t)0;
  uint4 val = make_uint4(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16),
                         h[4] | ((uint32_t)h[5] << 16), h[6] | ((uint32_t)h[7] << 16));
  *reinterpret_cast<uint4 *>(x0 + q * 8) = val;
}

// Pack FP32 weights w[cout][cin][27] (torch layout, tap = 9 dz + 3 dy + dx)
// into [chunk][COUTP][32] BF16 fragments.  flip != 0 packs the weights of
// the transposed convolution instead (data gradient): taps mirrored
// (26 - tap) and the roles of cin and cout exchanged.
__global__ void k_conv_pack(const float *__restrict__ w, int cin, int cout, int flip, int cinp, int coutp,
                            uint16_t *__restrict__ wk) {
  int nchunk = cinp == 32 ? 27 : 7;
  int64_t total = (int64_t)nchunk * coutp * 32;
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= total) return;
  int k = (int)(q % 32);
  int m = (int)((q / 32) % coutp);
  int c = (int)(q / (32 * coutp));
  int tap, ci;
  if (cinp == 32) {
    tap = c;
    ci = k;
  } else {
    tap = 4 * c + k / 8;
    ci = k % 8;
  }
  // the packed layer maps `cin_l` input channels to `cout_l` outputs
  int cin_l = flip ? cout : cin, cout_l = flip ? cin : cout;
  float val = 0.f;
  if (tap < 27 && ci < cin_l && m < cout_l) {
    if (flip) val = w[((int64_t)ci * cin + m) * 27 + (26 - tap)];  // w[co = ci][ci = m][mirrored tap]
    else val = w[((int64_t)m * cin + ci) * 27 + tap];
  }
  wk[q] = f2bf(val);
}

// Weight and bias gradient of one layer on MFMA:
//   dW[tap][co][ci] = sum over voxels v of dz[v][co] * x[v + off(tap)][ci]
// (x zero-padded), dB[co] = sum over v of dz[v][co]: K = 32 voxels per MFMA,
// 16 along x of two z planes.  Both operands need their channels' voxels
// side by side while the fields are channels-last, so the fragments are read
// from LDS with the transposing read (ds_read_b64_tr_b16: 16 lanes read 4
// voxels of 16 channels, lane i receives the 4 voxels of channel i); no
// transposed copy is made anywhere.
//
// A workgroup (8 waves, one per CU for the 32 -> 32 layer) walks columns of
// 16 (x) x 4 (z) voxels along y.  A stage holds WG_Y rows of the column: x
// with a halo of one plane on either side in z, dz with a halo of one voxel
// on either side in x.  Shifting dz rather than x along x leaves the x
// fragments the same for the three dx taps, and each x row fragment stays in
// registers for the three rows of dz that use it: a step reads 3 + 3
// fragments for its 27 MFMAs.  Stages are copied into a ring of NBUF LDS
// buffers with buffer_load ... lds, NBUF - 1 stages ahead, across item
// boundaries, with one barrier per stage.  A wave owns 16 output x 16 input
// channels of one z pair, all 27 taps in registers; 3-channel fields (padded
// to 8) pack two z taps (x) or two x taps (dz) into one 16-wide operand.  The
// waves whose operand holds the unshifted dz take the bias gradient with one
// more MFMA against ones.  The z pairs are added in LDS, the workgroup's sums
// go to part[block], and k_conv_wgrad_reduce adds the blocks in a fixed
// order (bit-reproducible).
// Bound by the matrix cores and, behind them, by the 200 bytes read per
// voxel.  32 -> 32 at 16 x 64^3 voxels: 253 us for the whole call (950
// TFLOP/s in the kernel) against 5,898 us for a form that transposed each
// tile into LDS with 2-byte stores and summed the bias in a pass of its own;
// 3 -> 32 93 us (1,941), 32 -> 3 107 us (3,437); 1 x 64^3: 37, 23 and 23 us
// (574, 321, 432).
constexpr int WG_X = 16, WG_Z = 4, WG_Y = 3;
constexpr int WG_THREADS = 512;

struct WgPlan {
  int nx, ny, nz;
  int tx, tz, ncol;  // column tiles in x and z, columns over the batch
  int ylen, nitems;  // rows of a work item, items = columns x y segments
  int64_t L;
  int cin, cout;
};

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 *lds_bf16x4_t;

// MFMA operand fragment of 8 voxels per lane: two transposing reads, the
// second `step` bytes (4 voxels) on
__device__ __forceinline__ bf16x8 read_tr(lds_bytes_t p, int step) {
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t)p);
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t)(p + step));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int CINP, int ZS>
struct WgShape {
  static constexpr int XV = CINP / 8, ZV = ZS / 8;                            // 16-byte chunks per voxel
  static constexpr int NXC = WG_Y * (WG_Z + 2) * WG_X * XV;                   // chunks per stage
  static constexpr int NZC = WG_Y * WG_Z * (WG_X + 2) * ZV;
  static constexpr int XW = (NXC + 63) / 64, ZW = (NZC + 63) / 64;            // copies of one wave
  static constexpr int NL = (XW + ZW + WG_THREADS / 64 - 1) / (WG_THREADS / 64);  // copies per wave and stage
  // LDS buffers: 131 KB for 32 -> 32 (one workgroup per CU), two workgroups per CU for the others
  static constexpr int NBUF = CINP == 32 && ZS == 8 ? 3 : 4;
  static constexpr int XBYTES = XW * 1024, STAGE = XBYTES + ZW * 1024;
  static constexpr int NA = ZS == 32 ? 3 : 1;                                 // dz operands of a step (x shifts)
  static constexpr int NB = CINP == 32 ? 3 : 1;                               // x operands of a row (z taps)
  static constexpr int NACC = NA * 3 * NB + 1;                                // and the bias
  // one more 1 KB slot takes the copies that even out the waves' counts
  static constexpr int LDS = NBUF * STAGE + 1024;
  static_assert(LDS >= 4 * NACC * 1024, "the z pairs are added in the stage buffers");
};

template <int CINP, int ZS>
__global__ __launch_bounds__(WG_THREADS, 2) void k_conv_wgrad(WgPlan P, const uint16_t *__restrict__ x,
                                                              const uint16_t *__restrict__ dz,
                                                              float *__restrict__ part) {
  using S = WgShape<CINP, ZS>;
  __shared__ __attribute__((aligned(1024))) char s_buf[S::LDS];
  const lds_bytes_t lds0 = (lds_bytes_t)s_buf;
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (int)gridDim.x;
  // neighbouring columns to the workgroups of one XCD (dispatch is round-robin)
  const int v0 = (nb & 7) ? (int)blockIdx.x : ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
  const uint32_t lds_base = (uint32_t)(uintptr_t)lds0;

  // -- copies: the cursor runs S::NBUF - 1 stages ahead of the computation
  int iv = v0, ist = 0;                     // item and stage of the next copies
  int ib = 0, iy0 = 0, iys = 0, iye = 0;    // its field, first x row, dz row range
  int inst = 0, ibuf = 0;
  uint32_t ioff[S::NL];                     // byte offset of the lane's chunk at row 0 of the field
  bool iin[S::NL];                          // inside the field in x and z
  auto begin_item = [&]() {
    const int col = iv % P.ncol, seg = iv / P.ncol;
    const int x0 = (col % P.tx) * WG_X, r = col / P.tx;
    const int z0 = (r % P.tz) * WG_Z;
    ib = r / P.tz;
    iys = seg * P.ylen;
    iye = min(P.ny, iys + P.ylen);
    inst = (iye - iys + 2 + WG_Y - 1) / WG_Y;
#pragma unroll
    for (int k = 0; k < S::NL; ++k) {
      const int w = wid + k * (WG_THREADS / 64);
      if (w < S::XW) {
        const int q = w * 64 + lane, v = q / S::XV, c = q % S::XV;
        const int gx = x0 + v % WG_X, gz = z0 - 1 + (v / WG_X) % (WG_Z + 2);
        iin[k] = q < S::NXC && gx < P.nx && gz >= 0 && gz < P.nz;
        ioff[k] = (uint32_t)((gx + P.nx * P.ny * gz) * (CINP * 2) + c * 16);
      } else {
        const int q = (w - S::XW) * 64 + lane, v = q / S::ZV, c = q % S::ZV;
        const int gx = x0 - 1 + v % (WG_X + 2), gz = z0 + (v / (WG_X + 2)) % WG_Z;
        iin[k] = q < S::NZC && gx >= 0 && gx < P.nx && gz < P.nz;
        ioff[k] = (uint32_t)((gx + P.nx * P.ny * gz) * (ZS * 2) + c * 16);
      }
    }
  };
  auto issue = [&]() {
    const bool live = iv < P.nitems;  // past the last item: copies of zeros, so every stage counts the same
    if (live && ist == 0) begin_item();
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)(x + (int64_t)ib * P.L * CINP), (short)0,
                                                                        (int)(P.L * CINP * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc((void *)(dz + (int64_t)ib * P.L * ZS), (short)0,
                                                                        (int)(P.L * ZS * 2), 0x00020000);
#pragma unroll
    for (int k = 0; k < S::NL; ++k) {
      const int w = wid + k * (WG_THREADS / 64);
      if (w < S::XW) {
        const int row = (w * 64 + lane) / (S::XV * WG_X * (WG_Z + 2));
        const int gy = iys - 1 + ist * WG_Y + row;
        const bool in = live && iin[k] && gy >= 0 && gy < P.ny;
        copy_to_lds(rx, lds_base + ibuf * S::STAGE + w * 1024,
                    in ? ioff[k] + (uint32_t)(gy * P.nx * (CINP * 2)) : 0x80000000u);
      } else {
        // step t of the item takes x row iys - 1 + t and dz row iys - 2 + t
        const int row = ((w - S::XW) * 64 + lane) / (S::ZV * (WG_X + 2) * WG_Z);
        const int gy = iys - 2 + ist * WG_Y + row;
        const bool in = live && iin[k] && gy >= iys && gy < iye;
        const uint32_t dst = w < S::XW + S::ZW ? ibuf * S::STAGE + w * 1024 : S::NBUF * S::STAGE;
        copy_to_lds(rz, lds_base + dst, in ? ioff[k] + (uint32_t)(gy * P.nx * (ZS * 2)) : 0x80000000u);
      }
    }
    ibuf = ibuf + 1 == S::NBUF ? 0 : ibuf + 1;
    if (live && ++ist == inst) {
      ist = 0;
      iv += nb;
    }
  };

  // -- this wave's fragments.  Lane l: voxels 8 ((l >> 4) & 1) .. + 8 along x
  // of plane (l >> 5) of the z pair; it reads voxel (l & 15) >> 2 of a group of 4
  const int zp = wid >> 2, qa = wid & 1, qb = (wid >> 1) & 1;
  const int l16 = lane & 15, c4 = l16 & 3;
  const int vox = 8 * ((lane >> 4) & 1) + (l16 >> 2), zr = 2 * zp + (lane >> 5);
  int xa, za[S::NA];
  if (CINP == 32) xa = (zr * WG_X + vox) * 64 + (16 * qb + 4 * c4) * 2;
  else xa = ((zr + min(2 * qb + (c4 >> 1), 2)) * WG_X + vox) * 16 + (c4 & 1) * 8;  // two z taps side by side
#pragma unroll
  for (int a = 0; a < S::NA; ++a) {
    // tap dx pairs x at p with dz at p + 1 - dx; dz is staged from x0 - 1
    if (ZS == 32) za[a] = S::XBYTES + (zr * (WG_X + 2) + vox + 2 - a) * 64 + (16 * qa + 4 * c4) * 2;
    else za[a] = S::XBYTES + (zr * (WG_X + 2) + vox + 2 - min(2 * qa + (c4 >> 1), 2)) * 16 + (c4 & 1) * 8;
  }
  const bool bias_wave = qb == 0 && (ZS == 32 || qa == 0);
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  floatx4 acc[S::NACC];
#pragma unroll
  for (int a = 0; a < S::NACC; ++a) acc[a] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (int k = 0; k < S::NBUF - 1; ++k) issue();
  bf16x8 xf[3][S::NB];
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int k = 0; k < S::NB; ++k) xf[d][k] = bf16x8{};
  int buf = 0;
  for (int v = v0; v < P.nitems; v += nb) {
    const int ys = (v / P.ncol) * P.ylen;
    const int nsteps = min(P.ny, ys + P.ylen) - ys + 2;
    for (int t0 = 0; t0 < nsteps; t0 += WG_Y) {
      // this wave's copies of the stage have landed (the later stages' may be
      // in flight), then every wave's have, and every wave is done with the
      // stage before, whose buffer takes the next copies
      __builtin_amdgcn_s_waitcnt(0x0f70 | ((S::NBUF - 2) * S::NL));
      __syncthreads();
      issue();
      const lds_bytes_t st = lds0 + buf * S::STAGE;
      buf = buf + 1 == S::NBUF ? 0 : buf + 1;
#pragma unroll
      for (int r = 0; r < WG_Y; ++r) {
        static_assert(WG_Y == 3, "the x row of step r stays in register slot r");
        const int t = t0 + r;
#pragma unroll
        for (int k = 0; k < S::NB; ++k)
          xf[r][k] = read_tr(st + xa + (r * (WG_Z + 2) + k) * WG_X * CINP * 2, 4 * CINP * 2);
        if (t < 2 || t >= nsteps) continue;  // no dz row (uniform)
        bf16x8 zf[S::NA];
#pragma unroll
        for (int a = 0; a < S::NA; ++a) zf[a] = read_tr(st + za[a] + r * WG_Z * (WG_X + 2) * ZS * 2, 4 * ZS * 2);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int a = 0; a < S::NA; ++a)
#pragma unroll
            for (int k = 0; k < S::NB; ++k) {
              floatx4 &d = acc[(a * 3 + dy) * S::NB + k];
              d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[a], xf[(r + 1 + dy) % 3][k], d, 0, 0, 0);
            }
        if (bias_wave)
          acc[S::NACC - 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[S::NA == 3 ? 1 : 0], ones, acc[S::NACC - 1], 0,
                                                                     0, 0);
      }
    }
  }
  // add the z pairs: the copies still in flight land first
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();
  float4 *s_acc = reinterpret_cast<float4 *>(s_buf);
  if (zp == 1) {
#pragma unroll
    for (int a = 0; a < S::NACC; ++a)
      s_acc[((wid & 3) * S::NACC + a) * 64 + lane] = make_float4(acc[a][0], acc[a][1], acc[a][2], acc[a][3]);
  }
  __syncthreads();
  if (zp == 1) return;
  // lane holds D[m = 4 (l / 16) + j][n = l % 16]
  const int count = 27 * P.cin * P.cout + P.cout;
  float *out = part + (int64_t)blockIdx.x * count;
#pragma unroll
  for (int a = 0; a < S::NACC; ++a) {
    const float4 o = s_acc[((wid & 3) * S::NACC + a) * 64 + lane];
    const float sum[4] = {acc[a][0] + o.x, acc[a][1] + o.y, acc[a][2] + o.z, acc[a][3] + o.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = 4 * (lane >> 4) + j;
      const int co = ZS == 32 ? 16 * qa + m : (m & 7);
      if (a == S::NACC - 1) {
        // 8-channel dz: rows 8 .. 15 hold the unshifted tap
        if (bias_wave && l16 == 0 && co < P.cout && (ZS == 32 || m >= 8)) out[27 * P.cin * P.cout + co] = sum[j];
        continue;
      }
      const int dy = (a / S::NB) % 3;
      const int dx = ZS == 32 ? a / (3 * S::NB) : 2 * qa + (m >> 3);
      const int ci = CINP == 32 ? 16 * qb + l16 : (l16 & 7);
      const int dzt = CINP == 32 ? a % S::NB : 2 * qb + (l16 >> 3);
      if (co < P.cout && ci < P.cin && dx < 3 && dzt < 3)
        out[((9 * dzt + 3 * dy + dx) * P.cout + co) * P.cin + ci] = sum[j];
    }
  }
}

// dW[co][ci][tap] (+)= sum over blocks of part[block][tap][co][ci], and the
// bias gradient behind it: 64 entries per workgroup, four threads per entry
// over every fourth block (coalesced), their sums added in order.
__global__ __launch_bounds__(256) void k_conv_wgrad_reduce(const float *__restrict__ part, int nblocks, int cin,
                                                           int cout, float *__restrict__ dw, float *__restrict__ db,
                                                           int accumulate) {
  __shared__ float s_p[4][64];
  const int nw = 27 * cin * cout, count = nw + cout;
  const int e = threadIdx.x & 63, k0 = threadIdx.x >> 6;
  const int q = blockIdx.x * 64 + e;
  float s = 0.f;
  if (q < count) {
#pragma unroll 8
    for (int k = k0; k < nblocks; k += 4) s += part[(int64_t)k * count + q];
  }
  s_p[k0][e] = s;
  __syncthreads();
  if (k0 != 0 || q >= count) return;
  s = (s_p[0][e] + s_p[1][e]) + (s_p[2][e] + s_p[3][e]);
  float *dst;
  if (q < nw) {
    const int ci = q % cin, co = (q / cin) % cout, tap = q / (cin * cout);
    dst = dw + (co * cin + ci) * 27 + tap;
  } else {
    if (!db) return;
    dst = db + (q - nw);
  }
  *dst = accumulate ? *dst + s : s;
}

// Loss L = mean over b, c, v of ((u_out - u_tgt) / s_b)^2 and its gradient
// with respect to the net output y (u_out = u + s y): dL/dy = 2 (u_out -
// u_tgt) / (s_b count), written as BF16 [B][L][8]; per-block loss partials.
__global__ __launch_bounds__(256) void k_mse_grad(ConvGeom G, const float *__restrict__ u_out,
                                                  const float *__restrict__ u_tgt, const float *__restrict__ scale,
                                                  uint16_t *__restrict__ dy, float *__restrict__ loss_part) {
  __shared__ float red[256];
  int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float l = 0.f;
  double cnt = 3.0 * (double)G.B * (double)G.L;
  if (q < (int64_t)G.B * G.L) {
    int b = (int)(q / G.L);
    int64_t v = q - (int64_t)b * G.L;
    float is = 1.0f / scale[b];
    uint16_t h[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) h[c] = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      int64_t ui = ((int64_t)b * 3 + c) * G.L + v;
      float d = (u_out[ui] - u_tgt[ui]) * is;
      l += d * d;
      h[c] = f2bf((float)(2.0 * d / cnt));
    }
    uint4 val = make_uint4(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16), 0, 0);
    *reinterpret_cast<uint4 *>(dy + q * 8) = val;
  }
  red[threadIdx.x] = l;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss_part[blockIdx.x] = (float)(red[0] / cnt);
}

// Adam (Kingma & Ba 2015) on FP32 parameters.
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float bc1,
                       float bc2) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float gi = g[i];
  float mi = b1 * m[i] + (1.f - b1) * gi;
  float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// Per-field checks of a velocity field u [B][3][L] (solid [B][L] nullable,
// one mask per field): the sum of the squared central-difference divergence
// over interior fluid nodes, their count, and the kinetic energy 1/2 |u|^2
// summed over fluid nodes.  Pass 1: a workgroup takes rpi = 256 / nx rows
// of x per iteration (one row when nx >= 256), strides over the (y, z) rows
// of its field, and writes its three sums to part [B][nblk][3]; no node
// coordinate needs a 64-bit division and no two workgroups add to one
// address.  Pass 2 (k_field_stats_reduce) sums a field's partials in a
// fixed order in double, so the result does not depend on scheduling.
constexpr int FS_MAX_BLOCKS = 2048;

__host__ __device__ inline int fs_lanes_per_row(int nx) { return nx >= 256 ? 256 : nx; }

inline int fs_blocks(int nx, int ny, int nz) {
  const int64_t rpi = 256 / fs_lanes_per_row(nx);
  const int64_t need = ((int64_t)ny * nz + rpi - 1) / rpi;
  return (int)(need < FS_MAX_BLOCKS ? need : FS_MAX_BLOCKS);
}

__global__ __launch_bounds__(256) void k_field_stats(ConvGeom G, const float *__restrict__ u,
                                                     const uint8_t *__restrict__ solid, float *__restrict__ part) {
  __shared__ float r0[256 / 64], r1[256 / 64], r2[256 / 64];
  const int b = blockIdx.y;
  float dsum = 0.f, dcnt = 0.f, ke = 0.f;
  const float *ux = u + (int64_t)b * 3 * G.L, *uy = ux + G.L, *uz = uy + G.L;
  const uint8_t *sb = solid ? solid + (int64_t)b * G.L : nullptr;
  const int64_t sy = G.nx, sz = (int64_t)G.nx * G.ny;
  const int rows = G.ny * G.nz;
  const int lpr = fs_lanes_per_row(G.nx), rpi = 256 / lpr;
  const int sub = threadIdx.x / lpr, i0 = threadIdx.x - sub * lpr;
  if (sub < rpi) {
    for (int r = blockIdx.x * rpi + sub; r < rows; r += gridDim.x * rpi) {
      const int j = r % G.ny, k = r / G.ny;
      const bool inner_row = j > 0 && k > 0 && j < G.ny - 1 && k < G.nz - 1;
      const int64_t row0 = (int64_t)r * G.nx;
      for (int i = i0; i < G.nx; i += lpr) {
        const int64_t v = row0 + i;
        if (sb && sb[v]) continue;
        ke += 0.5f * (ux[v] * ux[v] + uy[v] * uy[v] + uz[v] * uz[v]);
        if (inner_row && i > 0 && i < G.nx - 1) {
          const float d = 0.5f * (ux[v + 1] - ux[v - 1] + uy[v + sy] - uy[v - sy] + uz[v + sz] - uz[v - sz]);
          dsum += d * d;
          dcnt += 1.f;
        }
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    dsum += __shfl_xor(dsum, o, 64);
    dcnt += __shfl_xor(dcnt, o, 64);
    ke += __shfl_xor(ke, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    r0[threadIdx.x >> 6] = dsum;
    r1[threadIdx.x >> 6] = dcnt;
    r2[threadIdx.x >> 6] = ke;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const float *rr = threadIdx.x == 0 ? r0 : threadIdx.x == 1 ? r1 : r2;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 256 / 64; ++w) t += rr[w];
    part[((int64_t)b * gridDim.x + blockIdx.x) * 3 + threadIdx.x] = t;
  }
}

// out[b][c] = sum over the nblk partials of field b (one workgroup per
// field; fixed summation order, double accumulation).
__global__ __launch_bounds__(256) void k_field_stats_reduce(int nblk, const float *__restrict__ part,
                                                            float *__restrict__ out) {
  __shared__ double s[3][256];
  const int b = blockIdx.x;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  for (int q = threadIdx.x; q < nblk; q += 256) {
    const float *pq = part + ((int64_t)b * nblk + q) * 3;
    a0 += pq[0];
    a1 += pq[1];
    a2 += pq[2];
  }
  s[0][threadIdx.x] = a0;
  s[1][threadIdx.x] = a1;
  s[2][threadIdx.x] = a2;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      s[0][threadIdx.x] += s[0][threadIdx.x + h];
      s[1][threadIdx.x] += s[1][threadIdx.x + h];
      s[2][threadIdx.x] += s[2][threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x < 3) out[b * 3 + threadIdx.x] = (float)s[threadIdx.x][0];
}

// Acceptance of surrogate fields on the device (no host synchronisation):
// from field_stats of the input fields (prev) and of the predictions (new),
// accept[b] = 1 iff the prediction's RMS divergence is at most div_factor
// times the input's and its kinetic energy is within [ke_lo, ke_hi] times
// the input's; a non-finite prediction makes its sums non-finite and fails
// both comparisons.  reject[b] = 1 - accept[b] (the skip flag of the
// fallback branch is the acceptance, its run flag the rejection).
__global__ void k_field_accept(int B, const float *__restrict__ prev, const float *__restrict__ pred,
                               float div_factor, float ke_lo, float ke_hi, int32_t *__restrict__ accept,
                               int32_t *__restrict__ reject) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const float rms0 = sqrtf(prev[3 * b] / fmaxf(prev[3 * b + 1], 1.f));
  const float rms1 = sqrtf(pred[3 * b] / fmaxf(pred[3 * b + 1], 1.f));
  const float ratio = pred[3 * b + 2] / fmaxf(prev[3 * b + 2], 1e-30f);
  const bool ok = (rms1 <= div_factor * rms0 + 1e-12f) && (ratio >= ke_lo) && (ratio <= ke_hi);
  accept[b] = ok ? 1 : 0;
  if (reject) reject[b] = ok ? 0 : 1;
}

// u_out[b] = accept[b] ? u_pred[b] with zero velocity on solid nodes : u_alt[b]
__global__ void k_field_select(int B, int64_t L, const int32_t *__restrict__ accept, const float *__restrict__ u_pred,
                               const float *__restrict__ u_alt, const uint8_t *__restrict__ solid,
                               float *__restrict__ u_out) {
  const int b = blockIdx.y;
  const bool ok = accept[b] != 0;
  const float *src = (ok ? u_pred : u_alt) + (int64_t)b * 3 * L;
  const uint8_t *sb = solid ? solid + (int64_t)b * L : nullptr;
  float *dst = u_out + (int64_t)b * 3 * L;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < L; v += (int64_t)gridDim.x * blockDim.x) {
    const bool zero = ok && sb && sb[v];
#pragma unroll
    for (int c = 0; c < 3; ++c) dst[c * L + v] = zero ? 0.f : src[c * L + v];
  }
}

static int make_geom(int B, int nx, int ny, int nz, ConvGeom *G) {
  DW_REQUIRE(B >= 1 && nx >= 1 && ny >= 1 && nz >= 1, DW_EINVAL, "conv: bad field size");
  DW_REQUIRE(nx <= (1 << 20) && ny <= (1 << 20) && nz <= (1 << 20), DW_ERANGE, "conv: field too large");
  G->B = B;
  G->nx = nx;
  G->ny = ny;
  G->nz = nz;
  G->L = (int64_t)nx * ny * nz;
  // byte offsets within one field's 32-channel activations fit 31 bits
  DW_REQUIRE(G->L * 64 < ((int64_t)1 << 31), DW_ERANGE, "conv: field too large (at most 2^25 voxels)");
  DW_REQUIRE(G->L * B < ((int64_t)1 << 31), DW_ERANGE, "conv: batch too large (at most 2^31 voxels)");
  return DW_OK;
}

static FwdTiles fwd_tiles(const ConvGeom &G) {
  FwdTiles T;
  T.tx = (G.nx + FX - 1) / FX;
  T.ty = (G.ny + FY - 1) / FY;
  T.tz = (G.nz + FZ - 1) / FZ;
  T.n = T.tx * T.ty * T.tz * G.B;
  // columns, cut into the z segments that leave the fullest of the 512
  // resident workgroups the fewest tiles, counting one more per segment for
  // its first patch (nothing runs beside that copy): 12 fields of 64^3 are 768
  // columns of 16 tiles, two rounds of whole columns or three of halves
  // (32 -> 32: 184 us as the former, 148 as the latter)
  T.tzc = (G.nz + CZ - 1) / CZ;
  T.ncol = T.tx * T.ty * G.B;
  int64_t best = INT64_MAX;
  const int most = std::min(T.tzc, std::max(32, 1024 / T.ncol));
  for (int segs = 1; segs <= most; ++segs) {
    const int len = (T.tzc + segs - 1) / segs;
    const int64_t items = (int64_t)T.ncol * ((T.tzc + len - 1) / len), cost = (items + 511) / 512 * (len + 1);
    if (cost < best) {
      best = cost;
      T.zlen = len;
      T.nitems = (int)items;
    }
  }
  return T;
}

// persistent grids: four (8-channel inputs) and two workgroups per CU
static unsigned fwd_blocks(const FwdTiles &T) { return (unsigned)(T.n < 1024 ? T.n : 1024); }
static unsigned col_blocks(const FwdTiles &T) { return (unsigned)(T.nitems < 512 ? T.nitems : 512); }

}  // namespace dw

using namespace dw;

extern "C" int conv_pack_weights(const float *w, int cin, int cout, int flip, uint16_t *wk, void *stream) {
  DW_REQUIRE(w && wk, DW_EINVAL, "conv_pack_weights: NULL pointer");
  DW_REQUIRE((cin == 3 || cin == 32) && (cout == 3 || cout == 32), DW_EINVAL,
             "conv_pack_weights: channels must be 3 or 32");
  int cin_l = flip ? cout : cin, cout_l = flip ? cin : cout;
  int cinp = cin_l == 3 ? 8 : 32, coutp = cout_l == 3 ? 16 : 32;
  int nchunk = cinp == 32 ? 27 : 7;
  int64_t total = (int64_t)nchunk * coutp * 32;
  hipLaunchKernelGGL(k_conv_pack, dim3(grid_blocks(total, 256)), dim3(256), 0, (hipStream_t)stream, w, cin, cout,
                     flip, cinp, coutp, wk);
  return check_launch("conv_pack_weights");
}

extern "C" size_t conv_packed_weight_elems(int cin, int cout) {
  int cinp = cin == 3 ? 8 : 32, coutp = cout == 3 ? 16 : 32;
  return (size_t)(cinp == 32 ? 27 : 7) * coutp * 32;
}

extern "C" int conv_prep_input(int B, int nx, int ny, int nz, const float *u, const float *scale, uint16_t *x0,
                               void *stream) {
  ConvGeom G;
  int rc = make_geom(B, nx, ny, nz, &G);
  if (rc) return rc;
  DW_REQUIRE(u && scale && x0, DW_EINVAL, "conv_prep_input: NULL pointer");
  hipLaunchKernelGGL(k_conv_prep_input, dim3(grid_blocks((int64_t)B * G.L, 256)), dim3(256), 0,
                     (hipStream_t)stream, G, u, scale, x0);
  return check_launch("conv_prep_input");
}

extern "C" int conv3d_bf16(int B, int nx, int ny, int nz, int cin, int cout, int epilogue, const uint16_t *x,
                           const uint16_t *wk, const float *bias, uint16_t *y, uint16_t *zpre, const uint16_t *zgate,
                           const float *u, const float *scale, float *u_out, void *stream) {
  ConvGeom G;
  int rc = make_geom(B, nx, ny, nz, &G);
  if (rc) return rc;
  DW_REQUIRE(x && wk, DW_EINVAL, "conv3d_bf16: x / weights NULL");
  DW_REQUIRE((cin == 3 || cin == 32) && (cout == 3 || cout == 32), DW_EINVAL, "conv3d_bf16: channels 3 or 32");
  hipStream_t s = (hipStream_t)stream;
  const FwdTiles T = fwd_tiles(G);
  const unsigned nb = fwd_blocks(T), nb32 = col_blocks(T);
  if (epilogue == DW_CONV_HIDDEN) {
    DW_REQUIRE(cout == 32 && bias && y, DW_EINVAL, "conv3d_bf16: hidden layer needs cout 32, bias, y");
    if (cin == 3)
      hipLaunchKernelGGL((k_conv<8, 32, DW_CONV_HIDDEN>), dim3(nb), dim3(256), 0, s, G, T, x, wk, bias, cout, y, zpre,
                         nullptr, nullptr, nullptr, nullptr);
    else
      hipLaunchKernelGGL((k_conv<32, 32, DW_CONV_HIDDEN>), dim3(nb32), dim3(256), 0, s, G, T, x, wk, bias, cout, y,
                         zpre, nullptr, nullptr, nullptr, nullptr);
  } else if (epilogue == DW_CONV_OUTPUT) {
    DW_REQUIRE(cin == 32 && cout == 3 && bias && u && scale && u_out, DW_EINVAL,
               "conv3d_bf16: output layer needs 32 -> 3, bias, u, scale, u_out");
    hipLaunchKernelGGL((k_conv<32, 16, DW_CONV_OUTPUT>), dim3(nb32), dim3(256), 0, s, G, T, x, wk, bias, cout, nullptr,
                       nullptr, nullptr, u, scale, u_out);
  } else if (epilogue == DW_CONV_DGRAD) {
    // transposed convolution of the gradient: input channels = the layer's cout
    DW_REQUIRE(cin == 32 && y && zgate, DW_EINVAL, "conv3d_bf16: data gradient needs cin 32 (the layer input), y, zgate");
    if (cout == 3)
      hipLaunchKernelGGL((k_conv<8, 32, DW_CONV_DGRAD>), dim3(nb), dim3(256), 0, s, G, T, x, wk, nullptr, 32, y,
                         nullptr, zgate, nullptr, nullptr, nullptr);
    else
      hipLaunchKernelGGL((k_conv<32, 32, DW_CONV_DGRAD>), dim3(nb32), dim3(256), 0, s, G, T, x, wk, nullptr, 32, y,
                         nullptr, zgate, nullptr, nullptr, nullptr);
  } else {
    return set_error(DW_EINVAL, "conv3d_bf16: unknown epilogue %d", epilogue);
  }
  return check_launch("conv3d_bf16");
}

constexpr int WGRAD_BLOCKS = 512;
constexpr int BGRAD_BLOCKS = 256;

extern "C" size_t conv_wgrad_scratch_floats(void) {
  return (size_t)WGRAD_BLOCKS * 27 * 32 * 32 + (size_t)BGRAD_BLOCKS * 32;
}

// Work items of the weight gradient: columns cut into y segments.  Every
// item reads two rows beyond its own and the last workgroups of an uneven
// division run alone, so the segment count is the one with the least rows on
// the busiest workgroup.
static WgPlan wgrad_plan(const ConvGeom &G, int cin, int cout, int blocks) {
  WgPlan P;
  P.nx = G.nx;
  P.ny = G.ny;
  P.nz = G.nz;
  P.L = G.L;
  P.cin = cin;
  P.cout = cout;
  P.tx = (G.nx + WG_X - 1) / WG_X;
  P.tz = (G.nz + WG_Z - 1) / WG_Z;
  P.ncol = P.tx * P.tz * G.B;
  int64_t best = INT64_MAX;
  P.ylen = G.ny;
  for (int segs = 1; segs <= (G.ny + 3) / 4; ++segs) {
    const int len = (G.ny + segs - 1) / segs;
    const int64_t items = (int64_t)P.ncol * ((G.ny + len - 1) / len);
    const int64_t rows = (items + blocks - 1) / blocks * (len + 2);
    if (rows < best) {
      best = rows;
      P.ylen = len;
    }
    if (items >= 8 * (int64_t)blocks) break;
  }
  P.nitems = P.ncol * ((G.ny + P.ylen - 1) / P.ylen);
  return P;
}

extern "C" int conv3d_bf16_wgrad(int B, int nx, int ny, int nz, int cin, int cout, const uint16_t *x,
                                 const uint16_t *dz, float *dw, float *db, int accumulate, float *scratch,
                                 void *stream) {
  ConvGeom G;
  int rc = make_geom(B, nx, ny, nz, &G);
  if (rc) return rc;
  DW_REQUIRE(x && dz && dw && scratch, DW_EINVAL, "conv3d_bf16_wgrad: NULL pointer");
  DW_REQUIRE((cin == 3 || cin == 32) && (cout == 3 || cout == 32), DW_EINVAL, "conv3d_bf16_wgrad: channels");
  if (cin == 3 && cout == 3)
    return set_error(DW_EINVAL, "conv3d_bf16_wgrad: unsupported layer %d -> %d", cin, cout);
  hipStream_t s = (hipStream_t)stream;
  // one workgroup per CU for 32 -> 32 (131 KB of LDS), two for the others
  const int most = cin == 32 && cout == 32 ? 256 : 512;
  const WgPlan P = wgrad_plan(G, cin, cout, most);
  const int nb = P.nitems < most ? P.nitems : most;
  if (cin == 3)
    hipLaunchKernelGGL((k_conv_wgrad<8, 32>), dim3(nb), dim3(WG_THREADS), 0, s, P, x, dz, scratch);
  else if (cout == 32)
    hipLaunchKernelGGL((k_conv_wgrad<32, 32>), dim3(nb), dim3(WG_THREADS), 0, s, P, x, dz, scratch);
  else
    hipLaunchKernelGGL((k_conv_wgrad<32, 8>), dim3(nb), dim3(WG_THREADS), 0, s, P, x, dz, scratch);
  hipLaunchKernelGGL(k_conv_wgrad_reduce, dim3(grid_blocks(27 * (int64_t)cin * cout + cout, 64)), dim3(256), 0, s,
                     scratch, nb, cin, cout, dw, db, accumulate);
  return check_launch("conv3d_bf16_wgrad");
}

extern "C" int conv_mse_grad(int B, int nx, int ny, int nz, const float *u_out, const float *u_tgt,
                             const float *scale, uint16_t *dy, float *loss_part, void *stream) {
  ConvGeom G;
  int rc = make_geom(B, nx, ny, nz, &G);
  if (rc) return rc;
  DW_REQUIRE(u_out && u_tgt && scale && dy && loss_part, DW_EINVAL, "conv_mse_grad: NULL pointer");
  hipLaunchKernelGGL(k_mse_grad, dim3(grid_blocks((int64_t)B * G.L, 256)), dim3(256), 0, (hipStream_t)stream, G,
                     u_out, u_tgt, scale, dy, loss_part);
  return check_launch("conv_mse_grad");
}

extern "C" int adam_step(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                         float eps, int step, void *stream) {
  DW_REQUIRE(p && g && m && v && n >= 0 && step >= 1, DW_EINVAL, "adam_step: bad arguments");
  float bc1 = 1.f - powf(b1, (float)step), bc2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(grid_blocks(n, 256)), dim3(256), 0, (hipStream_t)stream, p, g, m, v, n, lr, b1, b2,
                     eps, bc1, bc2);
  return check_launch("adam_step");
}

extern "C" size_t field_stats_workspace_bytes(int B, int nx, int ny, int nz) {
  if (B < 1 || B > 65535 || nx < 1 || ny < 1 || nz < 1 || (int64_t)ny * nz >= (1LL << 31)) return 0;
  return (size_t)B * fs_blocks(nx, ny, nz) * 3 * sizeof(float);
}

extern "C" int field_stats(int B, int nx, int ny, int nz, const float *u, const uint8_t *solid, float *out, void *ws,
                           size_t ws_bytes, void *stream) {
  DW_REQUIRE(B >= 1 && nx >= 1 && ny >= 1 && nz >= 1 && B <= 65535, DW_EINVAL, "field_stats: bad size");
  DW_REQUIRE(u && out && ws, DW_EINVAL, "field_stats: NULL pointer");
  DW_REQUIRE((int64_t)ny * nz < (1LL << 31), DW_ERANGE, "field_stats: too many rows");
  const int nblk = fs_blocks(nx, ny, nz);
  DW_REQUIRE(ws_bytes >= (size_t)B * nblk * 3 * sizeof(float), DW_EWORKSPACE, "field_stats: workspace too small");
  ConvGeom G{};
  G.B = B;
  G.nx = nx;
  G.ny = ny;
  G.nz = nz;
  G.L = (int64_t)nx * ny * nz;
  float *part = static_cast<float *>(ws);
  hipLaunchKernelGGL(k_field_stats, dim3(nblk, B), dim3(256), 0, (hipStream_t)stream, G, u, solid, part);
  int rc = check_launch("field_stats");
  if (rc) return rc;
  hipLaunchKernelGGL(k_field_stats_reduce, dim3(B), dim3(256), 0, (hipStream_t)stream, nblk, part, out);
  return check_launch("field_stats_reduce");
}

extern "C" int field_accept(int B, const float *stats_prev, const float *stats_pred, float div_factor, float ke_lo,
                            float ke_hi, int32_t *accept, int32_t *reject, void *stream) {
  DW_REQUIRE(B >= 1 && stats_prev && stats_pred && accept, DW_EINVAL, "field_accept: bad arguments");
  DW_REQUIRE(reject != accept, DW_EINVAL, "field_accept: reject must not alias accept");
  hipLaunchKernelGGL(k_field_accept, dim3(grid_blocks(B, 64)), dim3(64), 0, (hipStream_t)stream, B, stats_prev,
                     stats_pred, div_factor, ke_lo, ke_hi, accept, reject);
  return check_launch("field_accept");
}

extern "C" int field_select(int B, int nx, int ny, int nz, const int32_t *accept, const float *u_pred,
                            const float *u_alt, const uint8_t *solid, float *u_out, void *stream) {
  DW_REQUIRE(B >= 1 && B <= 65535 && nx >= 1 && ny >= 1 && nz >= 1, DW_EINVAL, "field_select: bad size");
  DW_REQUIRE(accept && u_pred && u_alt && u_out, DW_EINVAL, "field_select: NULL pointer");
  const int64_t L = (int64_t)nx * ny * nz;
  unsigned bx = grid_blocks(L, 256);
  if (bx > 2048) bx = 2048;
  hipLaunchKernelGGL(k_field_select, dim3(bx, B), dim3(256), 0, (hipStream_t)stream, B, L, accept, u_pred, u_alt,
                     solid, u_out);
  return check_launch("field_select");
}
