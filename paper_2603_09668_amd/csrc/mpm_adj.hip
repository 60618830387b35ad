// Hand-written adjoints of the MPM substep for gfx950.
//
// Reverse P2G is a gather per particle (each particle reads the grid adjoint
// at its 27 stencil nodes); reverse G2P is a sorted scatter (particles
// grouped by cell tile, the grid adjoint summed on the matrix cores into LDS
// node blocks and added to the global grid with float atomics); reverse grid
// update is pointwise over the active node tiles.  All adjoint outputs
// accumulate (+=).
//
// Forward definitions differentiated here: Eq. P2G with the MLS-MPM stress
// term A = m C - dt V0 (4/dx^2) tau(F), the explicit grid update of
// Eq. continuum_mechanics with the wind acceleration, Eq. G2P with the APIC
// affine matrix and Eq. deformation_update.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "dw_internal.h"
#include "dw_kernels.h"
#include "dw_scatter.h"

namespace dw {

// skew(y) as a 3x3 matrix
__device__ __forceinline__ void cross_matrix(const float y[3], float Z[9]) {
  Z[0] = 0.f;   Z[1] = -y[2]; Z[2] = y[1];
  Z[3] = y[2];  Z[4] = 0.f;   Z[5] = -y[0];
  Z[6] = -y[1]; Z[7] = y[0];  Z[8] = 0.f;
}

// Vector-Jacobian product of the polar rotation R(F), F = R S:
// dR = R W with W skew solving S W + W S = R^T dF - dF^T R; in vector form
// (tr(S) I - S) w = k.  For a cotangent Rbar this gives
// Fbar += 2 R [y]x with y = (tr(S) I - S)^{-1} g, g the axial vector of
// skew(R^T Rbar).
__device__ __forceinline__ void polar_vjp(const float *F, const float *R, const float *Rbar, float *Fbar) {
  float S[9], G[9];
  matmul3_atb(R, F, S);
  matmul3_atb(R, Rbar, G);
  float g[3] = {0.5f * (G[7] - G[5]), 0.5f * (G[2] - G[6]), 0.5f * (G[3] - G[1])};
  float tr = S[0] + S[4] + S[8];
  float M[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) M[q] = -0.5f * (S[q] + S[(q % 3) * 3 + q / 3]);
  M[0] += tr;
  M[4] += tr;
  M[8] += tr;
  float d = det3(M);
  float MiT[9];
  inv_transpose3(M, d, MiT);  // M symmetric: inverse = inverse-transpose
  float y[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) y[a] = MiT[3 * a] * g[0] + MiT[3 * a + 1] * g[1] + MiT[3 * a + 2] * g[2];
  float Z[9], RZ[9];
  cross_matrix(y, Z);
  matmul3(R, Z, RZ);
#pragma unroll
  for (int q = 0; q < 9; ++q) Fbar[q] += 2.0f * RZ[q];
}

// Vector-Jacobian product of the Kirchhoff stress tau(F; mu, lam), F = I + H.
//   Neo-Hookean: tau = mu (F F^T - I) + lam log J I
//     Fbar += mu (tb + tb^T) F + lam tr(tb) F^{-T}
//   fixed-corotated: tau = 2 mu (F - R) F^T + lam (J - 1) J I
//     Fbar += 2 mu tb F + 2 mu tb^T (F - R) + polar_vjp(Rbar = -2 mu tb F)
//             + lam (2J - 1) J tr(tb) F^{-T}
// Also returns the cotangents of mu and lam.  Y = R - I (fixed-corotated only).
__device__ __forceinline__ void kirchhoff_vjp(const float *H, const float *Y, float mu, float lam, int material,
                                              const float *tb, float *Fbar, float &mu_bar, float &lam_bar) {
  float F[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) F[q] = H[q] + ((q % 4) == 0 ? 1.f : 0.f);
  float Jm1 = det_shift(H);
  float J = 1.0f + Jm1;
  float FiT[9];
  inv_transpose3(F, J, FiT);
  float trt = tb[0] + tb[4] + tb[8];
  if (material == DW_NEO_HOOKEAN) {
    float S[9], SF[9], HHt[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) S[q] = tb[q] + tb[(q % 3) * 3 + q / 3];
    matmul3(S, F, SF);
#pragma unroll
    for (int q = 0; q < 9; ++q) Fbar[q] += mu * SF[q] + lam * trt * FiT[q];
    matmul3_abt(H, H, HHt);
    float mb = 0.f;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) mb += tb[3 * i + j] * (H[3 * i + j] + H[3 * j + i] + HHt[3 * i + j]);
    mu_bar = mb;
    lam_bar = trt * log1pf(Jm1);
  } else {
    float R[9], D[9], TF[9], TtD[9], Rb[9], DFt[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      D[q] = H[q] - Y[q];
      R[q] = Y[q] + ((q % 4) == 0 ? 1.f : 0.f);
    }
    matmul3(tb, F, TF);
    matmul3_atb(tb, D, TtD);
    float cj = lam * (2.f * J - 1.f) * J * trt;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      Fbar[q] += 2.f * mu * (TF[q] + TtD[q]) + cj * FiT[q];
      Rb[q] = -2.f * mu * TF[q];
    }
    polar_vjp(F, R, Rb, Fbar);
    matmul3_abt(D, F, DFt);
    float mb = 0.f;
#pragma unroll
    for (int q = 0; q < 9; ++q) mb += tb[q] * DFt[q];
    mu_bar = 2.f * mb;
    lam_bar = trt * Jm1 * J;
  }
}

// Weight and derivative of the wave-uniform offset oz alone: the z weights of
// a layer loop need no registers between the layers.
__device__ __forceinline__ void bspline_z(float f, int oz, float &w, float &dw) {
  const float t = f - (1.5f - 0.5f * (float)oz), k = oz == 1 ? -1.0f : 0.5f;
  w = (oz == 1 ? 0.75f : 0.0f) + k * t * t;
  dw = 2.0f * k * t;
}

// three consecutive floats (the x-neighbours of a stencil row)
struct AdjRow {
  float v[3];
};

// sum over the 64 lanes of a wave
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

struct PAdj {
  const float *x, *v, *C, *F, *mass, *vol0, *E, *nu;
  const float *xr;  // position reference or NULL
  const int32_t *region;
  int n, n_regions;
  float *xb, *vb, *Cb, *Fb, *Eb;
  float *Epart;     // deterministic mode: per-wave region sums [waves][n_regions]
  int fresh;        // vb and Cb hold nothing yet: written, not added to
  int slots;        // Eb is [workgroups][n_regions]: each workgroup adds to its own row
};

// ---------------------------------------------------------- reverse P2G
// One particle per thread: 27 values in, 36 gathers of three x-neighbours, 24
// adjoints read and written.  What bounds it is the chain of memory round
// trips of a wave (256k particles are four waves per SIMD in all) and the
// line lookups of the gathers (some 40 lines per wave and gather).  So the
// round trips are few: the whole particle at once, the twelve rows of a
// z-layer at once, the old adjoints at once (one += after the other costs a
// round trip each); H and R - I wait in LDS meanwhile, which spares a second
// polar decomposition, and E_bar takes one atomic per workgroup (one per wave
// took 52 us of 4,000 waves), or none: a rollout gives each workgroup a row of
// its own and adds the rows in double, which also brings the E adjoint of 20k
// particles from 1e-6 of the exact one to 1e-7.  256k particles 65 -> 35 us,
// with rows 30 (77 MB of particle data: 15 us), 20k 19.7 -> 14.5.
// DET: the E adjoint is not added with atomics; every wave writes its
// per-region sums (fixed-order wave reductions) to P.Epart and
// k_ebar_reduce adds the waves in index order.
constexpr int P2G_ADJ_THREADS = 512;  // largest workgroup (p2g_adj_threads chooses)

template <bool DET>
__global__ __launch_bounds__(P2G_ADJ_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_p2g_adj(
    GridDev g, PAdj P, float dt, int material, const float *__restrict__ mbar, const float *__restrict__ mvbar,
    int64_t N) {
  // H and Y of every thread's particle over the row loop: [wave][18][64]
  extern __shared__ float s_keep_all[];
  float *s_keep = s_keep_all + (threadIdx.x >> 6) * (18 * 64) + (threadIdx.x & 63);
  const int n = P.n;
  float *const Eb = P.slots ? P.Eb + (size_t)blockIdx.x * P.n_regions : P.Eb;
  int run_reg = -1;      // region of the wave's running E sum (float atomics)
  float run_sum = 0.f;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; (p & ~63) < n; p += gridDim.x * blockDim.x) {
    const bool live = p < n;
    const uint32_t off = 4u * (uint32_t)p;
    float Ebar_p = 0.f;
    int r = 0;
    if (live) {
      // all of the particle in one round trip
      float F[9], Cm[9], vp[3];  // F holds H = F - I
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        F[q] = at_particle(P.F, q, n, off);
        Cm[q] = at_particle(P.C, q, n, off);
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) vp[a] = at_particle(P.v, a, n, off);
      const float m = at_particle(P.mass, 0, n, off), V0 = at_particle(P.vol0, 0, n, off);
      const int rp = at_particle(P.region, 0, n, off);
      const Coord cx = load_coord(P.xr, P.x, p, g.ox, g.inv_dx);
      const Coord cy = load_coord(P.xr, P.x, (size_t)n + p, g.oy, g.inv_dx);
      const Coord cz = load_coord(P.xr, P.x, 2 * (size_t)n + p, g.oz, g.inv_dx);
      const float X = coord_sum(cx), Y = coord_sum(cy), Z = coord_sum(cz);
      bool ok = isfinite(X) && isfinite(Y) && isfinite(Z) && fabsf(X) < 1e9f && fabsf(Y) < 1e9f && fabsf(Z) < 1e9f;
      int bx = 0, by = 0, bz = 0;
      if (ok) {
        bx = base_of(X); by = base_of(Y); bz = base_of(Z);
        ok = stencil_inside(g, bx, by, bz);
      }
      if (ok) {
        float f[3] = {coord_frac(cx, bx), coord_frac(cy, by), coord_frac(cz, bz)};
        float tau[9], A[9];  // A holds dx A
        r = rp;
        float Er = P.E[r], nur = P.nu[r];
        float mu, lam;
        lame(Er, nur, mu, lam);
        float Y[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        kirchhoff_shift(F, mu, lam, material, tau, nullptr, Y);
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          s_keep[q * 64] = F[q];
          s_keep[(9 + q) * 64] = Y[q];
        }
        float ks = dt * 4.0f * g.inv_dx * g.inv_dx;
#pragma unroll
        for (int q = 0; q < 9; ++q) A[q] = g.dx * (m * Cm[q] - ks * V0 * tau[q]);
        const float mom[3] = {m * vp[0], m * vp[1], m * vp[2]};
        float w[2][3], dw[2][3];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          bspline_w(f[a], w[a]);
          bspline_dw(f[a], dw[a]);
        }
        const float dx = g.dx;
        // Per node n (offset o, weight w_n, gradient gw_n, d_n = (o - f) dx):
        //   v_bar += m w gb,  A_bar += w gb d^T,
        //   x_bar += gw s - w A^T gb  with s = m mb + gb . (mom + A d).
        // Per row the x-neighbours reduce to Sw = sum w s, Sd = sum dw s, T = sum
        // w gb and U = sum w (ox - fx) gb, which the y and z weights then scale
        // (G = sum w gb: v_bar = m G, and the A^T term is A^T G).
        float G[3] = {0.f, 0.f, 0.f}, X[3] = {0.f, 0.f, 0.f};
        float O[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // The three rows of a z-layer together: twelve 12-byte loads (the three
        // x-neighbours of a row and array) in flight
#pragma unroll 1
        for (int oz = 0; oz < 3; ++oz) {
          const int64_t row0 = bx + (int64_t)g.nx * (by + (int64_t)g.ny * (bz + oz));
          AdjRow rm[3], rv[3][3];
#pragma unroll
          for (int oy = 0; oy < 3; ++oy) {
            const int64_t row = row0 + (int64_t)g.nx * oy;
            __builtin_memcpy(&rm[oy], mbar + row, sizeof(AdjRow));
#pragma unroll
            for (int a = 0; a < 3; ++a) __builtin_memcpy(&rv[oy][a], mvbar + a * N + row, sizeof(AdjRow));
          }
          float wz, dwz;
          bspline_z(f[2], oz, wz, dwz);
          const float dz = (float)oz - f[2];
          float cz3[3], Gz[3] = {0.f, 0.f, 0.f};
#pragma unroll
          for (int a = 0; a < 3; ++a) cz3[a] = mom[a] + A[3 * a + 2] * dz;
#pragma unroll
          for (int oy = 0; oy < 3; ++oy) {
            float Sw = 0.f, Sd = 0.f, T[3] = {0.f, 0.f, 0.f}, U[3] = {0.f, 0.f, 0.f};
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
              float s = m * rm[oy].v[ox];
#pragma unroll
              for (int a = 0; a < 3; ++a) {
                s += rv[oy][a].v[ox] * (cz3[a] + A[3 * a + 1] * ((float)oy - f[1]) + A[3 * a] * ((float)ox - f[0]));
                const float t = w[0][ox] * rv[oy][a].v[ox];
                T[a] += t;
                U[a] += ((float)ox - f[0]) * t;
              }
              Sw += w[0][ox] * s;
              Sd += dw[0][ox] * s;
            }
            const float wyz = w[1][oy] * wz;
            X[0] += wyz * Sd;
            X[1] += dw[1][oy] * wz * Sw;
            X[2] += w[1][oy] * dwz * Sw;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
              const float t = wyz * T[a];
              Gz[a] += t;
              O[3 * a] += wyz * U[a];
              O[3 * a + 1] += ((float)oy - f[1]) * t;
            }
          }
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            G[a] += Gz[a];
            O[3 * a + 2] += dz * Gz[a];
          }
        }
        // the old values of every adjoint in one round trip
        float vo[3] = {0.f, 0.f, 0.f}, xo[3] = {0.f, 0.f, 0.f}, Co[9], Fo[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) Co[q] = Fo[q] = 0.f;
        if (P.vb && !P.fresh) {
#pragma unroll
          for (int a = 0; a < 3; ++a) vo[a] = at_particle(P.vb, a, n, off);
        }
        if (P.xb) {
#pragma unroll
          for (int a = 0; a < 3; ++a) xo[a] = at_particle(P.xb, a, n, off);
        }
        if (P.Cb && !P.fresh) {
#pragma unroll
          for (int q = 0; q < 9; ++q) Co[q] = at_particle(P.Cb, q, n, off);
        }
        if (P.Fb) {
#pragma unroll
          for (int q = 0; q < 9; ++q) Fo[q] = at_particle(P.Fb, q, n, off);
        }
        float vbar[3], xbar[3], Abar[9];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          vbar[a] = m * G[a];
          // d (A d) / d x = -A   ->   -A^T G
          xbar[a] = g.inv_dx * (X[a] - (A[a] * G[0] + A[3 + a] * G[1] + A[6 + a] * G[2]));
#pragma unroll
          for (int b = 0; b < 3; ++b) Abar[3 * a + b] = dx * O[3 * a + b];
        }
        if (P.vb) {
#pragma unroll
          for (int a = 0; a < 3; ++a) at_particle(P.vb, a, n, off) = vo[a] + vbar[a];
        }
        if (P.xb) {
#pragma unroll
          for (int a = 0; a < 3; ++a) at_particle(P.xb, a, n, off) = xo[a] + xbar[a];
        }
        if (P.Cb) {
#pragma unroll
          for (int q = 0; q < 9; ++q) at_particle(P.Cb, q, n, off) = Co[q] + m * Abar[q];
        }
        if (P.Fb || P.Eb) {
          float H[9], Yr[9], tb[9], Fb[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < 9; ++q) {
            tb[q] = -ks * V0 * Abar[q];
            H[q] = s_keep[q * 64];
            Yr[q] = s_keep[(9 + q) * 64];
          }
          float mu_b, lam_b;
          kirchhoff_vjp(H, Yr, mu, lam, material, tb, Fb, mu_b, lam_b);
          if (P.Fb) {
#pragma unroll
            for (int q = 0; q < 9; ++q) at_particle(P.Fb, q, n, off) = Fo[q] + Fb[q];
          }
          // Eq. young_poisson: d mu / d E = 1 / (2 (1 + nu)), d lam / d E = nu / ((1 + nu)(1 - 2 nu))
          Ebar_p = mu_b / (2.f * (1.f + nur)) + lam_b * nur / ((1.f + nur) * (1.f - 2.f * nur));
        }
      }
    }
    if (P.Eb && DET) {
      // lane l of the wave keeps the sum of region r0 + l; one store per entry
      const int lane = threadIdx.x & 63;
      const int64_t wave = p >> 6;
      for (int r0 = 0; r0 < P.n_regions; r0 += 64) {
        float mine_sum = 0.f;
        unsigned long long pending = __ballot(live && r >= r0 && r < r0 + 64);
        while (pending) {
          const int leader = __ffsll(pending) - 1;
          const int rk = __shfl(r, leader, 64);
          const bool mine = live && r == rk;
          const float sum = wave_sum(mine ? Ebar_p : 0.f);
          if (lane == rk - r0) mine_sum = sum;
          pending &= ~__ballot(mine);
        }
        if (r0 + lane < P.n_regions) P.Epart[wave * P.n_regions + r0 + lane] = mine_sum;
      }
    } else if (P.Eb) {
      // a wave holds few regions: it sums each over its lanes
      unsigned long long pending = __ballot(live);
      const int lane = threadIdx.x & 63;
      if (!__ballot(live && r == run_reg)) {
        if (run_reg >= 0 && lane == 0 && run_sum != 0.f) atomicAdd(&Eb[run_reg], run_sum);
        run_reg = __builtin_amdgcn_readfirstlane(r);  // lane 0 of the loop is live
        run_sum = 0.f;
      }
      while (pending) {
        const int leader = __ffsll(pending) - 1;
        const int rk = __shfl(r, leader, 64);
        const bool mine = live && r == rk;
        const float sum = wave_sum(mine ? Ebar_p : 0.f);
        if (rk == run_reg) run_sum += sum;
        else if (lane == leader && sum != 0.f) atomicAdd(&Eb[rk], sum);
        pending &= ~__ballot(mine);
      }
    }
  }
  if (P.Eb && !DET) {
    // the waves' running sums merged over the workgroup
    __shared__ float s_sum[P2G_ADJ_THREADS / 64];
    __shared__ int s_reg[P2G_ADJ_THREADS / 64];
    const int nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) {
      s_reg[threadIdx.x >> 6] = run_reg;
      s_sum[threadIdx.x >> 6] = run_sum;
    }
    __syncthreads();
    if ((int)threadIdx.x < nw && s_reg[threadIdx.x] >= 0) {
      const int rk = s_reg[threadIdx.x];
      bool lead = true;
      float sum = 0.f;
      for (int w = 0; w < nw; ++w) {
        if (s_reg[w] != rk) continue;
        lead = lead && w >= (int)threadIdx.x;
        sum += s_sum[w];
      }
      if (lead && sum != 0.f) atomicAdd(&Eb[rk], sum);
    }
  }
}

// Workgroup size of the reverse P2G: the largest of 64 .. 512 that still
// gives every CU one, so that a small set spreads over the chip and a large
// one issues few E atomics.
static int p2g_adj_threads(int n) {
  int t = 64;
  while (t < P2G_ADJ_THREADS && (int64_t)n >= (int64_t)2 * t * cu_count()) t *= 2;
  return t;
}

// ... and how many: at most as many as fit at once, four waves per SIMD
static unsigned p2g_adj_blocks(int n) {
  const int threads = p2g_adj_threads(n);
  return std::min(grid_blocks(n, threads), (unsigned)(1024 / threads * cu_count()));
}

// E_bar += the column sums of the workgroups' rows, one wave per region, in
// double: hundreds of float additions into a sum whose terms cancel lose more
// than the terms do
__global__ __launch_bounds__(64) void k_e_slots(const float *__restrict__ slots, int rows, int R,
                                                float *__restrict__ Eb) {
  double t = 0.0;
  for (int b = threadIdx.x; b < rows; b += 64) t += (double)slots[(size_t)b * R + blockIdx.x];
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if (threadIdx.x == 0) Eb[blockIdx.x] += (float)t;
}

// E adjoint of the deterministic reverse P2G: region r adds the per-wave sums
// in wave order.
__global__ __launch_bounds__(64) void k_ebar_reduce(const float *__restrict__ part, int64_t waves, int R,
                                                    float *__restrict__ Eb) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  float s = 0.f;
  for (int64_t w = 0; w < waves; ++w) s += part[w * R + r];
  Eb[r] += s;
}

// --------------------------------------------------- reverse grid update

// v + v of the lane CTRL names (a DPP move within the row of 16)
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// W_bar += the force grid's trilinear transpose of the acceleration adjoints
// ab that the lanes of a wave hold (the nodes of one tile; any may be zero).
// A wind cell is usually wider than a node, so that a tile reaches at most four
// wind nodes per axis: the transpose then runs axis by axis, the four lanes
// along an axis adding their shares of each wind node and lane c keeping wind
// node c, and each lane ends with one wind node's three sums.  (36 lane sums
// in all; summing the 24 corner values of each wind cell over the wave took 7
// us more.)  A finer wind grid's nodes add their own shares.  A share is
// selected, not multiplied by zero: a NaN stays in its cell's corners.
__device__ __forceinline__ void force_grid_transpose(const WindDev &w, const GridDev &g, int i, int j, int k,
                                                     const float ab[3], float *__restrict__ Wbar) {
  const bool on = ab[0] != 0.f || ab[1] != 0.f || ab[2] != 0.f;
  if (!__ballot(on)) return;
  const int lane = threadIdx.x & 63;
  const float q[3] = {fminf(fmaxf((g.ox + g.dx * (float)i - w.lox) * w.sx, 0.f), (float)(w.nwx - 1)),
                      fminf(fmaxf((g.oy + g.dx * (float)j - w.loy) * w.sy, 0.f), (float)(w.nwy - 1)),
                      fminf(fmaxf((g.oz + g.dx * (float)k - w.loz) * w.sz, 0.f), (float)(w.nwz - 1))};
  const int nw[3] = {w.nwx, w.nwy, w.nwz}, step[3] = {lane & 3, (lane >> 2) & 3, lane >> 4};
  int ic[3], c0[3];
  float t[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lin_axis(q[d], nw[d], ic[d], t[d]);
    c0[d] = __builtin_amdgcn_readlane(ic[d], 0);  // the tile's first wind node
  }
  if (__ballot(ic[0] - c0[0] > 2 || ic[1] - c0[1] > 2 || ic[2] - c0[2] > 2)) {
    if (!on) return;
    for (int e = 0; e < 8; ++e) {
      const float wt = ((e & 1) ? t[0] : 1.f - t[0]) * ((e & 2) ? t[1] : 1.f - t[1]) * ((e & 4) ? t[2] : 1.f - t[2]);
      const int64_t idx =
          (ic[0] + (e & 1)) + (int64_t)w.nwx * ((ic[1] + ((e >> 1) & 1)) + (int64_t)w.nwy * (ic[2] + (e >> 2)));
      for (int a = 0; a < 3; ++a) atomicAdd(&Wbar[a * w.nw3 + idx], wt * ab[a]);
    }
    return;
  }
  float v[3] = {ab[0], ab[1], ab[2]};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    float keep[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int r = c - (ic[d] - c0[d]);  // 0: the cell's lower node, 1: its upper one
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        float u = r == 0 ? (1.f - t[d]) * v[a] : (r == 1 ? t[d] * v[a] : 0.f);
        if (d == 0) {
          u = dpp_add<0xB1>(u);  // quad_perm: the other one of the pair,
          u = dpp_add<0x4E>(u);  // the other pair
        } else if (d == 1) {
          u = dpp_add<0x124>(u);  // row_ror by 4, by 8
          u = dpp_add<0x128>(u);
        } else {
          u += __shfl_xor(u, 16, 64);
          u += __shfl_xor(u, 32, 64);
        }
        if (step[d] == c) keep[a] = u;
      }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = keep[a];
  }
  const int64_t idx = (c0[0] + step[0]) + (int64_t)w.nwx * ((c0[1] + step[1]) + (int64_t)w.nwy * (c0[2] + step[2]));
#pragma unroll
  for (int a = 0; a < 3; ++a)
    if (v[a] != 0.f) atomicAdd(&Wbar[a * w.nw3 + idx], v[a]);
}

// One node per lane, a node tile per wave.  FUSED (a rollout's reverse
// substep, force-grid wind): gmb and gmvb are written for every node of the
// active tiles (zero where the node has no mass or is pinned) instead of added
// to, gvb is cleared once read, which leaves it zero for the next substep's
// scatter, and ab goes straight into Wbar: no clear of ten grid arrays, no
// array accb and no pass over all nodes for the transpose (96^3 nodes, 16^3
// wind grid: 8 + 15 us and the clear -> 11).
template <bool FUSED>
__global__ __launch_bounds__(256) void k_grid_update_adj(GridDev g, float dt, float gx, float gy, float gz,
                                                         int bound, const float *__restrict__ gm,
                                                         const float *__restrict__ gmv, WindDev wind,
                                                         const uint8_t *__restrict__ pin,
                                                         const int32_t *__restrict__ node_tiles,
                                                         const int32_t *__restrict__ n_tiles,
                                                         float *__restrict__ gvb, float *__restrict__ gmb,
                                                         float *__restrict__ gmvb, float *__restrict__ accb,
                                                         float *__restrict__ Wbar, int64_t N) {
  int nt = *n_tiles;
  int sub = threadIdx.x >> 6, l = threadIdx.x & 63;
  for (int it = blockIdx.x * 4 + sub; it < nt; it += gridDim.x * 4) {
    int t = node_tiles[it];
    int tx = t % g.tx, ty = (t / g.tx) % g.ty, tz = t / (g.tx * g.ty);
    int i = tx * 4 + (l & 3), j = ty * 4 + ((l >> 2) & 3), k = tz * 4 + (l >> 4);
    const bool in_grid = i < g.nx && j < g.ny && k < g.nz;
    if (!FUSED && !in_grid) continue;
    const int64_t node = in_grid ? i + (int64_t)g.nx * (j + (int64_t)g.ny * k) : 0;
    const float m = in_grid ? gm[node] : 0.f;
    const bool on = m > 0.f && !(pin && pin[node]);
    if (!FUSED && !on) continue;
    float vb[3], mvb[3] = {0.f, 0.f, 0.f}, mb = 0.f, ab[3] = {0.f, 0.f, 0.f};
    if (FUSED && in_grid) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        vb[a] = gvb[a * N + node];
        gvb[a * N + node] = 0.f;
      }
    }
    if (on) {
      float im = 1.0f / m;
      float mv[3] = {gmv[node], gmv[N + node], gmv[2 * N + node]};
      const float vs[3] = {mv[0] * im, mv[1] * im, mv[2] * im};
      float ax, ay, az;
      wind_at_node(wind, g, i, j, k, node, vs[0], vs[1], vs[2], ax, ay, az);
      float v[3] = {vs[0] + dt * (gx + ax), vs[1] + dt * (gy + ay), vs[2] + dt * (gz + az)};
      if (!FUSED) {
#pragma unroll
        for (int a = 0; a < 3; ++a) vb[a] = gvb[a * N + node];
      }
      if ((i < bound && v[0] < 0.f) || (i >= g.nx - bound && v[0] > 0.f)) vb[0] = 0.f;
      if ((j < bound && v[1] < 0.f) || (j >= g.ny - bound && v[1] > 0.f)) vb[1] = 0.f;
      if ((k < bound && v[2] < 0.f) || (k >= g.nz - bound && v[2] > 0.f)) vb[2] = 0.f;
      // adjoint of the acceleration, and of the wind velocity U and of v* for
      // the relative drag a = k |r| r, r = U - v*: with J = k (|r| I + r r^T / |r|)
      // U_bar = J a_bar and v*_bar gets -J a_bar
      float vsb[3] = {vb[0], vb[1], vb[2]};
#pragma unroll
      for (int a = 0; a < 3; ++a) ab[a] = dt * vb[a];
      if (wind.mode == DW_WIND_LBM_DRAG_REL) {
        float U[3];
        float r[3] = {0.f, 0.f, 0.f};
        if (wind_velocity_at_node(wind, g, i, j, k, U[0], U[1], U[2])) {
          r[0] = U[0] - vs[0];
          r[1] = U[1] - vs[1];
          r[2] = U[2] - vs[2];
        }
        const float sp = sqrtf(r[0] * r[0] + r[1] * r[1] + r[2] * r[2]);
        float Jab[3] = {0.f, 0.f, 0.f};
        if (sp > 0.f) {
          const float rb = (r[0] * ab[0] + r[1] * ab[1] + r[2] * ab[2]) / sp;
#pragma unroll
          for (int a = 0; a < 3; ++a) Jab[a] = wind.k_drag * (sp * ab[a] + r[a] * rb);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          vsb[a] -= Jab[a];
          ab[a] = Jab[a];
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) mvb[a] = vsb[a] * im;
      mb = -(vsb[0] * mv[0] + vsb[1] * mv[1] + vsb[2] * mv[2]) * im * im;
    }
    if (FUSED) {
      if (in_grid) {
        gmb[node] = mb;
#pragma unroll
        for (int a = 0; a < 3; ++a) gmvb[a * N + node] = mvb[a];
      }
      force_grid_transpose(wind, g, i, j, k, ab, Wbar);
    } else {
      if (gmvb) {
#pragma unroll
        for (int a = 0; a < 3; ++a) gmvb[a * N + node] += mvb[a];
      }
      if (gmb) gmb[node] += mb;
      if (accb) {
#pragma unroll
        for (int a = 0; a < 3; ++a) accb[a * N + node] += ab[a];
      }
    }
  }
}

// ---------------------------------------------------------- reverse G2P

// Reverse G2P.  One workgroup per work item (a chunk of at most WORK_CHUNK
// sorted particles of one cell tile), one particle per thread.  Each thread
// applies the adjoints of the x, F and C updates and gathers the grid
// velocities once, for C_p of the forward and for x_bar; the scatter of the
// grid-velocity adjoint, v_bar_i += w_ip (vbt_p + kc Cbt_p (o - f_p)), has
// the P2G form w (q + A o) with q = vbt - kc Cbt f, A = kc Cbt and runs as
// the tile scatter of dw_scatter.h; node owners add the result into the
// global grid adjoint with float atomics.  DET: the particles of a cell take
// their slots in index order and the node owners write the item's 6^3 block
// to item_part instead, which k_det_gather<true> then adds to the grid
// adjoint in a fixed order (bit-reproducible with a deterministic sort).
// An item is a chain of phases with two workgroups per CU to overlap them
// (128 registers, 80 KB of LDS): the particle is loaded in one round trip
// ahead of the slot scan, one gather replaces two (v_p itself is not needed),
// and the row sums factor.  256k particles (735 items) 60 -> 41 us, 20k 23.3
// -> 15.5.
template <bool DET>
__global__ __launch_bounds__(SC_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_g2p_adj(
    GridDev g, float dt, const float *__restrict__ gv, int64_t N, const float *__restrict__ x,
    const float *__restrict__ xr, const float *__restrict__ F, int n, const float *__restrict__ xob, const float *__restrict__ vob,
    const float *__restrict__ Cob, const float *__restrict__ Fob, float *__restrict__ xb, float *__restrict__ Fb,
    float *__restrict__ gvb, const int32_t *__restrict__ perm, const int32_t *__restrict__ tile_start,
    const int32_t *__restrict__ item_tile, const int32_t *__restrict__ item_begin,
    const int32_t *__restrict__ n_items, float *__restrict__ item_part, int fresh) {
  __shared__ float s_dat[(SC_DAT - 1) * SC_PITCH + SC_TAIL];  // staged features in cell order
  __shared__ float s_wgt[SC_WGT * SC_PITCH + SC_TAIL];  // and weights
  __shared__ unsigned char s_cell[WORK_CHUNK];
  __shared__ __attribute__((aligned(16))) float s_node[SC_WAVES][SC_NODES][4];
  __shared__ int s_cnt[64], s_off[64], s_cur[64];
  __shared__ int s_udesc[SC_MAX_UNITS];
  __shared__ int s_nunits;
  __shared__ float s_gv[3][SC_NODES];  // grid velocities of the item's 6^3 node region
  float *s_node_flat = &s_node[0][0][0];
  const int ni = *n_items;
  const float kc = 4.0f * g.inv_dx;
  for (int it = blockIdx.x; it < ni; it += gridDim.x) {
    int tid = threadIdx.x;
    asm("" : "+v"(tid));  // what depends on it is made in the item's own phases: held over the items it would spill
    const int lane = tid & 63, wid = tid >> 6;
    const int tile = item_tile[it];
    const int b0 = item_begin[it];
    const int nb = min(WORK_CHUNK, tile_start[tile + 1] - b0);
    const int tx = tile % g.tx, ty = (tile / g.tx) % g.ty, tz = tile / (g.tx * g.ty);
    if (tid < 64) s_cnt[tid] = 0;
    for (int q = tid; q < SC_WAVES * SC_NODES; q += SC_THREADS)
      reinterpret_cast<float4 *>(s_node_flat)[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    // every stencil of the item lies in the tile's 6^3 node region: stage its
    // grid velocities for the gather below
    if (tid < SC_NODES) {
      const int gx = 4 * tx + tid % SC_L, gy = 4 * ty + (tid / SC_L) % SC_L, gz = 4 * tz + tid / (SC_L * SC_L);
      float a0 = 0.f, a1 = 0.f, a2 = 0.f;
      if (gx < g.nx && gy < g.ny && gz < g.nz) {
        const int64_t node = gx + (int64_t)g.nx * (gy + (int64_t)g.ny * gz);
        a0 = gv[node];
        a1 = gv[N + node];
        a2 = gv[2 * N + node];
      }
      s_gv[0][tid] = a0;
      s_gv[1][tid] = a1;
      s_gv[2][tid] = a2;
    }
    __syncthreads();
    // particle -> cell in the tile
    const bool has = tid < nb;
    const int p = has ? perm[b0 + tid] : 0;
    Coord cx = {0.f, 0.f}, cy = {0.f, 0.f}, cz = {0.f, 0.f};
    int bx = 0, by = 0, bz = 0, c = -1;
    // all of the particle in one round trip, which the slot scan hides
    const uint32_t off = 4u * (uint32_t)p;
    float Fp[9], Fo[9], Co[9], vo[3], xo[3];
#pragma unroll
    for (int q = 0; q < 9; ++q) Fp[q] = Fo[q] = Co[q] = 0.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) vo[a] = xo[a] = 0.f;
    if (has) {
      if (Fob) {
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          Fo[q] = at_particle(Fob, q, n, off);
          Fp[q] = at_particle(F, q, n, off);
        }
      }
      if (Cob) {
#pragma unroll
        for (int q = 0; q < 9; ++q) Co[q] = at_particle(Cob, q, n, off);
      }
      if (vob) {
#pragma unroll
        for (int a = 0; a < 3; ++a) vo[a] = at_particle(vob, a, n, off);
      }
      if (xob) {
#pragma unroll
        for (int a = 0; a < 3; ++a) xo[a] = at_particle(xob, a, n, off);
      }
      cx = load_coord(xr, x, p, g.ox, g.inv_dx);
      cy = load_coord(xr, x, (size_t)n + p, g.oy, g.inv_dx);
      cz = load_coord(xr, x, 2 * (size_t)n + p, g.oz, g.inv_dx);
      bx = base_of(coord_sum(cx));
      by = base_of(coord_sum(cy));
      bz = base_of(coord_sum(cz));
      const int lx = bx - 4 * tx, ly = by - 4 * ty, lz = bz - 4 * tz;
      if ((unsigned)lx <= 3u && (unsigned)ly <= 3u && (unsigned)lz <= 3u) {
        c = lx + 4 * (ly + 4 * lz);
        atomicAdd(&s_cnt[c], 1);
      }
    }
    if (DET) s_cell[tid] = (unsigned char)(c >= 0 ? c : 255);
    __syncthreads();
    if (wid == 0) sc_scan_units(lane, s_cnt, s_off, s_cur, s_udesc, &s_nunits);
    __syncthreads();
    if (c >= 0) {
      int slot;
      if (DET) {
        // fixed order: rank among the item's earlier particles of the same cell
        int rank = 0;
        for (int q = 0; q < tid; ++q) rank += s_cell[q] == c;
        slot = s_off[c] + rank;
      } else {
        slot = atomicAdd(&s_cur[c], 1);
      }
      float f[3] = {coord_frac(cx, bx), coord_frac(cy, by), coord_frac(cz, bz)};
      float w[2][3], dw[2][3];
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        bspline_w(f[a], w[a]);
        bspline_dw(f[a], dw[a]);
      }
      // F' = (I + dt C) F:  Fbar += (I + dt C)^T Fbar',  Cbar += dt Fbar' F^T
      float Cbt[9], vbt[3];
      if (Fob) {
        float FoFt[9];
        Fp[0] += 1.f;  // stored as F - I
        Fp[4] += 1.f;
        Fp[8] += 1.f;
        matmul3_abt(Fo, Fp, FoFt);
#pragma unroll
        for (int q = 0; q < 9; ++q) Cbt[q] = Co[q] + dt * FoFt[q];
      } else {
#pragma unroll
        for (int q = 0; q < 9; ++q) Cbt[q] = Co[q];
      }
      // x' = x + dt v_p
#pragma unroll
      for (int a = 0; a < 3; ++a) vbt[a] = vo[a] + dt * xo[a];
      // scatter features: q = vbt - kc Cbt f, A = kc Cbt
      float A[9], qv[3];
#pragma unroll
      for (int q = 0; q < 9; ++q) A[q] = kc * Cbt[q];
#pragma unroll
      for (int a = 0; a < 3; ++a) qv[a] = vbt[a] - (A[3 * a] * f[0] + A[3 * a + 1] * f[1] + A[3 * a + 2] * f[2]);
      sc_stage<false>(s_dat, s_wgt, slot, f, 0.f, qv, A);
      // One gather of the stencil's grid velocities v_i gives both C_p = kc
      // sum w v (o - f)^T and the gradient of the gather through the weights
      // and the offsets, x_bar += gw s - (w / dx) A^T v with s = v . (vbt + A (o - f))
      // (d o / d x = -I / dx).  Per row the x-neighbours reduce to V = sum w v,
      // D = sum w (ox - fx) v, Sw = sum w s and Sd = sum dw s.
      float B[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      float X[3] = {0.f, 0.f, 0.f}, G[3] = {0.f, 0.f, 0.f};
#pragma unroll 1
      for (int oz = 0; oz < 3; ++oz) {
        const int lz = (bx - 4 * tx) + SC_L * ((by - 4 * ty) + SC_L * (bz - 4 * tz + oz));
        float wz, dwz;
        bspline_z(f[2], oz, wz, dwz);
        float qz[3], Gz[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int a = 0; a < 3; ++a) qz[a] = vbt[a] + A[3 * a + 2] * ((float)oz - f[2]);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy) {
          float Sw = 0.f, Sd = 0.f, V[3] = {0.f, 0.f, 0.f}, D[3] = {0.f, 0.f, 0.f};
#pragma unroll
          for (int ox = 0; ox < 3; ++ox) {
            float sd = 0.f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
              const float vi = s_gv[a][lz + SC_L * oy + ox];
              sd += vi * (qz[a] + A[3 * a + 1] * ((float)oy - f[1]) + A[3 * a] * ((float)ox - f[0]));
              const float t = w[0][ox] * vi;
              V[a] += t;
              D[a] += ((float)ox - f[0]) * t;
            }
            Sw += w[0][ox] * sd;
            Sd += dw[0][ox] * sd;
          }
          const float wyz = w[1][oy] * wz;
          X[0] += wyz * Sd;
          X[1] += dw[1][oy] * wz * Sw;
          X[2] += w[1][oy] * dwz * Sw;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const float t = wyz * V[a];
            Gz[a] += t;
            B[3 * a] += wyz * D[a];
            B[3 * a + 1] += ((float)oy - f[1]) * t;
          }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          G[a] += Gz[a];
          B[3 * a + 2] += ((float)oz - f[2]) * Gz[a];
        }
      }
      float Fbo[9], xbo[3];  // old values in one round trip (fresh: there are none)
#pragma unroll
      for (int q = 0; q < 9; ++q) Fbo[q] = 0.f;
#pragma unroll
      for (int a = 0; a < 3; ++a) xbo[a] = 0.f;
      if (Fob && Fb && !fresh) {
#pragma unroll
        for (int q = 0; q < 9; ++q) Fbo[q] = at_particle(Fb, q, n, off);
      }
      if (xb && !fresh) {
#pragma unroll
        for (int a = 0; a < 3; ++a) xbo[a] = at_particle(xb, a, n, off);
      }
      if (Fob && Fb) {
        float Gm[9], GtFo[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) Gm[q] = dt * (kc * B[q]) + ((q % 4) == 0 ? 1.f : 0.f);
        matmul3_atb(Gm, Fo, GtFo);
#pragma unroll
        for (int q = 0; q < 9; ++q) at_particle(Fb, q, n, off) = Fbo[q] + GtFo[q];
      }
      if (xb) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
          at_particle(xb, a, n, off) =
              xbo[a] + (xo[a] + g.inv_dx * (X[a] - (A[a] * G[0] + A[3 + a] * G[1] + A[6 + a] * G[2])));
      }
    }
    __syncthreads();
    int lane_now = lane;
    asm("" : "+v"(lane_now));  // likewise the 30 constants of sc_lane
    const ScLane L = sc_lane<false>(lane_now);
    sc_units_mfma(L, wid, s_dat, s_wgt, s_udesc, s_nunits, s_node[wid]);
    __syncthreads();
    int node_now = tid;
    asm("" : "+v"(node_now));  // likewise
    if (node_now < SC_NODES) {
      const int tid = node_now;
      float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int w = 0; w < SC_WAVES; ++w) {
        s0 += s_node[w][tid][1];
        s1 += s_node[w][tid][2];
        s2 += s_node[w][tid][3];
      }
      if (DET) {
        float *dst = item_part + ((int64_t)it * SC_NODES + tid) * 4;
        dst[0] = 0.f;
        dst[1] = s0;
        dst[2] = s1;
        dst[3] = s2;
      } else if (s0 != 0.f || s1 != 0.f || s2 != 0.f) {
        const int ix = tid % SC_L, iy = (tid / SC_L) % SC_L, iz = tid / (SC_L * SC_L);
        const int64_t node = (4 * tx + ix) + (int64_t)g.nx * ((4 * ty + iy) + (int64_t)g.ny * (4 * tz + iz));
        atomicAdd(&gvb[node], s0);
        atomicAdd(&gvb[N + node], s1);
        atomicAdd(&gvb[2 * N + node], s2);
      }
    }
    __syncthreads();
  }
}

}  // namespace dw

using namespace dw;

int dw::run_p2g_adj(const dw_grid *grid, const dw_mpm_params *params, const dw_particles *p, const float *grid_m_bar,
                    const float *grid_mv_bar, dw_particles_bar *bar, float *E_bar, void *ws, size_t ws_bytes,
                    void *stream, int fresh, float *e_slots) {
  int rc = check_grid(grid);
  if (rc) return rc;
  DW_REQUIRE(params, DW_EINVAL, "mpm_p2g_adj: params is NULL");
  DW_REQUIRE(params->material == DW_FIXED_COROTATED || params->material == DW_NEO_HOOKEAN, DW_EINVAL,
             "mpm_p2g_adj: unknown material");
  rc = check_particles(p, true);
  if (rc) return rc;
  DW_REQUIRE(grid_m_bar && grid_mv_bar, DW_EINVAL, "mpm_p2g_adj: grid adjoints must be set");
  DW_REQUIRE(bar && bar->n == p->n, DW_EINVAL, "mpm_p2g_adj: bar->n must equal p->n");
  if (p->n == 0) return DW_OK;
  PAdj P;
  P.x = p->x; P.v = p->v; P.C = p->C; P.F = p->F; P.mass = p->mass; P.vol0 = p->vol0;
  P.E = p->E; P.nu = p->nu; P.region = p->region; P.n = p->n; P.xr = p->xref;
  P.xb = bar->x; P.vb = bar->v; P.Cb = bar->C; P.Fb = bar->F; P.Eb = E_bar;
  P.n_regions = p->n_regions;
  P.Epart = nullptr;
  P.fresh = fresh;
  P.slots = 0;
  GridDev g = make_grid(grid);
  int64_t N = (int64_t)grid->nx * grid->ny * grid->nz;
  hipStream_t s = (hipStream_t)stream;
  if (params->deterministic && E_bar) {
    const unsigned blocks = grid_blocks(p->n, 256);
    Workspace W;
    rc = bind_workspace(grid, p->n, ws, ws_bytes, &W, 1);
    if (rc) return rc;
    const int64_t waves = (int64_t)blocks * 4;
    DW_REQUIRE(waves * p->n_regions <= W.item_part_floats, DW_EWORKSPACE,
               "mpm_p2g_adj: %d regions need more deterministic scratch than the workspace holds", p->n_regions);
    P.Epart = W.item_part;
    hipLaunchKernelGGL(k_p2g_adj<true>, dim3(blocks), dim3(256), 18 * 256 * sizeof(float), s, g, P, params->dt,
                       params->material, grid_m_bar, grid_mv_bar, N);
    hipLaunchKernelGGL(k_ebar_reduce, dim3(grid_blocks(p->n_regions, 64)), dim3(64), 0, s, W.item_part,
                       ((int64_t)p->n + 63) / 64, p->n_regions, E_bar);
  } else {
    const int threads = p2g_adj_threads(p->n);
    if (e_slots) {
      P.Eb = e_slots;
      P.slots = 1;
    }
    hipLaunchKernelGGL(k_p2g_adj<false>, dim3(p2g_adj_blocks(p->n)), dim3(threads), 18 * threads * sizeof(float), s, g, P,
                       params->dt, params->material, grid_m_bar, grid_mv_bar, N);
  }
  return check_launch("mpm_p2g_adj");
}

int64_t dw::e_slot_floats(const dw_particles *p) { return (int64_t)p2g_adj_blocks(p->n) * p->n_regions; }

int dw::run_e_slots(const dw_particles *p, const float *e_slots, float *E_bar, void *stream) {
  hipLaunchKernelGGL(k_e_slots, dim3(p->n_regions), dim3(64), 0, (hipStream_t)stream, e_slots,
                     (int)p2g_adj_blocks(p->n), p->n_regions, E_bar);
  return check_launch("mpm_p2g_adj");
}

extern "C" int mpm_p2g_adj(const dw_grid *grid, const dw_mpm_params *params, const dw_particles *p,
                           const float *grid_m_bar, const float *grid_mv_bar, dw_particles_bar *bar, float *E_bar,
                           void *ws, size_t ws_bytes, void *stream) {
  return dw::run_p2g_adj(grid, params, p, grid_m_bar, grid_mv_bar, bar, E_bar, ws, ws_bytes, stream, 0, nullptr);
}

// W_bar given: the fused form (grid_v_bar is then cleared on the active tiles)
static int grid_update_adj(const dw_grid *grid, const dw_mpm_params *params, const float *grid_m, const float *grid_mv,
                           const dw_wind *wind, const uint8_t *pin, float *grid_v_bar, float *grid_m_bar,
                           float *grid_mv_bar, float *acc_bar, float *W_bar, const void *ws, size_t ws_bytes,
                           void *stream) {
  int rc = check_grid(grid);
  if (rc) return rc;
  DW_REQUIRE(params && grid_m && grid_mv && grid_v_bar, DW_EINVAL, "mpm_grid_update_adj: missing argument");
  Workspace W;
  rc = bind_workspace(grid, 0, ws, ws_bytes, &W);
  if (rc) return rc;
  WindDev wd;
  rc = make_wind(wind, grid, &wd);
  if (rc) return rc;
  GridDev g = make_grid(grid);
  int64_t N = (int64_t)grid->nx * grid->ny * grid->nz;
  auto k = W_bar ? k_grid_update_adj<true> : k_grid_update_adj<false>;
  hipLaunchKernelGGL(k, dim3(node_blocks(W.n_tiles)), dim3(256), 0, (hipStream_t)stream, g, params->dt,
                     params->gravity[0], params->gravity[1], params->gravity[2], params->bound, grid_m, grid_mv, wd,
                     pin, W.node_tiles, W.n_node_tiles, grid_v_bar, grid_m_bar, grid_mv_bar, acc_bar, W_bar, N);
  return check_launch("mpm_grid_update_adj");
}

extern "C" int mpm_grid_update_adj(const dw_grid *grid, const dw_mpm_params *params, const float *grid_m,
                                   const float *grid_mv, const dw_wind *wind, const uint8_t *pin,
                                   const float *grid_v_bar, float *grid_m_bar, float *grid_mv_bar, float *acc_bar,
                                   const void *ws, size_t ws_bytes, void *stream) {
  return grid_update_adj(grid, params, grid_m, grid_mv, wind, pin, const_cast<float *>(grid_v_bar), grid_m_bar,
                         grid_mv_bar, acc_bar, nullptr, ws, ws_bytes, stream);
}

int dw::run_grid_update_adj_fused(const dw_grid *grid, const dw_mpm_params *params, const float *grid_m,
                                  const float *grid_mv, const dw_wind *wind, const uint8_t *pin, float *grid_v_bar,
                                  float *grid_m_bar, float *grid_mv_bar, float *W_bar, const void *ws,
                                  size_t ws_bytes, void *stream) {
  return grid_update_adj(grid, params, grid_m, grid_mv, wind, pin, grid_v_bar, grid_m_bar, grid_mv_bar, nullptr,
                         W_bar, ws, ws_bytes, stream);
}

int dw::run_g2p_adj(const dw_grid *grid, const dw_mpm_params *params, const float *grid_v, const dw_particles *in,
                    const dw_particles_bar *out_bar, dw_particles_bar *in_bar, float *grid_v_bar, const void *ws,
                    size_t ws_bytes, void *stream, int fresh) {
  int rc = check_grid(grid);
  if (rc) return rc;
  DW_REQUIRE(params && grid_v && in && out_bar && in_bar && grid_v_bar, DW_EINVAL,
             "mpm_g2p_adj: missing argument");
  DW_REQUIRE(in->n >= 0 && out_bar->n == in->n && in_bar->n == in->n, DW_EINVAL, "mpm_g2p_adj: size mismatch");
  if (in->n == 0) return DW_OK;
  DW_REQUIRE(in->x && in->F, DW_EINVAL, "mpm_g2p_adj: in->x / in->F is NULL");
  Workspace W;
  const int det = params->deterministic ? 1 : 0;
  rc = bind_workspace(grid, in->n, ws, ws_bytes, &W, det);
  if (rc) return rc;
  GridDev g = make_grid(grid);
  int64_t N = (int64_t)grid->nx * grid->ny * grid->nz;
  hipStream_t s = (hipStream_t)stream;
  // at most this many work items: a partial chunk per tile and the whole chunks
  const unsigned blocks = (unsigned)std::min<int64_t>(2048, W.n_tiles + in->n / WORK_CHUNK);
  if (det) {
    hipLaunchKernelGGL(k_g2p_adj<true>, dim3(blocks), dim3(SC_THREADS), 0, s, g, params->dt, grid_v, N, in->x,
                       in->xref, in->F, in->n, out_bar->x, out_bar->v, out_bar->C, out_bar->F, in_bar->x, in_bar->F,
                       grid_v_bar, W.perm, W.tile_start, W.item_tile, W.item_begin, W.n_items, W.item_part, fresh);
    hipLaunchKernelGGL(k_det_gather<true>, dim3(node_blocks(W.n_tiles)), dim3(256), 0, s, g, W.node_tiles, W.n_node_tiles,
                       W.tile_count, W.item_first, W.item_part, (float *)nullptr, grid_v_bar, N, (int32_t *)nullptr);
  } else {
    hipLaunchKernelGGL(k_g2p_adj<false>, dim3(blocks), dim3(SC_THREADS), 0, s, g, params->dt, grid_v, N, in->x,
                       in->xref, in->F, in->n, out_bar->x, out_bar->v, out_bar->C, out_bar->F, in_bar->x, in_bar->F,
                       grid_v_bar, W.perm, W.tile_start, W.item_tile, W.item_begin, W.n_items, (float *)nullptr, fresh);
  }
  return check_launch("mpm_g2p_adj");
}

extern "C" int mpm_g2p_adj(const dw_grid *grid, const dw_mpm_params *params, const float *grid_v,
                           const dw_particles *in, const dw_particles_bar *out_bar, dw_particles_bar *in_bar,
                           float *grid_v_bar, const void *ws, size_t ws_bytes, void *stream) {
  return dw::run_g2p_adj(grid, params, grid_v, in, out_bar, in_bar, grid_v_bar, ws, ws_bytes, stream, 0);
}
