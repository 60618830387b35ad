// Substep loops of a differentiable rollout under a force-grid wind (one field
// per time slot): the forward of a run of substeps, and the reverse of a
// segment whose states, sorts and grids are kept.  A substep of a small scene
// is a dozen kernels of a few microseconds, so the launches themselves bound
// it; driving them from here instead of one binding call per entry point, and
// with fewer kernels, took 20k particles, 16 substeps with their gradient,
// from 3,500 to 2,130 us (256k particles: 4,640 to 3,860), and a last segment
// that the forward keeps for the reverse (seg->states with out) from 2,065 to
// 1,840 (3,730 to 3,330).
#include <hip/hip_runtime.h>

#include "dw_internal.h"

namespace dw {

// particle state arrays of n particles packed as x, v, C, F
template <typename T>
static void bind_state(T *p, float *base) {
  const size_t n = (size_t)p->n;
  p->x = base;
  p->v = base + 3 * n;
  p->C = base + 6 * n;
  p->F = base + 15 * n;
}

static int check_segment(const char *who, const dw_grid *grid, const dw_mpm_params *params, const dw_particles *p,
                         const dw_wind *wind, const dw_segment *seg) {
  int rc = check_grid(grid);
  if (rc) return rc;
  DW_REQUIRE(params && seg, DW_EINVAL, "%s: missing argument", who);
  rc = check_particles(p, true);
  if (rc) return rc;
  DW_REQUIRE(wind && wind->mode == DW_WIND_FORCE_GRID && wind->W, DW_EINVAL, "%s: needs a force-grid wind", who);
  DW_REQUIRE(seg->count >= 0 && seg->first >= 0 && seg->n_sub > 0 && seg->first + seg->count <= seg->n_sub &&
                 seg->slots > 0,
             DW_EINVAL, "%s: substeps out of range", who);
  DW_REQUIRE(seg->grids && seg->ws && seg->grid_stride >= 0 && seg->ws_stride >= 0 && seg->ws_stride % 256 == 0,
             DW_EINVAL, "%s: grids / ws missing or misaligned", who);
  return DW_OK;
}

static int64_t slot_of(const dw_segment *seg, int s) { return (int64_t)s * seg->slots / seg->n_sub; }

static dw_wind slot_wind(const dw_wind *wind, const dw_segment *seg, int s) {
  dw_wind w = *wind;
  w.W += slot_of(seg, s) * seg->slot_stride;
  return w;
}

}  // namespace dw

using namespace dw;

extern "C" int mpm_rollout(const dw_grid *grid, const dw_mpm_params *params, const dw_particles *p,
                           const dw_particles_bar *out, const dw_wind *wind, const uint8_t *pin,
                           const dw_segment *seg, int32_t *status_or, void *stream) {
  int rc = check_segment("mpm_rollout", grid, params, p, wind, seg);
  if (rc) return rc;
  DW_REQUIRE(seg->states || out, DW_EINVAL, "mpm_rollout: out is NULL");
  DW_REQUIRE(!out || (out->n == p->n && (p->n == 0 || (out->x && out->v && out->C && out->F))), DW_EINVAL,
             "mpm_rollout: out must hold the particles");
  const int64_t N = (int64_t)grid->nx * grid->ny * grid->nz;
  dw_particles in = *p;
  for (int i = 0; i < seg->count; ++i) {
    float *gm = seg->grids + i * seg->grid_stride, *gmv = gm + N, *gv = gmv + 3 * N;
    char *ws = (char *)seg->ws + i * seg->ws_stride;
    const dw_wind w = slot_wind(wind, seg, seg->first + i);
    if ((rc = mpm_sort(grid, params, in.x, in.xref, in.n, ws, seg->ws_bytes, stream))) return rc;
    if ((rc = mpm_p2g(grid, params, &in, gm, gmv, ws, seg->ws_bytes, stream))) return rc;
    if ((rc = run_grid_update(grid, params, gm, gmv, &w, pin, gv, ws, seg->ws_bytes, stream, status_or))) return rc;
    const bool last = i == seg->count - 1;
    if (seg->states && last && !out) break;  // the segment ends with its grid
    dw_particles to = in;
    if (seg->states && !last) {
      bind_state(&to, seg->states + (size_t)i * 24 * in.n);
    } else {
      to.x = out->x;
      to.v = out->v;
      to.C = out->C;
      to.F = out->F;
    }
    if ((rc = mpm_g2p(grid, params, gv, &in, &to, stream))) return rc;
    in = to;
  }
  return DW_OK;
}

extern "C" int mpm_rollout_adj(const dw_grid *grid, const dw_mpm_params *params, const dw_particles *p,
                               const dw_wind *wind, const uint8_t *pin, const dw_segment *seg, float *bars, int cur,
                               float *grid_bar, float *W_bar, float *E_bar, void *stream) {
  int rc = check_segment("mpm_rollout_adj", grid, params, p, wind, seg);
  if (rc) return rc;
  DW_REQUIRE(bars && grid_bar && W_bar && E_bar && (cur == 0 || cur == 1), DW_EINVAL,
             "mpm_rollout_adj: missing argument");
  DW_REQUIRE(seg->states || seg->count <= 1, DW_EINVAL, "mpm_rollout_adj: needs the segment's states");
  const int64_t N = (int64_t)grid->nx * grid->ny * grid->nz;
  float *gvb = grid_bar, *gmb = gvb + 3 * N, *gmvb = gmb + N, *accb = gmvb + 3 * N;
  const size_t state = (size_t)24 * p->n;
  hipStream_t s = (hipStream_t)stream;
  // the deterministic transpose gathers over all nodes, so it needs accb and a
  // clear of all ten arrays per substep
  const bool fused = !wind->deterministic;
  // accb is free in the fused form: the workgroups' rows of the E adjoint,
  // added up once per segment
  const int64_t n_slots = p->n > 0 ? e_slot_floats(p) : 0;
  float *e_slots = fused && !params->deterministic && n_slots > 0 && n_slots <= 3 * N ? accb : nullptr;
  if (e_slots && seg->count > 0)
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_blocks(n_slots / 4 + 4, 256)), dim3(256), 0, s, (int32_t *)e_slots,
                       n_slots, 0);
  for (int i = seg->count - 1; i >= 0; --i, cur ^= 1) {
    const float *gm = seg->grids + i * seg->grid_stride, *gmv = gm + N, *gv = gmv + 3 * N;
    char *ws = (char *)seg->ws + i * seg->ws_stride;
    const dw_wind w = slot_wind(wind, seg, seg->first + i);
    float *Wb = W_bar + slot_of(seg, seg->first + i) * seg->slot_stride;
    dw_particles in = *p;
    if (i > 0) bind_state(&in, seg->states + (size_t)(i - 1) * state);
    dw_particles_bar to = {in.n}, from = {in.n};
    bind_state(&from, bars + cur * state);
    bind_state(&to, bars + (cur ^ 1) * state);
    if (!fused)
      hipLaunchKernelGGL(k_fill_i32, dim3(grid_blocks(10 * N / 4 + 4, 256)), dim3(256), 0, s, (int32_t *)grid_bar,
                         10 * N, 0);
    if ((rc = run_g2p_adj(grid, params, gv, &in, &from, &to, gvb, ws, seg->ws_bytes, stream, 1))) return rc;
    if (fused) {
      if ((rc = run_grid_update_adj_fused(grid, params, gm, gmv, &w, pin, gvb, gmb, gmvb, Wb, ws, seg->ws_bytes,
                                          stream)))
        return rc;
    } else {
      if ((rc = mpm_grid_update_adj(grid, params, gm, gmv, &w, pin, gvb, gmb, gmvb, accb, ws, seg->ws_bytes, stream)))
        return rc;
      if ((rc = wind_to_grid_adj(grid, &w, accb, Wb, stream))) return rc;
    }
    if ((rc = run_p2g_adj(grid, params, &in, gmb, gmvb, &to, E_bar, ws, seg->ws_bytes, stream, 1, e_slots)))
      return rc;
  }
  if (e_slots && seg->count > 0) return run_e_slots(p, e_slots, E_bar, stream);
  return DW_OK;
}
