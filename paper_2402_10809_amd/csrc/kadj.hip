// lbm_adjoint: the reverse kernel and its checkpointing driver.
#include <algorithm>
#include <vector>

#include "adjoint.hpp"
#include "runtime.hpp"

using namespace lbmrt;

// Host side of lbm_adjoint: forward pass with checkpoints, then segment-wise
// recompute (recording pulled values, omega_prev and density) and reverse
// steps.  The checkpoint of segment s (s >= 1) is the record of the step before
// the segment's first, made by the forward pass; the recompute starts with that
// step from the record, which also gives the density of the step before the
// segment, which the porosity-jump gather of the segment's first reverse step
// needs.  A record is independent of the slot layout; the slots of a restarted
// state follow the parity of its time.  The forward pass records the last segment
// itself (that segment needs no checkpoint and no recompute); with one segment
// (ckpt_every >= T) nothing is recomputed.  The recompute reproduces the forward
// trajectory bit for bit, so the records are the same either way.  That the forms of
// the step the two take (with an objective or not, through the wave records or the
// link words, alone or joint, 64 or 256 work-items) round alike is the compiler's
// doing; the tests compare segment lengths on lattices that reach all of them.
extern "C" lbm_status lbm_adjoint(lbm_ctx* c, const lbm_objective* obj, int T, int ckpt, double* J,
                                  float* dJ_dphi) {
  CTX_CHECK(c);
  if (!obj || !J) return fail(LBM_E_INVALID, "obj and J must not be NULL");
  if (T < 1 || ckpt < 1) return fail(LBM_E_INVALID, "T and ckpt_every must be >= 1");
  if (obj->t_begin < 0 || obj->t_end > T || obj->t_begin >= obj->t_end)
    return fail(LBM_E_INVALID, "objective window must satisfy 0 <= t_begin < t_end <= T");
  if (c->grid.storage != LBM_STORE_FP32 || c->grid.shift_mode != 0)
    return fail(LBM_E_INVALID, "the adjoint supports FP32 storage with shift mode 0");
  if (c->q != 19) return fail(LBM_E_INVALID, "the adjoint is built for D3Q19");
  if (obj->fp64_adjoint && (uint64_t)Q * (uint64_t)c->nc * 8u >= (1ull << 31))
    return fail(LBM_E_INVALID, "FP64 adjoint populations need 19 * 8 bytes per cell below 2 GiB");
  if (obj->kind != LBM_OBJ_KINETIC && obj->kind != LBM_OBJ_WSS) return fail(LBM_E_INVALID, "unknown objective kind");
  if (c->nreg == 0) return fail(LBM_E_INVALID, "the objective region has no fluid cell");
  if (obj->kind == LBM_OBJ_WSS && c->nwss == 0) return fail(LBM_E_INVALID, "the objective region has no wall cell");
  const int okind = obj->kind;
  const int64_t ncount = okind == LBM_OBJ_WSS ? c->nwss : c->nreg;
  // without a gradient output only J is computed: forward pass, no checkpoints
  const bool want_grad = dJ_dphi != nullptr;
  const Layout L = make_layout(c->grid, c->nc, c->nrow, want_grad ? T : 0, want_grad ? ckpt : 0);
  if (c->ws_bytes < L.total)
    return fail(LBM_E_WORKSPACE, "workspace too small for this adjoint: need " + std::to_string(L.total) + " bytes");
  // The forward passes compute the collision in FP64: the reverse steps
  // differentiate along the recorded trajectory, and FP32 rounding of the
  // per-cell scalars moves it by a few 1e-6 of J over thousands of steps.
  struct ArithScope {
    lbm_ctx* c;
    int saved;
    ~ArithScope() { c->amode = saved; }
  } arith_scope{c, c->amode};
  c->amode = 2;
  const size_t nc = (size_t)c->nc, pl = (size_t)plane_cells(c->nc), nbox = c->nbox;
  float* ck = (float*)(c->ws + L.ck);
  float* rec = (float*)(c->ws + L.rec);
  float* rho = (float*)(c->ws + L.rho);
  double* omh = (double*)(c->ws + L.omh);
  double* phih = (double*)(c->ws + L.phih);
  double* objp = (double*)(c->ws + L.obj);
  const int nseg = (int)(((int64_t)T + ckpt - 1) / ckpt), s_last = nseg - 1, t0_last = s_last * ckpt;
  // On grids that leave the chip idle a reverse or a recompute step is bound by
  // the latency of its waves, so one launch takes a step of each: while segment s
  // is reversed, segment s - 1 is recomputed. On larger grids both are bound by
  // memory and take turns (the line between them: TOGETHER_CELLS).
  const bool together = nseg > 1 && c->nc <= TOGETHER_CELLS;
  // The record: slots of one step each, given out and taken back one by one, so
  // that a segment's record grows into the slots that reversing the one after it
  // has freed (ckpt + 1 slots serve both). held[s & 1][j] is the slot of step j of
  // segment s; the density of the step before a segment has a place of its own.
  std::vector<int> free_slots, held[2];
  if (want_grad) {
    const int steps = std::min(ckpt, T);  // of a segment
    for (int k = steps; k >= 0; --k) free_slots.push_back(k);
    held[0].assign(steps, 0);
    held[1].assign(steps, 0);
  }
  auto take_slot = [&](int s, int j) {
    held[s & 1][j] = free_slots.back();
    free_slots.pop_back();
  };
  auto give_slot = [&](int s, int j) { free_slots.push_back(held[s & 1][j]); };
  auto step_rec = [&](int s, int j) { return rec + (size_t)held[s & 1][j] * (Q + 1) * pl; };
  auto step_rho = [&](int s, int j) { return rho + (size_t)(j < 0 ? ckpt + 1 + (s & 1) : held[s & 1][j]) * pl; };
  auto slot_ck = [&](int s) { return ck + (size_t)s * (Q + 1) * pl; };

  // forward pass: objective and checkpoints
  lbm_status st = launch_init(c);
  if (st != LBM_OK) return st;
  const int nwave = blocks_for_nt(c->nc, 64);
  HIP_TRY(c, hipMemsetAsync(objp, 0, (size_t)nwave * 8, c->stream));
  for (int t = 0; t < T; ++t) {
    const bool in = t >= obj->t_begin && t < obj->t_end;
    float* r = nullptr;
    float* rr = nullptr;
    if (want_grad && t >= t0_last) {
      take_slot(s_last, t - t0_last);
      r = step_rec(s_last, t - t0_last);
      rr = step_rho(s_last, t - t0_last);
    } else if (want_grad && (t + 1) % ckpt == 0) {
      // the checkpoint of the segment that starts at t + 1; its density is the
      // last segment's, or is recorded again from the checkpoint
      r = slot_ck((t + 1) / ckpt);
      rr = step_rho(s_last, -1);
    }
    st = launch_step(c, in ? (okind == LBM_OBJ_WSS ? 3 : 2) : 0, r, rr);
    if (st != LBM_OK) return st;
  }
  double jsum = 0.0;
  st = finalize(c, objp, nwave, 1, 0u, &jsum);
  if (st != LBM_OK) return st;
  const double ew = 1.0 / ((double)(obj->t_end - obj->t_begin) * (double)ncount);
  *J = jsum * ew;
  if (!want_grad) {
    st = launch_init(c);
    if (st != LBM_OK) return st;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return LBM_OK;
  }

  // reverse sweep
  // adjoint of the pulled populations, in place, FP32 or FP64 (the
  // workspace holds room for FP64)
  const bool p64 = obj->fp64_adjoint != 0;
  const size_t pb = p64 ? 8 : 4;
  void* ph = (void*)(c->ws + L.ah);
  HIP_TRY(c, hipMemsetAsync(ph, 0, Q * pl * pb, c->stream));
  HIP_TRY(c, hipMemsetAsync(omh, 0, nc * 8, c->stream));
  HIP_TRY(c, hipMemsetAsync(phih, 0, nc * 8, c->stream));
  // extrapolation outflow: adjoints of the kept unknowns, per row, by parity
  // of the step (none after the last step)
  double* aside = (double*)(c->ws + L.aside);
  HIP_TRY(c, hipMemsetAsync(aside, 0, (size_t)2 * c->nrow * 5 * 8, c->stream));
  AdjBufs ab{};
  ab.code = (const uint32_t*)(c->ws + c->L.code);
  ab.links = (const uint32_t*)(c->ws + c->L.links);
  ab.delta = (const int*)(c->ws + c->L.delta);
  ab.phi = (const float*)(c->ws + c->L.phi);
  ab.shape = (const float*)(c->ws + c->L.shape);
  ab.wave = (const double*)(c->ws + c->L.wave);
  ab.omh = omh;
  ab.phih = phih;
  ab.ph = ph;
  ab.pl = (uint32_t)pl;
  // the start of the recompute of segment s: the rest state, or the step before
  // the segment from its checkpoint
  auto restart = [&](int s) -> lbm_status {
    if (s == 0) return launch_init(c);
    c->t = (int64_t)s * ckpt - 1;
    return launch_step(c, 0, slot_ck(s), step_rho(s, -1), true);
  };
  // single-wave workgroups on small grids, as the forward steps (whole call: 37 736
  // cells 2 348 -> 2 316 us, 118 304 5 090 -> 4 965 us, with the anisotropic medium and FP64
  // populations 6 820 -> 6 528 us)
  const bool narrow = step_width(c, BLOCK) == 64;
  // the reverse step of step j of segment s; with `next` also the recording of the
  // next step of segment s - 1 (at time c->t)
  auto reverse_step = [&](int s, int j, bool next) -> lbm_status {
    const int n = s * ckpt + j;
    ab.rec = step_rec(s, j);
    ab.rho_prev = step_rho(s, j - 1);
    ab.aside_in = aside + (size_t)((n + 1) & 1) * c->nrow * 5;
    ab.aside_out = aside + (size_t)(n & 1) * c->nrow * 5;
    const float ewn = (n >= obj->t_begin && n < obj->t_end) ? (float)ew : 0.0f;
    Bufs b = bufs(c);
    if (next) {
      const int i = (int)(c->t - (int64_t)(s - 1) * ckpt);
      take_slot(s - 1, i);
      b.rec = step_rec(s - 1, i);
      b.rho_rec = step_rho(s - 1, i);
    }
    auto reverse = [&](auto an, auto ph_type, auto odd) {
      using PH = decltype(ph_type);
      constexpr bool AN = decltype(an)::value, OD = decltype(odd)::value;
      const unsigned nw = (unsigned)blocks_for_nt(c->nc, 64);
      if (next)
        with_parity(c->t, [&](auto sodd) {
          constexpr bool SO = decltype(sodd)::value;
          if (narrow)
            hipLaunchKernelGGL((k_adjoint_and_step<AN, PH, OD, SO, 64>), dim3(2 * nw), dim3(64), 0, c->stream, c->P, ab,
                               (uint32_t)n, ewn, okind, nw, b);
          else
            hipLaunchKernelGGL((k_adjoint_and_step<AN, PH, OD, SO, BLOCK>), dim3(2 * c->nblk), dim3(BLOCK), 0, c->stream,
                               c->P, ab, (uint32_t)n, ewn, okind, (uint32_t)c->nblk, b);
        });
      else if (narrow)
        hipLaunchKernelGGL((k_adjoint<AN, PH, OD, 64>), dim3(nw), dim3(64), 0, c->stream, c->P, ab, (uint32_t)n, ewn,
                           okind);
      else
        hipLaunchKernelGGL((k_adjoint<AN, PH, OD, BLOCK>), dim3(c->nblk), dim3(BLOCK), 0, c->stream, c->P, ab,
                           (uint32_t)n, ewn, okind);
    };
    with_parity(n, [&](auto odd) {
      if (c->P.an_iters > 0 && p64) reverse(std::true_type{}, double{}, odd);
      else if (c->P.an_iters > 0) reverse(std::true_type{}, float{}, odd);
      else if (p64) reverse(std::false_type{}, double{}, odd);
      else reverse(std::false_type{}, float{}, odd);
    });
    HIP_TRY(c, hipGetLastError());
    if (next) c->t += 1;
    give_slot(s, j);
    return LBM_OK;
  };
  for (int s = s_last; s >= 0; --s) {
    const int nv = std::min(T - s * ckpt, ckpt);
    if (together && s > 0) {
      st = restart(s - 1);
      if (st != LBM_OK) return st;
    }
    for (int i = 0; i < nv; ++i) {
      st = reverse_step(s, nv - 1 - i, together && s > 0);
      if (st != LBM_OK) return st;
    }
    if (s == 0) break;
    if (!together) {
      st = restart(s - 1);
      if (st != LBM_OK) return st;
    }
    // the rest of segment s - 1 (all of it where the two take turns)
    for (int j = (int)(c->t - (int64_t)(s - 1) * ckpt); j < ckpt; ++j) {
      take_slot(s - 1, j);
      st = launch_step(c, 0, step_rec(s - 1, j), step_rho(s - 1, j));
      if (st != LBM_OK) return st;
    }
  }
  HIP_TRY(c, hipMemsetAsync(dJ_dphi, 0, nbox * 4, c->stream));
  if (p64)
    hipLaunchKernelGGL(k_adj_final<double>, dim3(c->nblk), dim3(BLOCK), 0, c->stream, c->P, ab.code, ab.links,
                       (const uint32_t*)(c->ws + c->L.rowbox), (const double*)ph, (uint32_t)pl, (const double*)phih,
                       (const double*)aside, dJ_dphi);
  else
    hipLaunchKernelGGL(k_adj_final<float>, dim3(c->nblk), dim3(BLOCK), 0, c->stream, c->P, ab.code, ab.links,
                       (const uint32_t*)(c->ws + c->L.rowbox), (const float*)ph, (uint32_t)pl, (const double*)phih,
                       (const double*)aside, dJ_dphi);
  HIP_TRY(c, hipGetLastError());
  // leave the context at the rest state
  st = launch_init(c);
  if (st != LBM_OK) return st;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return LBM_OK;
}
