// Reverse-time (adjoint) step of the VANSE Carreau-Yasuda collide-and-stream
// map, for the gradient of a region kinetic-energy objective with respect to
// the porosity field.
//
// The per-cell forward map of step n is
//   (pulled f_i, omega_prev, phi(x), phi~(x + c_i)) -> (q_i, omega, e)
// with the open-face fill, moments, explicit velocity with Darcy drag, force,
// equilibrium, corrected second moment Pi, semi-explicit shear rate,
// Carreau-Yasuda viscosity, relaxation rate and the BGK + Guo + porosity-jump
// collision (the paper's method section).  Its transpose is written out by hand
// below in terms of the weighted output adjoint a_i = w_i qhat_i and its
// moments s0 = sum a_i, s1 = sum a_i c_i, s2 = sum a_i c_i c_i, so the sweep
// stays in registers.  The streaming transpose takes qhat_i(x) from the
// consumer's pulled-value adjoint at x + c_i (or the cell's own opposite one
// across a wall).  One buffer holds them in place, in the forward step's AA
// pattern run backwards.  With a_i the adjoint of step n+1's pulled f_i:
//   n odd:  a_i(x) sits at slot (i, x).  The reverse step of n reads qhat_i(x)
//           from slot (i, x + c_i) ((opp i, x) across a wall) and writes its own
//           adjoint a_i(x) to slot (opp i, x - c_i) ((i, x) across a wall);
//   n even: qhat_i(x) is therefore at slot (opp i, x), and the reverse step
//           writes a_i(x) to slot (i, x).
// Within one reverse step every slot is read and written by one work-item, so
// no two race, and after step 0 the adjoints sit at (i, x).  One buffer of 19
// planes (179 MB on 2.36 M cells) instead of two stays in the Infinity Cache
// from one reverse step to the next while the record streams past it.  The porosity-jump term couples q_i(x) to phi(x + c_i); that
// contribution is gathered by the consumer cell from the producer's recorded
// density of the previous step, so no atomics are needed.
//
// With the extrapolation outflow, an outflow cell's unknowns (c_x = -1) are
// state: step n computes them as (1 - c_s) times the cell's own value of step
// n-1 plus c_s times the -x neighbour's pulled value of step n-1.  The reverse
// step of n leaves the unknowns' total adjoints per row (aside_out); the reverse
// step of n-1 adds (1 - c_s) of them to the outflow cell's unknowns and c_s of
// them to the -x neighbour's pulled values.
//
// AN: the anisotropic permeability of the method section's Remark, whose
// fixed-point iterates the reverse step goes back through.
//
// Supported: FP32 storage, shift mode 0, with or without Forchheimer drag,
// isotropic or anisotropic permeability, D3Q19.  The recompute uses the same
// arithmetic type as the forward step.
#pragma once
#include "step.hpp"

namespace lbm {

struct AdjBufs {
  const uint32_t* code;   // (row << xbits) | x per compact cell
  const uint32_t* links;  // link word per compact cell
  const int* delta;       // neighbour-row deltas
  const float* phi;       // porosity per compact cell
  const float* shape;     // inflow profile per row
  const double* wave;     // sampled inflow waveform
  const float* rec;       // record of step n: [19][pl] pulled values (after the fill), [pl] omega_prev
  const float* rho_prev;  // density of step n-1 per compact cell (read but not used at n = 0)
  void* ph;               // adjoint of the pulled populations, [19][pl] (FP32 or FP64), in place
  uint32_t pl;            // cells per plane of rec and ph (plane_cells)
  double* omh;            // per cell: in adjoint of omega_n, out adjoint of omega_{n-1}
  double* phih;           // per cell: porosity adjoint accumulator
  const double* aside_in; // extrapolation outflow: per row, adjoints of the 5 c_x = -1 unknowns of step n+1
  double* aside_out;      // the same for step n
};

// One FP32 value per lane from a buffer straight into LDS (the wave's 64
// consecutive slots at lds): the load occupies no register while in flight.
__device__ __forceinline__ void gather_to_lds(__amdgpu_buffer_rsrc_t r, float* lds, uint32_t voff, uint32_t soff = 0) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 4, voff, soff, 0, 0);
}
// One adjoint population to the buffer (FP32 or FP64).
template <class PH>
__device__ __forceinline__ void put_adjoint(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, double v) {
  if constexpr (std::is_same<PH, double>::value) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, voff, soff, 0);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)v), r, voff, soff, 0);
  }
}

// The kernel's first argument (Params) read again from the kernel arguments:
// the constants of a later phase are loaded there instead of being held in
// scalar registers (and spilled to vector lanes) from the start.
typedef const __attribute__((address_space(4))) Params CParams;
__device__ __forceinline__ const CParams& params_again() {
  uint64_t a = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return *(const CParams*)a;
}

// One reverse step at every fluid cell.  Arithmetic in FP64 (the adjoint
// recursion has the same slow modes as the forward map, so FP32 rounding of
// per-cell scalars would accumulate the same way); the adjoint populations are
// stored in FP32 or FP64 (PH).
//
// What bounds it: 290 B per cell (record and adjoint populations, mostly from
// beyond the L2) next to about 1 400 VALU instructions per wave, each of which
// alone takes about 100 us on 2.36 M cells, so the waves in flight decide how
// far the two overlap.  With FP32 populations the kernel is held to 168 VGPRs
// for 3 waves per SIMD: 141 us per reverse step at 2.36 M cells (512x320x320
// vessel; 133 us even, 150 us odd), against 169 us at 2 waves and 182 us when
// it also held the neighbours' adjoints in registers and had two population
// buffers.  What keeps the registers down:
//   - the gathers go straight to LDS and are read there where they are used,
//     qhat twice; so do the per-cell accumulators (omega and porosity adjoints);
//   - positions, the tests of the link word and the constants are made again in
//     the later phases (opaque lk, params_again) instead of being held;
//   - at odd n, 11 of the record's values wait in LDS during the forward
//     recompute (53 248 B per workgroup: three workgroups fit the 160 KiB).
// FP64 populations need 60 KB of LDS and the anisotropic medium 20 KB for its
// iterates, so two workgroups per CU, and get the registers of 2 waves per SIMD.
template <bool AN, class PH, bool ODD, int NT>
__device__ __forceinline__ void adjoint_body(const Params& p, const AdjBufs& a, uint32_t t, float ew, int kind,
                                             uint32_t block) {
  using R = double;
  constexpr bool P64 = std::is_same<PH, double>::value;  // FP64 adjoint populations
  // The neighbour gathers (adjoint populations of step n+1 and, for the
  // porosity-jump term, densities of step n-1 at x + c_I) go straight to LDS at
  // the start, so that their latency overlaps the forward recompute without
  // holding registers.  Each wave reads back only the slots its own loads
  // wrote: no barrier, one wait for the loads.
  __shared__ float sq[Q][NT], sr[Q - 1][NT], sh[4][NT];
  // the last pulled values of the record, across the forward recompute (see above)
  constexpr int SDN = ODD && !P64 && !AN ? 11 : 0;
  __shared__ float sd[SDN > 0 ? SDN : 1][NT];
  // anisotropic permeability: |u_m| of the first iterates
  constexpr int NIT = AN ? 10 : 1;
  __shared__ double sn[NIT][NT];
  // FP64 adjoint populations: their high words (the low words go to sq)
  __shared__ float sqh[P64 ? Q : 1][NT];
  const uint32_t c = block * NT + threadIdx.x;
  if (c >= (uint32_t)p.nc) return;
  uint32_t lk = a.links[c];
  if (lk & LK_DEAD) return;
  Pos q = position(p, c, a.code[c]);
  load_deltas(a.delta, q);
  const bool reg = (lk & LK_REG) != 0;
  const float phx_f = ldo(a.phi, c);
  const uint32_t tid = threadIdx.x, wb = tid & ~63u;  // this lane, and its wave's first slot
  // Then the record: the forward recompute waits for these loads only, while
  // the gathers issued after them are still in flight.  The per-cell adjoints
  // read-modified-written at the end are gathered here too, so that neither
  // read stalls the wave later (a wait there would also wait for the stores).
  // Loads complete in issue order for the wait counter, so the row's deltas,
  // which the gather addresses need, are kept ahead of all of these.
  asm volatile("" ::: "memory");
  float d[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) d[i] = __builtin_nontemporal_load(&a.rec[(size_t)i * a.pl + c]);
  const float omp = __builtin_nontemporal_load(&a.rec[(size_t)Q * a.pl + c]);
  constexpr uint32_t PB = sizeof(PH);  // bytes per adjoint population
  const uint32_t plb = a.pl * PB;      // bytes per plane of adjoint populations
  const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(a.ph, (short)0, (int)(plb * (uint32_t)Q), 0x00020000);
  {
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.rho_prev), (short)0,
                                                                        (int)((uint32_t)p.nc * 4u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(a.phih, (short)0, (int)((uint32_t)p.nc * 8u),
                                                                        0x00020000);
    gather_to_lds(rh, &sh[0][wb], c * 8u);
    gather_to_lds(rh, &sh[1][wb], c * 8u + 4u);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(a.omh, (short)0, (int)((uint32_t)p.nc * 8u),
                                                                        0x00020000);
    gather_to_lds(ro, &sh[2][wb], c * 8u);
    gather_to_lds(ro, &sh[3][wb], c * 8u + 4u);
    gather_to_lds(rq, &sq[0][wb], c * PB);
    if constexpr (P64) gather_to_lds(rq, &sqh[0][wb], c * PB + 4u);
    sfor<1, Q>([&](auto ic) {
      constexpr int I = decltype(ic)::value;
      const bool fl = ((lk >> OPP[I]) & 1u) == 0;  // x + c_I is a fluid cell
      const uint32_t tgt = fl ? src_of<OPP[I]>(p, q) : c;  // x + c_I (the cell itself across a wall)
      // the slot of qhat_I at this parity (see the layout above)
      const uint32_t vo = ODD ? (fl ? (uint32_t)I * plb + tgt * PB : (uint32_t)OPP[I] * plb + c * PB) : c * PB;
      const uint32_t so = ODD ? 0u : (uint32_t)OPP[I] * plb;
      gather_to_lds(rq, &sq[I][wb], vo, so);
      if constexpr (P64) gather_to_lds(rq, &sqh[I][wb], vo + 4u, so);
      gather_to_lds(rr, &sr[I - 1][wb], tgt * 4u);
    });
  }

  // ---- forward recompute from the record --------------------------------
  // the record holds the filled values; the Zou-He fills are recomputed for
  // their transposes below (the extrapolation's unknowns are inputs)
  const bool extrap = p.outlet == 2;
  if (!(extrap && (lk & LK_OUT))) open_fill(p, q.row, lk, t, a.shape, a.wave, nullptr, d);
  const Sums<R> sm = moment_sums<R>(d);
  Macro<R> M;
#pragma unroll
  for (int i = 0; i < SDN; ++i) sd[i][tid] = d[Q - SDN + i];
  macro_sums<R, AN>(p, phx_f, sm, omp, M, [&](int m, R n) {
    if (m < NIT) sn[m][tid] = n;
  });
  const R phx = (R)phx_f;
  const R iphi = fast_rcp(phx);
  const auto& kc = params_again().d;
  const R iU = kc.iU;
  const R S = phx + sm.s * iU;  // sum f = phi rho
  const R mx = sm.mx * iU, my = sm.my * iU, mz = sm.mz * iU;
  const R om1 = 1.0 - phx;
  const R kn = kc.kcd * kc.nu_d;
  const R dark = kn * om1 * om1 * iphi * iphi;  // phi nu / k
  const R C0 = 0.5 + 0.25 * dark;
  const R D = phx * dark;                       // phi^2 nu / k
  const R rho = M.rho, ux = M.ux, uy = M.uy, uz = M.uz, uu = M.uu;
  const R Fx = M.Fx, Fy = M.Fy, Fz = M.Fz;
  const R om = M.omega, irho = fast_rcp(rho);
  const R Nn = M.pnorm;  // |Pi|_F
  // Carreau-Yasuda viscosity and its derivative in the shear rate, in FP64
  // like the forward passes of the adjoint
  const R shear = M.shear_r;
  const R la = M.cy_la, fac = M.cy_fac;  // (lambda g)^a and (1 + (lambda g)^a)^((n-1)/a)
  // derivative of (lambda g)^a in g
  const R dla = p.cy_a2 ? 2.0 * kc.lam * kc.lam * shear : ((la > 0.0 && shear > 0.0) ? kc.cy_a * la * fast_rcp(shear) : 0.0);
  const R hh = 1.0 + la;
  const R nu = kc.nu_inf + kc.dnu * fac;
  const R dnu = kc.dnu * kc.cy_e * fac * fast_rcp(hh) * dla;

  // ---- the adjoint of the post-collision populations (staged in LDS) ------
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  // as stored (FP32 or FP64); FP32 values are widened exactly where used, which
  // keeps them in half the registers
  auto rdq = [&](int i) -> PH {
    if constexpr (P64) {
      const uint64_t lo = __builtin_bit_cast(uint32_t, sq[i][tid]), hi = __builtin_bit_cast(uint32_t, sqh[i][tid]);
      return __builtin_bit_cast(double, lo | (hi << 32));
    } else {
      return sq[i][tid];
    }
  };
  // (opaque here and below, so that the tests of its bits are made where they
  // are used instead of being held as 18 lane masks from the gathers on)
  asm volatile("" : "+v"(lk));
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < SDN; ++i) d[Q - SDN + i] = sd[i][tid];
  // moments of a_i = w_i qhat_i over the opposite pairs, in units of 1/36 (36 w_i
  // is 2 on the axis pairs, 1 on the edges), and their sum over the fluid neighbours
  R s0 = 12.0 * (R)rdq(0), s1x = 0.0, s1y = 0.0, s1z = 0.0, s2[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  R sfl = 0.0, qd = (R)rdq(0) * (R)d[0], qd2 = 0.0;
  sfor<0, (Q - 1) / 2>([&](auto kc_) {
    constexpr int I = 1 + 2 * decltype(kc_)::value, J = I + 1;
    const PH qi = rdq(I), qj = rdq(J);
    const bool fi = ((lk >> J) & 1u) == 0, fj = ((lk >> I) & 1u) == 0;  // x + c_I, x + c_J is a fluid cell
    const R ai = I < 7 ? (R)qi + (R)qi : (R)qi, aj = I < 7 ? (R)qj + (R)qj : (R)qj;
    qd = fma((R)qi, (R)d[I], qd);
    qd2 = fma((R)qj, (R)d[J], qd2);
    const R P = ai + aj, Mi = ai - aj;
    s0 += P;
    if constexpr (CX[I] != 0) { s1x += CX[I] > 0 ? Mi : -Mi; s2[0] += P; }
    if constexpr (CY[I] != 0) { s1y += CY[I] > 0 ? Mi : -Mi; s2[1] += P; }
    if constexpr (CZ[I] != 0) { s1z += CZ[I] > 0 ? Mi : -Mi; s2[2] += P; }
    if constexpr (CX[I] * CY[I] != 0) s2[3] += CX[I] * CY[I] > 0 ? P : -P;
    if constexpr (CX[I] * CZ[I] != 0) s2[4] += CX[I] * CZ[I] > 0 ? P : -P;
    if constexpr (CY[I] * CZ[I] != 0) s2[5] += CY[I] * CZ[I] > 0 ? P : -P;
    const R z = (R)0;
    sfl += fi ? ai : z;
    sfl += fj ? aj : z;
  });
  // the porosity-jump sum over the fluid neighbours; in a wave of uniform
  // porosity every term is zero (across a wall the cell's own porosity stands
  // for the neighbour's: an exact zero too)
  R sjump = 0.0;
  if (!__all((lk & LK_UNI) != 0u)) {
    asm volatile("" ::: "memory");
    q = position(p, c, a.code[c]);
    load_deltas(a.delta, q);
    float pn[Q];
    sfor<1, Q>([&](auto ic) {
      constexpr int I = decltype(ic)::value;
      pn[I] = ldo(a.phi, ((lk >> OPP[I]) & 1u) == 0 ? src_of<OPP[I]>(p, q) : c);
    });
    sfor<1, Q>([&](auto ic) {
      constexpr int I = decltype(ic)::value;
      const R ai = I < 7 ? (R)rdq(I) + (R)rdq(I) : (R)rdq(I);
      sjump = fma(ai, (R)pn[I] - phx, sjump);
    });
  }
  constexpr R W36 = 1.0 / 36.0;
  s0 *= W36; s1x *= W36; s1y *= W36; s1z *= W36; sfl *= W36; sjump *= W36;
#pragma unroll
  for (int k = 0; k < 6; ++k) s2[k] *= W36;
  qd = (qd + qd2) * iU;  // sum qhat_i (f_i - w_i phi)

  const R pr = phx * rho;
  const R K = 1.0 - 0.5 * om, keep = 1.0 - om;
  const R uF = ux * Fx + uy * Fy + uz * Fz;
  R s2ux, s2uy, s2uz, s2Fx, s2Fy, s2Fz;
  sym_mv(s2, ux, uy, uz, s2ux, s2uy, s2uz);
  sym_mv(s2, Fx, Fy, Fz, s2Fx, s2Fy, s2Fz);
  const R s1u = s1x * ux + s1y * uy + s1z * uz;
  const R s1F = s1x * Fx + s1y * Fy + s1z * Fz;
  const R us2u = ux * s2ux + uy * s2uy + uz * s2uz;
  const R us2F = ux * s2Fx + uy * s2Fy + uz * s2Fz;
  const R Aeq = phx * M.rm1 - 1.5 * pr * uu;

  // WSS objective term of a region wall cell: e = |tau|, tau = sigma n -
  // (n . sigma n) n, sigma = (omega/2 - 1) Pi.  d|tau| = t . d sigma n with
  // the unit t = tau/|tau|, i.e. the symmetric tensor sym(t n) against d sigma;
  // it reaches Pi scaled by (omega/2 - 1) and omega through Pi/2.
  R wG[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  R wom = 0.0;
  if (kind == 1 && reg && ew != 0.0f) {
    float nw[3];
    if (wall_normal(lk, nw)) {
      R tau[3];
      const R tm = wall_tau(M, nw, tau);
      if (tm > 0.0) {
        const R e = (R)ew / tm;
        const R tx = e * tau[0], ty = e * tau[1], tz = e * tau[2];
        const R nx = nw[0], ny = nw[1], nz = nw[2];
        const R sh[6] = {tx * nx, ty * ny, tz * nz, 0.5 * (tx * ny + ty * nx), 0.5 * (tx * nz + tz * nx),
                         0.5 * (ty * nz + tz * ny)};
        const R sg = 0.5 * M.omega - 1.0;
#pragma unroll
        for (int k = 0; k < 6; ++k) wG[k] = sg * sh[k];
        wom = 0.5 * (sh[0] * M.P[0] + sh[1] * M.P[1] + sh[2] * M.P[2] +
                     2.0 * (sh[3] * M.P[3] + sh[4] * M.P[4] + sh[5] * M.P[5]));
      }
    }
  }

  // collision: q = (1-omega) f + omega feq + K g + w rho (phi~ - phi)
  const uint64_t om_lo = __builtin_bit_cast(uint32_t, sh[2][tid]), om_hi = __builtin_bit_cast(uint32_t, sh[3][tid]);
  R omh = __builtin_bit_cast(double, om_lo | (om_hi << 32)) + wom + (Aeq * s0 + 3.0 * pr * s1u + 4.5 * pr * us2u - qd) -
          0.5 * (3.0 * s1F - 3.0 * s0 * uF + 9.0 * us2F);
  R uhx = K * (9.0 * s2Fx - 3.0 * s0 * Fx), uhy = K * (9.0 * s2Fy - 3.0 * s0 * Fy),
    uhz = K * (9.0 * s2Fz - 3.0 * s0 * Fz);
  R Fhx = K * (3.0 * s1x - 3.0 * s0 * ux + 9.0 * s2ux), Fhy = K * (3.0 * s1y - 3.0 * s0 * uy + 9.0 * s2uy),
    Fhz = K * (3.0 * s1z - 3.0 * s0 * uz + 9.0 * s2uz);
  // equilibrium w phi rho (1 + 3 c.u + 4.5 (c.u)^2 - 1.5 u.u), weighted by omega
  const R brk = om * (s0 * (1.0 - 1.5 * uu) + 3.0 * s1u + 4.5 * us2u);
  const R pro = pr * om;
  uhx += pro * (3.0 * s1x + 9.0 * s2ux - 3.0 * s0 * ux);
  uhy += pro * (3.0 * s1y + 9.0 * s2uy - 3.0 * s0 * uy);
  uhz += pro * (3.0 * s1z + 9.0 * s2uz - 3.0 * s0 * uz);
  R rhoh = phx * brk + sjump;
  R phh = rho * brk - rho * sfl;

  // relaxation rate omega = 2 rho / (6 nu + rho), nu = CY(shear)
  const R rden = 0.5 * om * irho;  // 1 / (6 nu + rho)
  const R id2 = rden * rden;
  rhoh += omh * 12.0 * nu * id2;
  const R nuh = -omh * 12.0 * rho * id2;
  const R gh = nuh * dnu;
  const R omph = gh * 3.0 * Nn * irho;      // adjoint of omega_prev
  const R Nh = gh * 3.0 * (R)omp * irho;
  rhoh -= gh * shear * irho;
  // Pi = sum f c c - phi rho (I/3 + u u) + (F u + u F)/2, |Pi|_F
  const R gsc = Nn > 0.0 ? Nh * fast_rcp(Nn) : 0.0;
  R G[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) G[k] = gsc * M.P[k] + wG[k];
  R Gux, Guy, Guz, GFx, GFy, GFz;
  sym_mv(G, ux, uy, uz, Gux, Guy, Guz);
  sym_mv(G, Fx, Fy, Fz, GFx, GFy, GFz);
  const R tP = (G[0] + G[1] + G[2]) * (1.0 / 3.0) + ux * Gux + uy * Guy + uz * Guz;
  rhoh -= phx * tP;
  phh -= rho * tP;
  uhx += GFx - 2.0 * pr * Gux;
  uhy += GFy - 2.0 * pr * Guy;
  uhz += GFz - 2.0 * pr * Guz;
  Fhx += Gux; Fhy += Guy; Fhz += Guz;
  // kinetic-energy objective e = rho |u|^2 / 2 on region cells
  const R eh = (reg && kind == 0) ? (R)ew : 0.0;
  rhoh += eh * 0.5 * uu;
  uhx += eh * rho * ux; uhy += eh * rho * uy; uhz += eh * rho * uz;
  // force F = rho (g - D u - E |u| u), D = phi^2 nu / k and, with Forchheimer
  // drag, E = phi^3 C_F sqrt(1/k) = K2 (1 - phi) for 0 < phi <= 1 (C_F = 1.75 /
  // sqrt(150 phi^3)), K2 = 1.75 sqrt(K_c / (150 d^2)); d|u|/du := 0 at u = 0.
  // Anisotropic (AN): F = rho (g - D M^-1 u - E |u| M^-1/2 u).
  const bool forch = p.forch != 0;
  const R K2 = kc.fk2;
  const R E = forch ? K2 * om1 : 0.0;
  const R un = forch ? rsqrt_(uu) : 0.0;
  const R dD = -kn * (1.0 - phx * phx) * iphi * iphi;      // dD/dphi
  const R ddark = -2.0 * kn * om1 * iphi * iphi * iphi;    // d(phi nu / k)/dphi
  rhoh += (Fhx * Fx + Fhy * Fy + Fhz * Fz) * irho;
  R vhx, vhy, vhz;
  const R iS = iphi * irho;
  const R vx = mx * iS + 0.5 * kc.gx * iphi, vy = my * iS + 0.5 * kc.gy * iphi, vz = mz * iS + 0.5 * kc.gz * iphi;
  if constexpr (AN) {
    R Mi[6], Mh[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) { Mi[k] = kc.Mi[k]; Mh[k] = kc.Mh[k]; }
    R kdx, kdy, kdz, khx, khy, khz, mfx, mfy, mfz, hfx, hfy, hfz;
    sym_mv(Mi, ux, uy, uz, kdx, kdy, kdz);
    sym_mv(Mh, ux, uy, uz, khx, khy, khz);
    sym_mv(Mi, Fhx, Fhy, Fhz, mfx, mfy, mfz);
    sym_mv(Mh, Fhx, Fhy, Fhz, hfx, hfy, hfz);
    uhx -= rho * (D * mfx + E * un * hfx);
    uhy -= rho * (D * mfy + E * un * hfy);
    uhz -= rho * (D * mfz + E * un * hfz);
    const R Fkd = Fhx * kdx + Fhy * kdy + Fhz * kdz, Fkh = Fhx * khx + Fhy * khy + Fhz * khz;
    if (forch && un > 0.0) {
      const R t = rho * E * Fkh / un;
      uhx -= t * ux; uhy -= t * uy; uhz -= t * uz;
      phh += rho * un * Fkh * K2;
    }
    phh -= rho * Fkd * dD;
    // the fixed-point iterates u_{m+1} = X_m^-1 v, X_m = A + n_m B, n_m = |u_m|,
    // u_0 = v, A = Id + (phi nu / 2k) M^-1, B = C1 M^-1/2: back through the
    // iterates.  n_m alone fixes X_m and so u_{m+1}, and the forward recompute
    // left the first NIT of them in LDS; one adjugate of X_m serves both u_{m+1}
    // and the adjoint (X symmetric).  (Recomputing every u_m from v instead took
    // 27 solves for 6 iterates, now 6: 24.7 -> 20.6 us per reverse step at
    // 118 304 cells with FP64 populations.)
    const R ha = 0.5 * dark, hb = forch ? 0.5 * K2 * om1 * iphi : 0.0;
    struct Adj {
      R a00, a11, a22, a01, a02, a12, id;
      __device__ __forceinline__ void apply(R bx, R by, R bz, R& yx, R& yy, R& yz) const {
        yx = (a00 * bx + a01 * by + a02 * bz) * id;
        yy = (a01 * bx + a11 * by + a12 * bz) * id;
        yz = (a02 * bx + a12 * by + a22 * bz) * id;
      }
    };
    // X^-1 of X = A + n B (the adjugate over the determinant)
    auto inverse = [&](R n) {
      R X[6];
      const R nb = n * hb;
#pragma unroll
      for (int k = 0; k < 6; ++k) X[k] = ha * Mi[k] + nb * Mh[k] + (k < 3 ? 1.0 : 0.0);
      Adj r;
      r.a00 = X[1] * X[2] - X[5] * X[5]; r.a11 = X[0] * X[2] - X[4] * X[4]; r.a22 = X[0] * X[1] - X[3] * X[3];
      r.a01 = X[4] * X[5] - X[3] * X[2]; r.a02 = X[3] * X[5] - X[4] * X[1]; r.a12 = X[3] * X[4] - X[0] * X[5];
      r.id = fast_rcp(X[0] * r.a00 + X[3] * r.a01 + X[4] * r.a02);
      return r;
    };
    // n_m; past the kept ones from the last of them
    auto norm_of = [&](int m) {
      const int k = m < NIT ? m : NIT - 1;
      R n = sn[k][tid];
      for (int j = k; j < m; ++j) {
        R x, y, z;
        inverse(n).apply(vx, vy, vz, x, y, z);
        n = rsqrt_(x * x + y * y + z * z);
      }
      return n;
    };
    R bx = ux, by = uy, bz = uz;        // u_{m+1}
    R ubx = uhx, uby = uhy, ubz = uhz;  // its adjoint
    vhx = 0.0; vhy = 0.0; vhz = 0.0;
    // only two contractions of the adjoints of A and B are needed:
    // aM = sum_m Xh_m : M^-1 and bM = sum_m n_m Xh_m : M^-1/2
    // (the iterates of a wave of pure fluid are all v, and none was kept)
    R aM = 0.0, bM = 0.0, n = __all(phx == 1.0) ? rsqrt_(vx * vx + vy * vy + vz * vz) : norm_of(p.an_iters - 1);
    Adj X = inverse(n);
    for (int m = p.an_iters - 1; m >= 0; --m) {
      R wx, wy, wz;
      X.apply(ubx, uby, ubz, wx, wy, wz);
      vhx += wx; vhy += wy; vhz += wz;
      const R Xh[6] = {-wx * bx, -wy * by, -wz * bz, -(wx * by + wy * bx), -(wx * bz + wz * bx),
                       -(wy * bz + wz * by)};
      R xi = 0.0, xh = 0.0;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        xi += Xh[k] * Mi[k];
        xh += Xh[k] * Mh[k];
      }
      aM += xi;
      bM += n * xh;
      // d/dn of X = n B, contracted with Xh, then through n = |u_m|
      const R g = n > 0.0 ? hb * xh * fast_rcp(n) : 0.0;
      // nothing further back depends on u_m: every remaining term is zero (pure
      // fluid, whose B is zero, leaves after its last iterate)
      if (__all(g == 0.0)) {
        ubx = 0.0; uby = 0.0; ubz = 0.0;
        break;
      }
      if (m > 0) {
        n = norm_of(m - 1);
        X = inverse(n);
        X.apply(vx, vy, vz, bx, by, bz);  // u_m
      } else {
        bx = vx; by = vy; bz = vz;        // u_0
      }
      ubx = g * bx; uby = g * by; ubz = g * bz;
    }
    vhx += ubx; vhy += uby; vhz += ubz;  // u_0 = v
    phh += aM * 0.5 * ddark;
    if (forch) phh += bM * (-0.5 * K2 * iphi * iphi);
  } else {
    uhx -= rho * D * Fhx; uhy -= rho * D * Fhy; uhz -= rho * D * Fhz;
    const R Dh = -rho * (Fhx * ux + Fhy * uy + Fhz * uz);
    phh += Dh * dD;
    if (forch && un > 0.0) {
      const R ku = rho * E * (Fhx * ux + Fhy * uy + Fhz * uz) / un;
      uhx -= rho * E * un * Fhx + ku * ux;
      uhy -= rho * E * un * Fhy + ku * uy;
      uhz -= rho * E * un * Fhz + ku * uz;
      phh -= Dh * un * K2;
    }
    // u = v / den: without Forchheimer den = 2 C0; with it den = C0 + sqrt(C0^2
    // + C1 |v|), C1 = phi^2 C_F sqrt(1/k) / 2 = K2 (1 - phi) / (2 phi)
    R C0h;
    if (!forch) {
      const R i2c = fast_rcp(2.0 * C0);
      vhx = uhx * i2c; vhy = uhy * i2c; vhz = uhz * i2c;
      C0h = -(uhx * ux + uhy * uy + uhz * uz) * 2.0 * i2c;
    } else {
      const R C1 = 0.5 * K2 * om1 * iphi;
      const R vn = rsqrt_(vx * vx + vy * vy + vz * vz);
      const R sq = rsqrt_(C0 * C0 + C1 * vn);
      const R iden = fast_rcp(C0 + sq);
      vhx = uhx * iden; vhy = uhy * iden; vhz = uhz * iden;
      const R denh = -(uhx * ux + uhy * uy + uhz * uz) * iden;
      const R isq = sq > 0.0 ? 0.5 * fast_rcp(sq) : 0.0;
      C0h = denh * (1.0 + 2.0 * C0 * isq);
      const R C1h = denh * vn * isq;
      const R vnh = denh * C1 * isq;
      if (vn > 0.0) {
        const R g = vnh * fast_rcp(vn);
        vhx += g * vx; vhy += g * vy; vhz += g * vz;
      }
      phh += C1h * (-0.5 * K2 * iphi * iphi);
    }
    phh += 0.25 * C0h * ddark;
  }
  // v = m / S + g / (2 phi)
  const R mhx = vhx * iS, mhy = vhy * iS, mhz = vhz * iS;
  R Sh = -(vhx * mx + vhy * my + vhz * mz) * iS * iS;
  phh -= (vhx * kc.gx + vhy * kc.gy + vhz * kc.gz) * 0.5 * iphi * iphi;
  // rho = S / phi
  Sh += rhoh * iphi;
  phh -= rhoh * rho * iphi;

  // adjoint of the (filled) pulled populations; the odd part flips sign within
  // an opposite pair.  qhat is read from LDS again rather than held across the
  // sweep, and the position (for the stores) and the open-face rows likewise.
  asm volatile("" : "+v"(lk) : : "memory");
  q = position(p, c, a.code[c]);
  if (ODD) load_deltas(a.delta, q);
  R fh[Q];
  fh[0] = fma(keep, (R)rdq(0), Sh);
  sfor<0, (Q - 1) / 2>([&](auto kc_) {
    constexpr int I = 1 + 2 * decltype(kc_)::value, J = I + 1;
    constexpr int cx = CX[I], cy = CY[I], cz = CZ[I];
    R ev = Sh, od = 0.0;
    if constexpr (cx != 0) { ev += G[0]; od += cx > 0 ? mhx : -mhx; }
    if constexpr (cy != 0) { ev += G[1]; od += cy > 0 ? mhy : -mhy; }
    if constexpr (cz != 0) { ev += G[2]; od += cz > 0 ? mhz : -mhz; }
    if constexpr (cx * cy != 0) ev = fma(2.0 * (cx * cy), G[3], ev);
    if constexpr (cx * cz != 0) ev = fma(2.0 * (cx * cz), G[4], ev);
    if constexpr (cy * cz != 0) ev = fma(2.0 * (cy * cz), G[5], ev);
    fh[I] = fma(keep, (R)rdq(I), ev + od);
    fh[J] = fma(keep, (R)rdq(J), ev - od);
  });

  // the -x neighbour of an extrapolation-outflow cell: its c_x = -1 pulled
  // values enter the next step's unknowns with weight c_s
  if (extrap && (lk & LK_UPS)) {
    const double* e = a.aside_in + (size_t)q.row * 5;
#pragma unroll
    for (int k = 0; k < 5; ++k) fh[XOUT[k]] += (R)CS * e[k];
  }
  // transpose of the open-face fill: the unknowns' adjoints flow to the knowns
  const bool in = (lk & LK_IN) != 0;
  const bool outl = (lk & LK_OUT) != 0;
  if (outl && extrap) {
    // kept unknowns: total adjoint = this step's part + (1 - c_s) (or 1
    // without a fluid -x neighbour) times the next step's; it goes to the row
    // buffer, not to the pulled-value adjoints (no producer streams there)
    const double* e = a.aside_in + (size_t)q.row * 5;
    double* o = a.aside_out + (size_t)q.row * 5;
    const R wo = ((lk >> 1) & 1u) ? (R)1 : (R)1 - (R)CS;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const bool unk = (lk >> (LK_UNK + k)) & 1u;
      o[k] = unk ? (double)(fh[XOUT[k]] + wo * e[k]) : 0.0;
      if (unk) fh[XOUT[k]] = 0.0;
    }
  }
  if (in) {
    const R uin = (R)inflow_amplitude(p, a.wave, t) * (R)a.shape[q.row];
    fh[2] += fh[1]; fh[8] += fh[7]; fh[10] += fh[9]; fh[12] += fh[11]; fh[14] += fh[13];
    const R rinh = uin * (1.0 / 3.0) * fh[1] + uin * (1.0 / 6.0) * (fh[7] + fh[9] + fh[11] + fh[13]);
    const R nyh = 0.5 * (fh[9] - fh[7]), nzh = 0.5 * (fh[13] - fh[11]);
    const R k = rinh / (1.0 - uin);
    fh[0] += k; fh[3] += k; fh[4] += k; fh[5] += k; fh[6] += k; fh[15] += k; fh[16] += k; fh[17] += k; fh[18] += k;
    fh[2] += 2.0 * k; fh[8] += 2.0 * k; fh[10] += 2.0 * k; fh[12] += 2.0 * k; fh[14] += 2.0 * k;
    fh[3] += nyh; fh[4] -= nyh; fh[15] += nyh; fh[16] -= nyh; fh[17] += nyh; fh[18] -= nyh;
    fh[5] += nzh; fh[6] -= nzh; fh[15] += nzh; fh[16] -= nzh; fh[17] -= nzh; fh[18] += nzh;
    fh[1] = 0.0; fh[7] = 0.0; fh[9] = 0.0; fh[11] = 0.0; fh[13] = 0.0;
  } else if (outl && !extrap) {
    const R ro = kc.rho_out;
    fh[1] += fh[2]; fh[7] += fh[8]; fh[9] += fh[10]; fh[11] += fh[12]; fh[13] += fh[14];
    const R uxh = -ro * (1.0 / 3.0) * fh[2] - ro * (1.0 / 6.0) * (fh[8] + fh[10] + fh[12] + fh[14]);
    const R nyh = 0.5 * (fh[8] - fh[10]), nzh = 0.5 * (fh[12] - fh[14]);
    const R k = uxh / ro;
    fh[0] += k; fh[3] += k; fh[4] += k; fh[5] += k; fh[6] += k; fh[15] += k; fh[16] += k; fh[17] += k; fh[18] += k;
    fh[1] += 2.0 * k; fh[7] += 2.0 * k; fh[9] += 2.0 * k; fh[11] += 2.0 * k; fh[13] += 2.0 * k;
    fh[3] += nyh; fh[4] -= nyh; fh[15] += nyh; fh[16] -= nyh; fh[17] += nyh; fh[18] -= nyh;
    fh[5] += nzh; fh[6] -= nzh; fh[15] += nzh; fh[16] -= nzh; fh[17] -= nzh; fh[18] += nzh;
    fh[2] = 0.0; fh[8] = 0.0; fh[10] = 0.0; fh[12] = 0.0; fh[14] = 0.0;
  }
  // into the slots just read: at odd n to where the producer x - c_i finds it
  // among its own (the cell's own slot across a wall), at even n to (i, x)
  sfor<0, Q>([&](auto ic) {
    constexpr int I = decltype(ic)::value;
    const bool push = ODD && I > 0 && ((lk >> I) & 1u) == 0;  // x - c_I is a fluid cell
    if constexpr (ODD && I > 0)
      put_adjoint<PH>(rq, push ? (uint32_t)OPP[I] * plb + src_of<I>(p, q) * PB : (uint32_t)I * plb + c * PB, 0u, fh[I]);
    else
      put_adjoint<PH>(rq, c * PB, (uint32_t)I * plb, fh[I]);
  });
  a.omh[c] = omph;

  // porosity-jump term of step n-1: q_i(x - c_i) depends on phi(x) when
  // x - c_i is a fluid producer; its adjoint is w_i rho_{n-1}(x - c_i) fh_i(x).
  if (t > 0u) {
    R jump_a = 0.0, jump_e = 0.0;
    sfor<1, Q>([&](auto ic) {
      constexpr int J = decltype(ic)::value;
      // rho_{n-1}(x + c_J), staged in LDS; every slot is read and selected, so
      // that the LDS reads are not serialised behind branches
      const float r = ((lk >> OPP[J]) & 1u) == 0 ? sr[J - 1][tid] : 0.0f;
      if constexpr (J < 7) jump_a = fma((R)r, fh[OPP[J]], jump_a);
      else jump_e = fma((R)r, fh[OPP[J]], jump_e);
    });
    phh += W36 * fma(2.0, jump_a, jump_e);
  }
  const uint64_t ph_lo = __builtin_bit_cast(uint32_t, sh[0][tid]), ph_hi = __builtin_bit_cast(uint32_t, sh[1][tid]);
  a.phih[c] = __builtin_bit_cast(double, ph_lo | (ph_hi << 32)) + phh;
}

template <bool AN, class PH>
constexpr int adjoint_waves() { return AN || std::is_same<PH, double>::value ? 2 : 3; }

template <bool AN, class PH, bool ODD, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(adjoint_waves<AN, PH>())))
void k_adjoint(Params p, AdjBufs a, uint32_t t, float ew, int kind) {
  adjoint_body<AN, PH, ODD, NT>(p, a, t, ew, kind, xcd_block(blockIdx.x, gridDim.x, ODD));
}

// The reverse step of n and a recording step (parity SODD) of the segment before
// it in one launch, the first nblk workgroups and the others: neither depends on
// the other.  For grids that leave the chip idle, where either step is bound by
// the latency of its waves (launch in lbm_adjoint).  With both bodies in one kernel
// most anisotropic forms and one or two of the others need 36 bytes of scratch per
// work-item for scalars beyond the vector lanes that hold spilled ones; k_adjoint
// needs none.
template <bool AN, class PH, bool ODD, bool SODD, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(adjoint_waves<AN, PH>())))
void k_adjoint_and_step(Params p, AdjBufs a, uint32_t t, float ew, int kind, uint32_t nblk, Bufs b) {
  if (blockIdx.x < nblk)
    adjoint_body<AN, PH, ODD, NT>(p, a, t, ew, kind, xcd_block(blockIdx.x, nblk, ODD));
  else
    step_body<float, false, SODD, 0, 1, double, false, NT, AN, 0, true>(
        p, b, xcd_block(blockIdx.x - nblk, nblk, SODD) * NT + threadIdx.x, blockIdx.x == nblk);
}

// Rest state f_i(0, x) = w_i phi(x) on the known links (and on the
// extrapolation outflow's unknowns, whose adjoints of step 0 are in aside0),
// then scatter the total into the box-layout gradient.
template <class PH>
__global__ __launch_bounds__(BLOCK) void k_adj_final(Params p, const uint32_t* code, const uint32_t* links,
                                                     const uint32_t* rowbox, const PH* ph0, uint32_t pl, const double* total,
                                                     const double* aside0, float* grad) {
  const uint32_t c = blockIdx.x * BLOCK + threadIdx.x;
  if (c >= (uint32_t)p.nc) return;
  const uint32_t lk = links[c];
  if (lk & LK_DEAD) return;
  const Pos q = position(p, c, code[c]);
  double s = total[c];
#pragma unroll
  for (int i = 0; i < Q; ++i) s += (double)kw(i) * (1.0 / 36.0) * (double)ldo(ph0, (uint32_t)i * pl + c);
  if (p.outlet == 2 && (lk & LK_OUT)) {
#pragma unroll
    for (int k = 0; k < 5; ++k) s += (double)kw(XOUT[k]) * (1.0 / 36.0) * aside0[(size_t)q.row * 5 + k];
  }
  grad[(size_t)rowbox[q.row] + (size_t)q.x] = (float)s;
}

}  // namespace lbm
