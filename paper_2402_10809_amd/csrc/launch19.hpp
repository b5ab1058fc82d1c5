// Launches of the D3Q19 kernels for one storage type S (instantiated in
// k19_f32.hip, k19_f16.hip and k19_bf16.hip).
#pragma once
#include "runtime.hpp"

namespace lbmrt {

template <class S>
void step19(lbm_ctx* c, const lbm::Bufs& b, int diag, int rec) {
  constexpr int NT = std::is_same<S, float>::value ? 256 : STEP_NT16;
  const int nt = diag == 1 ? NT : step_width(c, NT, std::is_same<S, float>::value && c->amode != 2 ? NARROW_FP32_D3Q19 : NARROW_GRID);
  const dim3 grid((unsigned)blocks_for_nt(c->nc, nt)), block((unsigned)nt);
  with_shift(c->grid.shift_mode, [&](auto shw) {
    constexpr bool SH = decltype(shw)::value;
    with_arith<S>(c->amode, [&](auto rt) {
      using R = typename decltype(rt)::T;
      constexpr bool PJ = decltype(rt)::proj;
      with_rounding<S>(c->grid.rounding, [&](auto cr) {
        constexpr int RM = decltype(cr)::value;
        with_parity(c->t, [&](auto odd) {
          constexpr bool OD = decltype(odd)::value;
          // AN: anisotropic permeability (every form, the adjoint's included)
          auto go = [&](auto an) {
            constexpr bool AN = decltype(an)::value;
            if (diag == 0 && !rec) {
              if constexpr (sizeof(S) == 2) {
                // wave records: when the state exceeds the Infinity Cache, and
                // with rounding to nearest, whose step has the fewest VALU
                // instructions (with stochastic rounding they gain nothing)
                if (c->beyond_cache || RM == 0)
                  hipLaunchKernelGGL((k_step<S, SH, OD, 0, 0, R, PJ, NT, AN, RM, true>), grid, block, 0,
                                     c->stream, c->P, b);
                else
                  hipLaunchKernelGGL((k_step<S, SH, OD, 0, 0, R, PJ, NT, AN, RM, false>), grid, block, 0,
                                     c->stream, c->P, b);
              } else {
                hipLaunchKernelGGL((k_step<S, SH, OD, 0, 0, R, PJ, NT, AN, RM>), grid, block, 0, c->stream,
                                   c->P, b);
              }
            } else if (diag == 1) {
              hipLaunchKernelGGL((k_step<S, SH, OD, 1, 0, R, PJ, NT, AN, RM>), grid, block, 0, c->stream, c->P,
                                 b);
            } else if constexpr (std::is_same<S, float>::value) {
              // the adjoint's forms (FP32 storage only)
              if (rec) {
                // the recording step, with the objective term in the forward
                // pass, and the step from a checkpoint's record (the
                // adjoint's passes compute in FP64)
                if constexpr (!SH && std::is_same<R, double>::value) {
                  if (rec == 2)
                    hipLaunchKernelGGL((k_step<S, false, OD, 0, 2, R, PJ, NT, AN>), grid, block, 0, c->stream, c->P,
                                       b);
                  else if (diag == 2)
                    hipLaunchKernelGGL((k_step<S, false, OD, 2, 1, R, PJ, NT, AN>), grid, block, 0, c->stream, c->P,
                                       b);
                  else if (diag == 3)
                    hipLaunchKernelGGL((k_step<S, false, OD, 3, 1, R, PJ, NT, AN>), grid, block, 0, c->stream, c->P,
                                       b);
                  else
                    hipLaunchKernelGGL((k_step<S, false, OD, 0, 1, R, PJ, NT, AN>), grid, block, 0, c->stream, c->P,
                                       b);
                }
              } else if (diag == 2) {
                hipLaunchKernelGGL((k_step<S, SH, OD, 2, 0, R, PJ, NT, AN>), grid, block, 0, c->stream, c->P,
                                   b);
              } else {
                hipLaunchKernelGGL((k_step<S, SH, OD, 3, 0, R, PJ, NT, AN>), grid, block, 0, c->stream, c->P,
                                   b);
              }
            }
          };
          if (c->P.an_iters > 0) go(std::true_type{});
          else go(std::false_type{});
        });
      });
    });
  });
}

// The forms of k_moments and k_diag: shift, arithmetic, parity, anisotropy.
template <class S, class Fn>
void with_state_form(lbm_ctx* c, Fn&& fn) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    with_arith<S>(c->amode == 2 ? 2 : 0, [&](auto rt) {
      with_parity(c->t, [&](auto odd) {
        if (c->P.an_iters > 0) fn(shw, rt, odd, std::true_type{});
        else fn(shw, rt, odd, std::false_type{});
      });
    });
  });
}

template <class S>
void moments19(lbm_ctx* c, const lbm::Bufs& b, const lbm::Dense& out) {
  with_state_form<S>(c, [&](auto shw, auto rt, auto odd, auto an) {
    hipLaunchKernelGGL((k_moments<S, decltype(shw)::value, decltype(odd)::value, typename decltype(rt)::T,
                                  decltype(an)::value>),
                       dim3(c->nblk + dense_blocks(out)), dim3(BLOCK), 0, c->stream, c->P, b, (uint32_t)c->t,
                       (uint32_t)c->nblk, out);
  });
}

template <class S>
void diag19(lbm_ctx* c, const lbm::Bufs& b) {
  with_state_form<S>(c, [&](auto shw, auto rt, auto odd, auto an) {
    hipLaunchKernelGGL((k_diag<S, decltype(shw)::value, decltype(odd)::value, typename decltype(rt)::T,
                               decltype(an)::value>),
                       dim3(diag_blocks(c)), dim3(BLOCK), 0, c->stream, c->P, b, (uint32_t)c->t, diag_run(c));
  });
}

template <class S>
void init19(lbm_ctx* c, const lbm::Bufs& b) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    hipLaunchKernelGGL((k_init<S, decltype(shw)::value>), dim3(c->nblk), dim3(BLOCK), 0, c->stream, c->P, b,
                       c->omega0);
  });
}

template <class S>
void state_out19(lbm_ctx* c, const lbm::Bufs& b, double* f, float* omega, int i0, int i1) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    with_parity(c->t, [&](auto odd) {
      hipLaunchKernelGGL((k_state_out<S, decltype(shw)::value, decltype(odd)::value>), dim3(c->nblk), dim3(BLOCK), 0,
                         c->stream, c->P, b, (const uint32_t*)(c->ws + c->L.wrank), f, omega, i0, i1, (uint32_t)c->nf);
    });
  });
}

template <class S>
void state_in19(lbm_ctx* c, const lbm::Bufs& b, const double* f, const float* omega, int i0, int i1) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    with_parity(c->t, [&](auto odd) {
      hipLaunchKernelGGL((k_state_in<S, decltype(shw)::value, decltype(odd)::value>), dim3(c->nblk), dim3(BLOCK), 0,
                         c->stream, c->P, b, (const uint32_t*)(c->ws + c->L.wrank), f, omega, i0, i1, (uint32_t)c->nf);
    });
  });
}

}  // namespace lbmrt

#define LBM_INSTANTIATE19(S)                                                                                    \
  namespace lbmrt {                                                                                             \
  template void step19<S>(lbm_ctx*, const lbm::Bufs&, int, int);                                                \
  template void moments19<S>(lbm_ctx*, const lbm::Bufs&, const lbm::Dense&);                                    \
  template void diag19<S>(lbm_ctx*, const lbm::Bufs&);                                                          \
  template void init19<S>(lbm_ctx*, const lbm::Bufs&);                                                          \
  template void state_out19<S>(lbm_ctx*, const lbm::Bufs&, double*, float*, int, int); \
  template void state_in19<S>(lbm_ctx*, const lbm::Bufs&, const double*, const float*, int, int); \
  }
