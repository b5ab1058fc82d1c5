// Launches of the D3Q27 kernels for one storage type S (instantiated in
// k27_f32.hip and k27_16.hip).
#pragma once
#include "runtime.hpp"

namespace lbmrt {

template <class S>
void step27(lbm_ctx* c, const lbm::q27::Bufs27& b, int diag) {
  constexpr int NT = std::is_same<S, float>::value ? 256 : STEP_NT16;
  const int nt = diag == 1 ? NT : step_width(c, NT);
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
          if (diag == 0)
            hipLaunchKernelGGL((q27::k_step<S, SH, OD, 0, R, PJ, NT, RM>), grid, block, 0, c->stream, c->P, b);
          else
            hipLaunchKernelGGL((q27::k_step<S, SH, OD, 1, R, PJ, NT, RM>), grid, block, 0, c->stream, c->P, b);
        });
      });
    });
  });
}

template <class S, class Fn>
void with_state_form27(lbm_ctx* c, Fn&& fn) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    with_arith<S>(c->amode == 2 ? 2 : 0, [&](auto rt) {
      with_parity(c->t, [&](auto odd) { fn(shw, rt, odd); });
    });
  });
}

template <class S>
void moments27(lbm_ctx* c, const lbm::q27::Bufs27& b, const lbm::Dense& out) {
  with_state_form27<S>(c, [&](auto shw, auto rt, auto odd) {
    hipLaunchKernelGGL((q27::k_moments<S, decltype(shw)::value, decltype(odd)::value, typename decltype(rt)::T>),
                       dim3(c->nblk + dense_blocks(out)), dim3(BLOCK), 0, c->stream, c->P, b, (uint32_t)c->t,
                       (uint32_t)c->nblk, out);
  });
}

template <class S>
void diag27(lbm_ctx* c, const lbm::q27::Bufs27& b) {
  with_state_form27<S>(c, [&](auto shw, auto rt, auto odd) {
    hipLaunchKernelGGL((q27::k_diag<S, decltype(shw)::value, decltype(odd)::value, typename decltype(rt)::T>),
                       dim3(diag_blocks(c)), dim3(BLOCK), 0, c->stream, c->P, b, (uint32_t)c->t, diag_run(c));
  });
}

template <class S>
void init27(lbm_ctx* c, const lbm::q27::Bufs27& b) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    hipLaunchKernelGGL((q27::k_init<S, decltype(shw)::value>), dim3(c->nblk), dim3(BLOCK), 0, c->stream, c->P, b,
                       c->omega0);
  });
}

template <class S>
void state_out27(lbm_ctx* c, const lbm::q27::Bufs27& b, double* f, float* omega, int i0, int i1) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    with_parity(c->t, [&](auto odd) {
      hipLaunchKernelGGL((q27::k_state_out<S, decltype(shw)::value, decltype(odd)::value>), dim3(c->nblk), dim3(BLOCK), 0,
                         c->stream, c->P, b, (const uint32_t*)(c->ws + c->L.wrank), f, omega, i0, i1, (uint32_t)c->nf);
    });
  });
}

template <class S>
void state_in27(lbm_ctx* c, const lbm::q27::Bufs27& b, const double* f, const float* omega, int i0, int i1) {
  with_shift(c->grid.shift_mode, [&](auto shw) {
    with_parity(c->t, [&](auto odd) {
      hipLaunchKernelGGL((q27::k_state_in<S, decltype(shw)::value, decltype(odd)::value>), dim3(c->nblk), dim3(BLOCK), 0,
                         c->stream, c->P, b, (const uint32_t*)(c->ws + c->L.wrank), f, omega, i0, i1, (uint32_t)c->nf);
    });
  });
}

}  // namespace lbmrt

#define LBM_INSTANTIATE27(S)                                                                                      \
  namespace lbmrt {                                                                                               \
  template void step27<S>(lbm_ctx*, const lbm::q27::Bufs27&, int);                                                \
  template void moments27<S>(lbm_ctx*, const lbm::q27::Bufs27&, const lbm::Dense&);                               \
  template void diag27<S>(lbm_ctx*, const lbm::q27::Bufs27&);                                                     \
  template void init27<S>(lbm_ctx*, const lbm::q27::Bufs27&);                                                     \
  template void state_out27<S>(lbm_ctx*, const lbm::q27::Bufs27&, double*, float*, int, int); \
  template void state_in27<S>(lbm_ctx*, const lbm::q27::Bufs27&, const double*, const float*, int, int); \
  }
