// Host runtime shared by the translation units of liblbm.so: the context, the
// workspace layout, the launch helpers, and the per-storage launch functions
// (each family of kernels is instantiated in a translation unit of its own so
// that the library builds in parallel).
#pragma once
#include "lbm.h"

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <type_traits>
#include <vector>

#include "layout.hpp"
#include "step.hpp"
#include "step27.hpp"

namespace lbmrt {

using namespace lbm;

// Error message of the last failure (thread-local) and status.
lbm_status fail(lbm_status s, const std::string& msg);

inline size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }
inline size_t store_bytes(int storage) { return storage == LBM_STORE_FP32 ? 4 : 2; }
inline int qof(const lbm_grid& g) { return g.velocity_set == 27 ? 27 : 19; }
inline int blocks_for(int64_t n) { return (int)((n + BLOCK - 1) / BLOCK); }
inline int blocks_for_nt(int64_t n, int nt) { return (int)((n + nt - 1) / nt); }

// Work-items per workgroup of the step kernel: 256 on large grids, single waves on
// small ones (step_width).
constexpr int STEP_NT_MIN = 64;
constexpr int MAX_WAVE_TABLE = 1024;  // samples of a sampled inflow waveform
constexpr int STEP_NT16 = 256;  // work-items per workgroup of the 16-bit step kernels
// Infinity Cache (last-level, memory-side) of MI355X, bytes.
constexpr size_t INFINITY_CACHE_BYTES = (size_t)256 << 20;
inline int step_nt(int storage) { return storage == LBM_STORE_FP32 ? 256 : STEP_NT16; }

// Compact cells up to which lbm_adjoint records a segment in the launches that
// reverse the one after it (k_adjoint_and_step). Whole call, the two in turn ->
// together: 11 968 cells 2 235 -> 1 748 us, 37 736 2 932 -> 2 345 us, 118 304 6 005 ->
// 5 061 us (checkpoints every 16 or 20 steps); 296 748 5 986 -> 5 500 us, 538 068
// 9 089 -> 8 538 us, 823 756 12 786 -> 12 187 us, 1 308 792 18 728 -> 18 643 us (with the
// anisotropic medium and FP64 populations 19 396 -> 19 037 and 28 665 -> 32 568 us
// for the last two), 2 360 212 27 023 -> 31 349 us.  One line for the four forms, just
// below the largest size at which each of those measured gains; alone, the isotropic
// FP32 form breaks even at about 1.3 M cells, the anisotropic FP64 form loses there.
constexpr int64_t TOGETHER_CELLS = 786432;

struct Layout {
  size_t A, code, links, phi, omega, delta, rel, winfo, wrank, shape, rowbox, lines, stage, part, diag, obj, tc, wave, side;
  // adjoint
  size_t ck, rec, rho, ah, omh, phih, aside;
  int nck, ckpt, T;
  size_t total;
};

}  // namespace lbmrt

// A context: its host layout (box, rows, per-cell tables, fluid-cell lists)
// plus the run's parameters, workspace and state.
struct lbm_ctx : lbmrt::HostLayout {
  lbm_grid grid{};
  lbm_rheology rh{};
  lbm_porous po{};
  lbm_open op{};
  size_t nbox = 0;
  int nblk = 0;                   // blocks of BLOCK work-items over the compact cells
  int sblk = 0;                   // blocks of the step kernel
  size_t state_bytes = 0;         // the step's state: populations and per-cell arrays
  bool beyond_cache = false;      // it exceeds the Infinity Cache
  int64_t nwss = 0;               // region cells on the wall (with a wall normal)
  int q = 19;                     // velocity set
  double U = 36.0;
  int device = 0;                 // HIP device of the workspace (current at lbm_create)
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  lbmrt::Layout L{};
  int64_t t = 0;                  // time; its parity selects the slot layout
  bool poisoned = false;
  lbm::Params P{};
  float omega0 = 1.0f;
  double* host_out = nullptr;     // slot of pinned, mapped memory for a reduction's result (null: none, see finalize)
  int amode = 1;                  // collision arithmetic: 0 FP32, 1 FP32 + projection, 2 FP64
};

#define HIP_TRY(ctx, expr)                                                                      \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess) {                                                                     \
      if (ctx) (ctx)->poisoned = true;                                                          \
      return ::lbmrt::fail(LBM_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_));    \
    }                                                                                           \
  } while (0)

#define CTX_CHECK(ctx)                                                                          \
  do {                                                                                          \
    if (!(ctx)) return ::lbmrt::fail(LBM_E_INVALID, "null context");                            \
    if ((ctx)->poisoned) return ::lbmrt::fail(LBM_E_STATE, "context poisoned by an earlier device error"); \
  } while (0)

namespace lbmrt {

struct TF32 { using T = float; };
struct TF16 { using T = _Float16; };
struct TBF16 { using T = __bf16; };
// Arithmetic of the collision: FP32, FP32 with the FP64 momentum projection,
// or FP64.
struct RF32 { using T = float; static constexpr bool proj = false; };
struct RF32P { using T = float; static constexpr bool proj = true; };
struct RF64 { using T = double; static constexpr bool proj = false; };

template <class Fn>
void with_shift(int shw, Fn&& fn) {
  if (shw) fn(std::true_type{}); else fn(std::false_type{});
}

// Rounding of the 16-bit storage forms (lbm_rounding, see round16 in
// step.hpp); FP32 storage has one form.
template <class S, class Fn>
void with_rounding(int rounding, Fn&& fn) {
  using std::integral_constant;
  if constexpr (std::is_same<S, float>::value) fn(integral_constant<int, 0>{});
  else if (rounding == LBM_ROUND_NEAREST) fn(integral_constant<int, 0>{});
  else if (rounding == LBM_ROUND_CONSERVE) fn(integral_constant<int, 1>{});
  else fn(integral_constant<int, 2>{});
}

// Arithmetic for storage S: the FP64 and projected forms only exist for FP32
// storage.  mode: 0 FP32, 1 FP32 + projection, 2 FP64.
template <class S, class Fn>
void with_arith(int mode, Fn&& fn) {
  if constexpr (std::is_same<S, float>::value) {
    if (mode == 2) fn(RF64{});
    else if (mode == 1) fn(RF32P{});
    else fn(RF32{});
  } else {
    fn(RF32{});
  }
}

template <class Fn>
void with_parity(int64_t t, Fn&& fn) {
  if (t & 1) fn(std::true_type{}); else fn(std::false_type{});
}

Layout make_layout(const lbm_grid& g, int64_t nc, int64_t nrow, int T, int ckpt);
lbm::Bufs bufs(lbm_ctx* c);
lbm::q27::Bufs27 bufs27(lbm_ctx* c);

// Per-storage launch functions (kernels instantiated in their own units).
// diag: 0 none, 1 diagnostics partials, 2 region kinetic energy, 3 region
// wall shear stress, accumulated into the objective partials; rec: 1 record
// the step for the adjoint, 2 step from a record (FP32 storage, shift mode 0 only).
template <class S> void step19(lbm_ctx* c, const lbm::Bufs& b, int diag, int rec);
template <class S> void moments19(lbm_ctx* c, const lbm::Bufs& b, const lbm::Dense& out);
template <class S> void diag19(lbm_ctx* c, const lbm::Bufs& b);
template <class S> void init19(lbm_ctx* c, const lbm::Bufs& b);
// FP64 populations of directions [i0, i1) and omega (null: neither read nor
// written) in fluid order, device to device.
template <class S> void state_out19(lbm_ctx* c, const lbm::Bufs& b, double* f, float* omega, int i0, int i1);
template <class S> void state_in19(lbm_ctx* c, const lbm::Bufs& b, const double* f, const float* omega, int i0, int i1);
template <class S> void step27(lbm_ctx* c, const lbm::q27::Bufs27& b, int diag);
template <class S> void moments27(lbm_ctx* c, const lbm::q27::Bufs27& b, const lbm::Dense& out);
template <class S> void diag27(lbm_ctx* c, const lbm::q27::Bufs27& b);
template <class S> void init27(lbm_ctx* c, const lbm::q27::Bufs27& b);
template <class S> void state_out27(lbm_ctx* c, const lbm::q27::Bufs27& b, double* f, float* omega, int i0, int i1);
template <class S> void state_in27(lbm_ctx* c, const lbm::q27::Bufs27& b, const double* f, const float* omega, int i0,
                                   int i1);

// Workgroups of k_moments outside the rows.
inline unsigned dense_blocks(const lbm::Dense& out) {
  return out.rest ? (out.nbox + lbm::DENSE_REST - 1) / lbm::DENSE_REST : 0u;
}

// Blocks of 256 cells per workgroup of k_diag, and its workgroups (no more
// than the context's blocks, whose partial rows the workspace holds).
inline uint32_t diag_run(const lbm_ctx* c) { return (uint32_t)((c->nblk + DIAG_BLOCKS - 1) / DIAG_BLOCKS); }
inline int diag_blocks(const lbm_ctx* c) { return (c->nblk + (int)diag_run(c) - 1) / (int)diag_run(c); }

// Work-items per workgroup of a step: single waves on grids of less than `line`
// workgroups of 256, where whole workgroups leave some CUs with one more than others
// and a wave waits for its CU's memory pipe.  At most three (FP32 D3Q19 step) or four
// (the others) workgroups per CU, from both widths at 16 to 1 300 workgroups (boxes,
// channels, vessels; whole -> single waves, us per step):
//   FP32 D3Q19: 272 workgroups 6.05 -> 5.82, 733 8.60 -> 8.50, 760 8.20 -> 8.28; above three
//     per CU 880 9.15 -> 8.80, but 781 8.8 -> 9.4, 800 8.6 -> 9.0, 992 9.1 -> 9.4, 1 020 8.8 -> 9.3;
//   16-bit D3Q19: 528 6.39 -> 6.09, 720 6.71 -> 6.55, 981 7.98 -> 7.88, 1 040 8.16 -> 8.22;
//   D3Q27, FP32 and BF16: 528 9.01 -> 8.85 and 7.44 -> 7.22, 900 11.11 -> 11.21 and 9.23 ->
//     9.18, 989 11.61 -> 11.34 and 10.28 -> 10.13, 1 020 11.50 -> 11.57 and 9.29 -> 9.35;
//   a gradient of 40 steps (FP32; anisotropic, FP64 populations): 285 977 -> 920 and
//     1 197 -> 1 134, 911 1 631 -> 1 616 and 2 215 -> 2 167.
// Where the workgroups come out even (just below a multiple of 256) the two are
// equal or single waves up to 2 % slower; on 2.36 M cells they are 1 % slower.
constexpr int NARROW_FP32_D3Q19 = 768, NARROW_GRID = 1024;
inline int step_width(const lbm_ctx* c, int nt, int line = NARROW_GRID) { return c->nblk < line ? 64 : nt; }

// Storage dispatch for the per-storage launch functions.
template <class Fn>
void with_storage(int storage, Fn&& fn) {
  if (storage == LBM_STORE_FP32) fn(TF32{});
  else if (storage == LBM_STORE_FP16) fn(TF16{});
  else fn(TBF16{});
}

// Kernels without a storage type (kmisc.hip).
void launch_finalize(hipStream_t s, const double* part, int nparts, int n, uint32_t ops, double* out);
// n > 0 floats to zero, by a kernel, so that the calls that clear can be captured: memsets
// recorded into a graph left wrong values on its replays.
void launch_zero(hipStream_t s, float* p, size_t n);
void launch_copy(hipStream_t s, const void* src, void* dst, size_t n16, unsigned blocks);
void launch_probe(hipStream_t s, int kind, const void* src, void* dst, size_t n16, unsigned blocks);
lbm_status set_porosity_device(lbm_ctx* c, const float* phib, uint32_t* bad_cell);
lbm_status launch_wave_info(lbm_ctx* c);

// Runtime operations shared by the ABI functions (lbm.hip).
lbm_status launch_init(lbm_ctx* c);
// from: rec holds the record to step from (b.t = c->t) instead of receiving one
lbm_status launch_step(lbm_ctx* c, int diag, float* rec, float* rho_rec, bool from = false);
// dev_out: device area for the reduced vector of a context without a host slot (null: the workspace's)
lbm_status finalize(lbm_ctx* c, const double* part, int nparts, int n, uint32_t ops, double* out,
                    double* dev_out = nullptr);

}  // namespace lbmrt
