// Launchers of the pass kernels: launch geometry, the choice between the component-split
// passes (sgp_passes.hpp) and the line kernels (sgp_lines.hpp), and the per-plan dispatch.
#pragma once
#include <hip/hip_ext.h>

#include "sgp_lines.hpp"

namespace sgp {

// ---------------------------------------------------------------------------
// Launch geometry of a register plan (N, E): TL = N/E threads per line and
// component; W lines per block so that a block has 320 threads (W = 64/TL), or one
// line of 5 TL threads when TL > 64.  Every instantiation of a plan (alone or in
// an ensemble) uses this geometry, so its results do not depend on the caller.
// ---------------------------------------------------------------------------
template <int N, int E>
struct Geo {
  static constexpr int TL = N / E;
  static constexpr int W = TL >= 64 ? 1 : 64 / TL;
  static constexpr int NT = W * 5 * TL;
};

// Blocks of a pass with W lines per block.
template <int W, int KIND>
static long pass_blocks(const PassArgs& a) {
  return KindInfo<KIND>::XL ? (a.nlines + W - 1) / W : ((a.ncols + W - 1) / W) * a.nouter;
}

// ev: null, or two events that the dispatch itself stamps with the kernel's start
// and end (timing without marker packets between the kernels).
template <typename T, int N, int E, int W, int KIND>
static hipError_t pass_w(cx<T>* psi, const PassArgs& a, hipStream_t st, const hipEvent_t* ev) {
  constexpr int NT = W * 5 * (N / E);
  const long nblocks = pass_blocks<W, KIND>(a) + ((KIND == C_PROP || KIND == C_KIN) && a.advance_clock ? 1 : 0);
  if (ev)
    hipExtLaunchKernelGGL((k_pass<T, N, E, W, KIND>), dim3((unsigned)nblocks), dim3(NT), 0, st, ev[0], ev[1], 0, psi,
                          a);
  else
    hipLaunchKernelGGL((k_pass<T, N, E, W, KIND>), dim3((unsigned)nblocks), dim3(NT), 0, st, psi, a);
  return hipGetLastError();
}

template <typename T, int N, int E, int KIND>
static hipError_t line_n(cx<T>* psi, const PassArgs& a, hipStream_t st, const hipEvent_t* ev) {
  constexpr int W = 64 / (N / E);
  const long tiles = pass_blocks<W, KIND>(a);
  const long nblocks = (tiles + kLineWaves - 1) / kLineWaves +
                       ((KIND == C_PROP || KIND == C_KIN) && a.advance_clock ? 1 : 0);
  if (ev)
    hipExtLaunchKernelGGL((k_line<T, N, E, KIND>), dim3((unsigned)nblocks), dim3(64 * kLineWaves), 0, st, ev[0], ev[1],
                          0, psi, a);
  else
    hipLaunchKernelGGL((k_line<T, N, E, KIND>), dim3((unsigned)nblocks), dim3(64 * kLineWaves), 0, st, psi, a);
  return hipGetLastError();
}

// Lines per block: Geo's W, or, where that would leave CUs without a block (fewer than 256
// blocks), one line, but at least 40 threads: lines of 16 and 32 points have 10 or 20, and a
// step of many such lines spends its time on the start of their blocks.  TS2 step in us with
// one line / 40 / 80 threads / Geo's W: 16x16 complex64 10.8 / 10.1 / 10.3 / 12.1, 16x512 16.0 /
// 13.4 / 13.5 / 15.2, 32^3 complex128 18.1 / 16.8 / 17.0 / 23.9, 16x16x128 18.9 / 15.3 / 15.4 /
// 20.7 (Geo's W in an older build); 64 points (40 threads a line) 10.7 / - / 11.3 / 13.7.
// Nothing of a line's arithmetic depends on W.
template <typename T, int N, int E, int KIND>
static hipError_t pass_n(cx<T>* psi, const PassArgs& a, hipStream_t st, const hipEvent_t* ev) {
  constexpr int W = Geo<N, E>::W, TL = Geo<N, E>::TL;
  if constexpr (W > 1) {
    if (pass_blocks<W, KIND>(a) < 256) return pass_w<T, N, E, (TL < 8 ? 8 / TL : 1), KIND>(psi, a, st, ev);
  }
  return pass_w<T, N, E, W, KIND>(psi, a, st, ev);
}

template <typename T, int N, int E>
static hipError_t pass_kind(int kind, cx<T>* psi, const PassArgs& a, hipStream_t st, const hipEvent_t* ev) {
  switch (kind) {
    case X_FIRST: return pass_n<T, N, E, X_FIRST>(psi, a, st, ev);
    case X_MID: return pass_n<T, N, E, X_MID>(psi, a, st, ev);
    case X_LAST: return pass_n<T, N, E, X_LAST>(psi, a, st, ev);
    case X_NLONLY: return pass_n<T, N, E, X_NLONLY>(psi, a, st, ev);
    case C_PROP: return pass_n<T, N, E, C_PROP>(psi, a, st, ev);
    case C_KIN: return pass_n<T, N, E, C_KIN>(psi, a, st, ev);
    case XA_FIRST: return pass_n<T, N, E, XA_FIRST>(psi, a, st, ev);
    case XA_MID: return pass_n<T, N, E, XA_MID>(psi, a, st, ev);
    case XA_LAST: return pass_n<T, N, E, XA_LAST>(psi, a, st, ev);
    case C_ADJ: return pass_n<T, N, E, C_ADJ>(psi, a, st, ev);
    case X_SHEAR: return pass_n<T, N, E, X_SHEAR>(psi, a, st, ev);
    case C_SHEAR: return pass_n<T, N, E, C_SHEAR>(psi, a, st, ev);
    case X_FWD: return pass_n<T, N, E, X_FWD>(psi, a, st, ev);
    case X_INV: return pass_n<T, N, E, X_INV>(psi, a, st, ev);
    default: return hipErrorInvalidValue;
  }
}

// All pass kernels of one register-plan width E (every supported
// line length with that E).  Each (T, E) pair is compiled in its own translation
// unit.
#define SGP_FOR_PLAN_N(E, X)                                     \
  X(16, E) X(32, E) X(64, E) X(128, E) X(192, E) X(256, E) X(384, E) X(512, E) X(768, E)

template <typename T, int E>
hipError_t launch_pass_e(int kind, void* psi, const PassArgs& a, int n, hipStream_t st, const hipEvent_t* ev) {
  cx<T>* p = reinterpret_cast<cx<T>*>(psi);
#define SGP_CASE(NN, EE) \
  case NN:               \
    if constexpr (plan_ok(NN, EE, (int)sizeof(T))) return pass_kind<T, NN, EE>(kind, p, a, st, ev); \
    break;
  switch (n) { SGP_FOR_PLAN_N(E, SGP_CASE) default: break; }
#undef SGP_CASE
  return hipErrorInvalidValue;
}

template <typename T, int N, int E>
static hipError_t line_kind(int kind, cx<T>* psi, const PassArgs& a, hipStream_t st, const hipEvent_t* ev) {
  switch (kind) {
    case X_FIRST: return line_n<T, N, E, X_FIRST>(psi, a, st, ev);
    case X_MID: return line_n<T, N, E, X_MID>(psi, a, st, ev);
    case X_LAST: return line_n<T, N, E, X_LAST>(psi, a, st, ev);
    case C_PROP: return line_n<T, N, E, C_PROP>(psi, a, st, ev);
    case C_KIN: return line_n<T, N, E, C_KIN>(psi, a, st, ev);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int E>
hipError_t launch_line_e(int kind, void* psi, const PassArgs& a, int n, hipStream_t st, const hipEvent_t* ev) {
  cx<T>* p = reinterpret_cast<cx<T>*>(psi);
#define SGP_CASE(NN, EE) \
  case NN:               \
    if constexpr (line_ok(NN, EE, (int)sizeof(T))) return line_kind<T, NN, EE>(kind, p, a, st, ev); \
    break;
  switch (n) { SGP_FOR_PLAN_N(E, SGP_CASE) default: break; }
#undef SGP_CASE
  return hipErrorInvalidValue;
}

template <typename T, int E>
hipError_t launch_line_batched_e(int kind, const int2* it, const PassArgs* ar, long nitems, hipStream_t st) {
  if constexpr (batched_line_plan(E, (int)sizeof(T))) {
    dim3 g((unsigned)nitems), b(64 * kLineWaves);
    switch (kind) {
      case X_FIRST: hipLaunchKernelGGL((k_line_batched<T, X_FIRST, E>), g, b, 0, st, it, ar); break;
      case X_MID: hipLaunchKernelGGL((k_line_batched<T, X_MID, E>), g, b, 0, st, it, ar); break;
      case X_LAST: hipLaunchKernelGGL((k_line_batched<T, X_LAST, E>), g, b, 0, st, it, ar); break;
      case C_PROP: hipLaunchKernelGGL((k_line_batched<T, C_PROP, E>), g, b, 0, st, it, ar); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

// Batched passes of one plan width (compiled with that width's unit).
template <typename T, int E, int NMAX>
static hipError_t launch_batched_nmax(int kind, const int2* it, const PassArgs* ar, long nitems, hipStream_t st) {
  dim3 g((unsigned)nitems), b(320);
  switch (kind) {
    case X_FIRST: hipLaunchKernelGGL((k_pass_batched<T, X_FIRST, E, NMAX>), g, b, 0, st, it, ar); break;
    case X_MID: hipLaunchKernelGGL((k_pass_batched<T, X_MID, E, NMAX>), g, b, 0, st, it, ar); break;
    case X_LAST: hipLaunchKernelGGL((k_pass_batched<T, X_LAST, E, NMAX>), g, b, 0, st, it, ar); break;
    case C_PROP: hipLaunchKernelGGL((k_pass_batched<T, C_PROP, E, NMAX>), g, b, 0, st, it, ar); break;
    case XA_FIRST: hipLaunchKernelGGL((k_pass_batched<T, XA_FIRST, E, NMAX>), g, b, 0, st, it, ar); break;
    case XA_MID: hipLaunchKernelGGL((k_pass_batched<T, XA_MID, E, NMAX>), g, b, 0, st, it, ar); break;
    case XA_LAST: hipLaunchKernelGGL((k_pass_batched<T, XA_LAST, E, NMAX>), g, b, 0, st, it, ar); break;
    case C_ADJ: hipLaunchKernelGGL((k_pass_batched<T, C_ADJ, E, NMAX>), g, b, 0, st, it, ar); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// nmax: the longest line among the launch's instances
template <typename T, int E>
hipError_t launch_batched_e(int kind, const int2* it, const PassArgs* ar, long nitems, int nmax, hipStream_t st) {
  if constexpr (E == 12 || E == 24) {
    if (nmax > 512) return launch_batched_nmax<T, E, 768>(kind, it, ar, nitems, st);
  }
  if (nmax > 512) return hipErrorInvalidValue;
  return launch_batched_nmax<T, E, 512>(kind, it, ar, nitems, st);
}

}  // namespace sgp
