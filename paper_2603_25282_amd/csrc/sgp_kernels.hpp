// Kernel argument block and launchers shared by the host library and the kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace sgp {

enum { X_FIRST = 0, X_MID = 1, X_LAST = 2, X_NLONLY = 3,
       // y-lines: FFT, exp(-i d (nu_x^2 + nu_y^2)/2) exp(i d Q) / N^d, inverse FFT
       C_PROP = 4,
       // z-lines (3D): FFT, exp(-i d nu_z^2/2), inverse FFT per component
       C_KIN = 5,
       // adjoints: of X_FIRST (iFFT, NL adjoint), of X_MID (iFFT, NL adjoint, FFT),
       // of X_LAST (NL adjoint, FFT), of C_PROP (FFT, P^H and parameter partials, iFFT)
       XA_FIRST = 7, XA_MID = 8, XA_LAST = 9, C_ADJ = 10,
       // rotation mapping (RSDA shears, Sec. 3.1): FFT, phase exp(i nu a w), inverse FFT
       // along x (w = y of the line) or along y (w = x of the column); and bare
       // transforms along x (for the lab-frame Algorithm 1 mode)
       X_SHEAR = 11, C_SHEAR = 12, X_FWD = 13, X_INV = 14 };
enum { NGRAD = 5 };  // adjoint parameter slots: gamma, Omega, c0, c1, c2
// observables passes; OBS_JX / OBS_JY: the x-line and y-column parts of <u, J_z v>
enum { OBS_X = 0, OBS_Y = 1, OBS_Z = 2, OBS_JX = 3, OBS_JY = 4 };
enum { CLOCK_ARG = 0, CLOCK_DEVICE = 1 };
enum { NOBS = 28 };  // partial sums per block of the observables kernels

// One pass over lines of the state ([nz][ny][nx][5] complex).  X kinds use the
// x-line fields, column kinds (C_*) the column fields; both read the tables.
struct PassArgs {
  // x-lines
  long nlines;           // ny * nz (a z-slab launch: ny * its planes)
  int ny;
  int z0;                // first plane of a z-slab launch of an x-pass (trap's z coordinate)
  // columns (lines along y or z)
  long stride;           // element stride along the line (5 nx or 5 nx ny)
  long ncols;            // lines along the contiguous x axis (nx)
  long nouter;           // outer slabs (2D y-lines: 1; 3D y-lines: nz; z-lines: ny)
  long outer_stride;     // elements between outer slabs
  int dim;
  int n_q;               // points along y (the q axis of the propagator)
  const void* tw;        // FFT twiddles of the line's axis
  // propagator
  const void* cs;        // (C - 1, S) per (q, p)
  const void* kin_a;     // exp(-i d nu^2/2) - 1 along x
  const void* kin_l;     // ... along the line
  double nu_scale_a;     // pi / Lx
  double nu_scale_q;     // pi / Ly
  double nu_scale_l;     // pi / L of the line's axis (observables)
  double norm;           // 1 / N^d
  // geometry and physics
  double L[3], h[3];     // half-widths and spacings (unused axes: 0)
  double g2[3];          // squared trap frequencies (gz^2 = 0 in 2D)
  double Omega, gamma;
  double c0, c0p, c1, c2;  // c0, c0 + c2/5, c1, c2
  double d;              // substep duration (nonlinear: the flow time; linear: the clock advance)
  double* clock;         // device clock s of the rotating frame
  double s_arg;          // clock value passed by the host (CLOCK_ARG; then written to *clock)
  double trap_c, trap_s; // cos and sin of Omega s_arg (CLOCK_ARG)
  int clock_mode;
  int advance_clock;
  int kin_conj;          // C_KIN: the conjugate phase (its adjoint)
  // batched passes
  void* state;           // the instance's state
  int n_line;            // length of the pass's lines
  // adjoint support
  void* store;           // forward: where to write the pointwise-stage input (or null)
  const void* fwd;       // adjoint: the stored pointwise-stage input of the forward pass
  double* gacc;          // adjoint: per-line parameter slots [line][NGRAD], accumulated
  // rotation mapping
  double shear;          // shear coefficient a: f(x, y) <- f(x + a y, y) (x) or f(x, y + a x) (y)
  double cphase;         // component phase: psi_l *= exp(i l cphase) when cphase_on
  int cphase_on;
};

// Register plans of the FFT line kernels: E elements per thread of a line of
// length N (the radix sequence follows from N and E, see Plan<N, E>).  E = 8 for
// powers of two and 12 for 3 * 2^k (192, 384, 768) are the defaults; the others are
// autotuning alternatives (E = 4: twice the threads, E = 16 / 24: more registers per
// thread; E = 24 needs more LDS than a CU has in FP64, so it is FP32 only).
// esize: bytes of one real (4 or 8).
constexpr bool plan_ok(int n, int e, int esize) {
  return (n == 192 || n == 384 || n == 768) ? (e == 12 || (e == 24 && esize == 4))
                    : ((n == 16 || n == 32 || n == 64 || n == 128 || n == 256 || n == 512) &&
                       (e == 4 || e == 8 || (e == 16 && n >= 64)));
}
constexpr int default_elems(int n) { return n % 3 == 0 ? 12 : 8; }
constexpr int kPlanElems[] = {4, 8, 12, 16, 24};
// lines per block of the pass kernels for line length n with plan width e
constexpr int lines_per_block(int n, int e) { return n / e >= 64 ? 1 : 64 / (n / e); }
// lines per block of the observables kernels (their LDS tile holds psi and its
// derivative: at most 512 points per block)
constexpr int obs_lines_per_block(int n, int e) {
  int w = lines_per_block(n, e);
  while (w > 1 && w * n > 512) w /= 2;
  return w;
}

// The line kernels (sgp_lines.hpp: five components per thread): points per thread of a
// pass over lines of length n of a 3D grid of npts points, or 0 where the component-split
// kernel of the axis's plan runs.  Measured in step, complex64 unless noted, component-split
// against the line kernel in us (the split one at its default width unless a width is given;
// shapes nx x ny x nz):
//   * small grids have too few lines: 64^3 x 11.9 against 14.9, 128x64x64 17.9 against
//     20.5 (complex128 39.7 against 27.5); 128^3: x 57.7 against 51.0.
//   * y-lines of 64 to 256 points: below 2^21 points the split kernel is as fast or faster
//     (64x64x256 21.6 against 22.5, 768x64x32 28.6 / 30.3, 768x128x16 35.3 / 37.1, 384x256x16
//     35.0 / 37.6), at 2^21 they are equal on average (128^3 42.7 / 43.0, 64x256x128
//     47.0 / 45.5, 512x64x64 36.9 / 39.4, 256x64x128 37.4 / 35.7), above it the line kernel
//     (256x64x256 68.7 / 64.2, 128x128x256 82.8 / 80.2, 256x256x64 89.3 / 85.6, 256^3
//     408 / 395).
//   * powers of two up to 256 run E = 4 (radix 4, 5 wavefronts per SIMD): with E = 8 the
//     x-pass takes 52.9 and the y-pass 47.5 at 128^3 (3 wavefronts per SIMD).  512: E = 8,
//     the widest line that fits a wavefront: x 70.2 against 55.3, y of 64x512x512 441 / 428.
//   * 3 * 2^k: E = 12 (192^3: x 222 against 179, y 217 against 172; y of 128x384x64
//     113 / 83).
//   * z-pass (three transforms' worth of traffic and little arithmetic): the component-split
//     kernel streams faster while the state fits the Infinity Cache (128^3 32.6 / 39.8, 192^3
//     136.5 / 142, 256 points at 2^22 68.7 / 77.3, 512 at 2^22 80.3 / 91.5), the line kernel
//     beyond it, from 2^23 points (192x256x192 205 / 194, 256 points 183 / 165.5, 512 points
//     271 / 206); 64 and 128 points are as fast or faster split there too (256x256x64 53.0 /
//     61.0, 256x256x128 157 / 158, 256x512x128 301 / 304), 384 and 768 on the line kernel
//     everywhere (64x64x384 47.0 / 39.2, 32x64x768 46.9 / 43.2).
//   * complex128: E = 4 (128x128x64: x 48.5 against 39.0, y 62.5 against 43.1); z-lines of
//     64 stay (192x128x64 42.6 / 48.8).  z-lines of 128 and 256 within the cache are faster
//     split with E = 4 (64x128x128 33.6 / 38.1, 64x64x256 35.8 / 37.7) but not at the default
//     width that untuned programs run (whole TS2 step of 64x128x128 126.2 / 123.9, of
//     64x64x128 74.6 / 73.5; z of 64x64x256 51.7 / 37.7), so they run the line kernel, as
//     beyond the cache (256x128x128 157 / 141).  512: E = 8 (32x64x512 50.5 / 39.1);
//     3 * 2^k would need 240 registers of state.
constexpr long line_points_min(int esize) { return esize == 4 ? 1L << 20 : 1L << 19; }
constexpr int line_elems(int kind, int n, int esize, long npts) {
  const bool y = kind == C_PROP, z = kind == C_KIN, p2 = n == 64 || n == 128 || n == 256;
  if (npts < line_points_min(esize) || !(kind == X_FIRST || kind == X_MID || kind == X_LAST || y || z)) return 0;
  if (esize == 8) return p2 ? (z && n == 64 ? 0 : 4) : n == 512 ? 8 : 0;
  if (z) {
    const bool beyond = npts >= 1L << 23;  // a state larger than the Infinity Cache
    return (n == 256 || n == 512) && beyond ? 8 : n == 384 || n == 768 || (n == 192 && beyond) ? 12 : 0;
  }
  if (y && p2 && npts < 1L << 21) return 0;
  return p2 ? 4 : n == 512 ? 8 : (n == 192 || n == 384 || n == 768) ? 12 : 0;
}
// (n, e) pairs with a compiled line kernel
constexpr bool line_ok(int n, int e, int esize) {
  return e == 4 ? (n == 64 || n == 128 || n == 256) : e == 8 ? (n == 512 || (n == 256 && esize == 4))
                : (e == 12 && esize == 4 && (n == 192 || n == 384 || n == 768));
}

// Plans whose line kernels an ensemble partition can run (for every length of that width).
constexpr bool batched_line_plan(int e, int esize) { return e == 4 || (e == 12 && esize == 4); }
// wavefront tiles per block of a line kernel
constexpr int kLineWaves = 4;
constexpr int line_blocks(int n, int e) { return n / (64 / (n / e)) / kLineWaves; }  // of a 2D n x n grid
template <typename T>
hipError_t launch_line_batched(int kind, int e, const void* items, const void* args, long nitems, hipStream_t st);
template <typename T, int E>
hipError_t launch_line_batched_e(int kind, const int2* items, const PassArgs* args, long nitems, hipStream_t st);

// ev: null, or a start / end event pair stamped by the kernel's dispatch
template <typename T>
hipError_t launch_line(int kind, void* psi, const PassArgs& a, int n, int e, hipStream_t st,
                       const hipEvent_t* ev = nullptr);
template <typename T>
hipError_t launch_pass(int kind, void* psi, const PassArgs& a, int n, int e, hipStream_t st,
                       const hipEvent_t* ev = nullptr);
template <typename T>
hipError_t launch_obs(int kind, const void* psi, const PassArgs& a, int n, int e, double* part, hipStream_t st);
// Deterministic sum of block partials: out[q] = sum over b < nb of part[b nq + q],
// q < nq, in a fixed order (one block per q).
hipError_t launch_sum_partials(const double* part, long nb, int nq, double* out, hipStream_t st);
template <typename T>
hipError_t launch_build_tables(void* cs, void* kin_x, void* kin_y, void* kin_z, const int* n, const double* L,
                               int dim, double Omega, double gamma, double d, hipStream_t st);
// Plans the batched ensemble kernels run: the 320-thread geometry (n/e <= 64).
constexpr bool batched_plan_ok(int n, int e, int esize) { return n >= 64 && plan_ok(n, e, esize) && n / e <= 64; }
// batched passes of one plan width e: items = int2 (instance, tile) of instances
// using width e along the pass's axis, args = PassArgs per instance
// nmax: the longest line among the instances of the launch
template <typename T>
hipError_t launch_pass_batched(int kind, int e, const void* items, const void* args, long nitems, int nmax,
                               hipStream_t st);

// per-plan-width launchers, each (T, E) compiled in its own translation unit
template <typename T, int E>
hipError_t launch_pass_e(int kind, void* psi, const PassArgs& a, int n, hipStream_t st, const hipEvent_t* ev);
template <typename T, int E>
hipError_t launch_line_e(int kind, void* psi, const PassArgs& a, int n, hipStream_t st, const hipEvent_t* ev);
template <typename T, int E>
hipError_t launch_obs_e(int kind, const void* psi, const PassArgs& a, int n, double* part, hipStream_t st);

}  // namespace sgp
