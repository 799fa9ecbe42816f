// Split-step kernels for the rotating SOC spin-2 GPE on gfx950.
//
// State layout: [nz][ny][nx][5] complex (components innermost).
//
// One linear substep of the compact splitting (Sec. 3.1) in 2D is two passes over
// the state; each pass reads and writes every value once:
//   X-pass (lines along x): inverse FFT along x, exact nonlinear flow per point
//                           (Sec. 3.2) with the trap at R(Omega s) x, forward FFT.
//   Y-pass (lines along y): forward FFT along y, exact linear propagator per
//                           wavevector (eq. sl1), inverse FFT along y.
// Between passes the state is held x-transformed (Fourier in x, physical in y).
// The first X-pass of a call starts from physical data (no inverse FFT) and the
// last one ends in physical data (no forward FFT).
// 3D adds one pass: the propagator is the product of its part in (nu_p, nu_q) (spin and
// in-plane kinetic) and exp(-i d nu_r^2/2) (Sec. 3.1, 3D: Q does not depend on nu_r), and
// the first acts on each z-plane, the second on each z-line alone.  So the Y-pass applies
// the former and goes back to y at once, and the
//   Z-pass (lines along z): forward FFT along z, z kinetic phase, inverse FFT along z
// needs no transform along y around it: three round trips of the state per substep.
// (Four round trips, with the y transforms in passes of their own around a z-pass,
// measured 0.479 against 0.419 ms per TS4 step at 128^3 and 4.60 against 3.86 at 256^3.)
//
// Work split inside a block: W lines x 5 components; each (line, component) is
// transformed by TL = N/E threads holding E elements each (register Stockham FFT
// with LDS exchanges).  The pointwise stage (nonlinear flow or propagator) needs the
// 5 components of a point together: the block writes its lines into an LDS tile
// (components innermost), every thread updates whole points from the tile, and
// the FFT threads read their elements back.
#pragma once
#include <type_traits>

#include "sgp_device.hpp"
#include "sgp_kernels.hpp"

namespace sgp {

// LDS line stride of the FFT exchanges: N + N/8 (one pad slot per 8) plus a per-length
// extra that spreads the 5 component lines of adjacent lanes over the 32 banks
// (chosen with a bank-conflict model of every exchange pattern; complex values are
// interleaved, one 8- or 16-byte LDS access each).
template <int N> struct PadLine {
  static constexpr int extra = N == 512 ? 13 : N == 256 ? 13 : N == 128 ? 13 : N == 64 ? 5 : N == 384 ? 2
                             : N == 768 ? 13 : N == 192 ? 5 : N == 32 ? 9 : N == 16 ? 1 : 1;
  static constexpr int size = N + N / 8 + extra;
};

// Block index -> logical tile index so that the 8 XCDs (which take blocks round
// robin) each process one contiguous range of tiles and share their L2 lines.
__device__ __forceinline__ long xcd_tile(long b, long nblocks) {
  if (nblocks % 8) return b;
  return (b % 8) * (nblocks / 8) + b / 8;
}

// Trap rotation cos/sin(Omega s): the host's values (first pass of a call, adjoint passes)
// or the device clock's slots 1, 2, which hold cos and sin of the current angle (written
// by whichever pass last moved the clock).
__device__ __forceinline__ void trap_angle(const PassArgs& a, double& c, double& s) {
  const double* src = a.clock_mode == CLOCK_ARG ? nullptr : a.clock;
  c = src ? src[1] : a.trap_c;
  s = src ? src[2] : a.trap_s;
}

// Move the device clock by a.d (one thread).
__device__ __forceinline__ void advance_clock(const PassArgs& a) {
  const double s1 = a.clock[0] + a.d;
  double sn, cn;
  sincos(a.Omega * s1, &sn, &cn);
  a.clock[0] = s1;
  a.clock[1] = cn;
  a.clock[2] = sn;
}

// The trap at R(Omega s) x.
__device__ __forceinline__ double trap_potential(const PassArgs& a, double ct, double st, double x, double y,
                                                 double z) {
  const double X = ct * x + st * y, Y = -st * x + ct * y;
  return 0.5 * (a.g2[0] * X * X + a.g2[1] * Y * Y + a.g2[2] * z * z);
}

// Coefficients of the propagator that a column (kx) shares.
template <typename T>
struct PropCoef {
  T Om, nup, ga, norm, norm_lo;
  double nu_q;
  int n_q;
  __device__ __forceinline__ PropCoef(const PassArgs& a, int kx) {
    const int px = kx < (int)a.ncols / 2 ? kx : kx - (int)a.ncols;
    Om = T(a.Omega);
    ga = T(a.gamma);
    nup = T(px * a.nu_scale_a);
    norm = T(a.norm);
    // 1/N^d as a (hi, lo) pair: exact for powers of two, compensated otherwise
    norm_lo = T(a.norm - (double)norm);
    nu_q = a.nu_scale_q;
    n_q = a.n_q;
  }
};

// The propagator's in-plane part with 1/N^d at (kx, kl) from the table entry (C - 1, S)
// and the kinetic increments along x and y.
template <typename T>
__device__ __forceinline__ void prop_point(const PropCoef<T>& P, int kl, T Cm1, T S, cx<T> ka, cx<T> kl1,
                                           cx<T> (&p)[5]) {
  const int pq = kl < P.n_q / 2 ? kl : kl - P.n_q;
  const T nuq = T(pq * P.nu_q);
  // alpha - 1 = (C - 1) - i S Omega; beta = i S gamma a = S gamma (nu_p - i nu_q)
  const cx<T> as = mk<T>(Cm1, -S * P.Om);
  const cx<T> beta = mk<T>(S * P.ga * P.nup, -S * P.ga * nuq);
  const cx<T> ss = ka + kl1 + ka * kl1;  // kinetic phase - 1
  scale_phase<T>(P.norm, P.norm_lo, ss, p);
  sym4_apply_inc<T>(as, beta, p);
}

// ---------------------------------------------------------------------------
// Generic pass.  KIND selects the line direction and the stages:
//   X_FIRST: load phys -> NL -> FFTx -> store       X_MID: iFFTx -> NL -> FFTx
//   X_LAST:  iFFTx -> NL -> store phys              X_NLONLY: NL only
//   C_PROP:  FFT -> propagator -> iFFT (y column)   C_KIN: FFT -> phase -> iFFT (z column)
// ---------------------------------------------------------------------------
template <int KIND> struct KindInfo {
  static constexpr bool XL = KIND == X_FIRST || KIND == X_MID || KIND == X_LAST || KIND == X_NLONLY ||
                             KIND == XA_FIRST || KIND == XA_MID || KIND == XA_LAST || KIND == X_SHEAR ||
                             KIND == X_FWD || KIND == X_INV;
  static constexpr bool SHEAR = KIND == X_SHEAR || KIND == C_SHEAR;
  static constexpr bool XADJ = KIND == XA_FIRST || KIND == XA_MID || KIND == XA_LAST;
  static constexpr bool ADJ = XADJ || KIND == C_ADJ;
  static constexpr bool PW = (XL && !SHEAR && KIND != X_FWD && KIND != X_INV) || KIND == C_PROP ||
                             KIND == C_ADJ;  // has a pointwise stage (on the LDS tile)
  // which transforms the pass runs (forward: exp(-i..), inverse: exp(+i..))
  static constexpr bool HF = KIND == X_FIRST || KIND == X_MID || KIND == XA_MID || KIND == XA_LAST ||
                             KIND == C_PROP || KIND == C_ADJ || SHEAR || KIND == X_FWD || KIND == C_KIN;
  static constexpr bool HI = KIND == X_MID || KIND == X_LAST || KIND == XA_FIRST || KIND == XA_MID ||
                             KIND == C_PROP || KIND == C_ADJ || SHEAR || KIND == X_INV || KIND == C_KIN;
};

// LDS cx<T> values of the staged twiddle table of a pass.
template <int N, int E, int KIND>
constexpr int pass_tw() {
  return KindInfo<KIND>::HF || KindInfo<KIND>::HI ? 2 * TwSize<N, E>::entries : 0;
}

// LDS elements (per re / im array) a pass needs.
template <int N, int W, int KIND>
constexpr int pass_lds() {
  constexpr int TILE = KindInfo<KIND>::PW ? W * N * 5 : 0;
  constexpr int XCH = W * 5 * PadLine<N>::size;
  return TILE > XCH ? TILE : XCH;
}

// The i-th point of thread tid in a pointwise stage of P points on NT threads.  complex128:
// the last, partial round leaves out the first wavefront; of a block's five wavefronts the
// first shares its SIMD with the fifth and already carries two wavefronts' transforms
// (512^2: 134.1 -> 131.5 us per TS4 step; complex64 81.8 -> 85.1, so not there).
template <typename T, int P, int NT>
__device__ __forceinline__ int pass_point(int i, int tid) {
  if (sizeof(T) == 8 && NT > 64 && P % NT != 0 && P % NT <= NT - 64 && (i + 1) * NT > P && i > 0)
    return i * NT + (tid >= 64 ? tid - 64 : tid + NT - 64);
  return i * NT + tid;
}

// One level of the tree sums over a wavefront of two values at once, in lane exchanges of the
// vector unit.  H = 32: a's sums over lanes l, l + 32 in the lower half and b's in the upper;
// H = 16: a's sums over rows (of 16 lanes) 2 r, 2 r + 1 in row 2 r and b's in row 2 r + 1.
template <int H>
__device__ __forceinline__ double half_sums(double a, double b) {
  uint32_t x[2], y[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t wa = i ? (uint32_t)__double2hiint(a) : (uint32_t)__double2loint(a);
    const uint32_t wb = i ? (uint32_t)__double2hiint(b) : (uint32_t)__double2loint(b);
    // a's upper half (odd rows) and b's lower half (even rows) change places
    const auto r = H == 32 ? __builtin_amdgcn_permlane32_swap(wa, wb, false, false)
                           : __builtin_amdgcn_permlane16_swap(wa, wb, false, false);
    x[i] = r[0];
    y[i] = r[1];
  }
  return __hiloint2double((int)x[1], (int)x[0]) + __hiloint2double((int)y[1], (int)y[0]);
}

// The value of lane l + OFF of the row (of no use in the row's last OFF lanes).
template <int OFF>
__device__ __forceinline__ double row_down(double a) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(a), 0x100 + OFF, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(a), 0x100 + OFF, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Parameter partials of an adjoint pass, one value per line and parameter (NQ parameters),
// summed in an order that depends on the line's length only, so that it is the same for any
// number of lines in a block: every SG consecutive points by a tree (offsets SG/2, ..., 1),
// then the line's SG-point sums one after the other.  The points go to the threads as in a
// forward pass.  (Given to their own line's threads, 5 N/E of them, every wavefront of a block
// had points in the last, partly full round, and the sums took four barriers: a TS2 step of
// the adjoint 988 instead of 910 us for 96 complex64 grids, 375 instead of 307 at 128^3.)  A
// block of whole wavefronts runs the tree in registers, the 64 points of a round being one
// line's, with lane exchanges of the vector unit (through __shfl_down 1012 and 368 us); any
// other block keeps the points' values in LDS.
template <int N, int E, int W, int KIND>
struct GradSum {
  static constexpr int NT = W * 5 * (N / E), WN = W * N;
  static constexpr int Q0 = KindInfo<KIND>::XADJ ? 1 : 0, NQ = KindInfo<KIND>::XADJ ? 4 : 2;  // Q0 .. Q0 + NQ - 1
  static constexpr int SG = N < 64 ? N : 64;
  static constexpr bool WAVES = NT % 64 == 0;
  static constexpr int size = !KindInfo<KIND>::ADJ ? 0 : WAVES ? WN / SG * NQ : NQ * WN;
  static_assert(N % SG == 0 && (!WAVES || WN % 64 == 0), "whole wavefronts of points");

  // the values of point pt (all points of a wavefront at once)
  static __device__ __forceinline__ void add(double* red, int pt, const double (&v)[NQ]) {
    if constexpr (WAVES && SG == 64) {
      // parameters side by side: half a wavefront (two) or a row of 16 lanes (four) each
      double t;
      if constexpr (NQ == 4) t = half_sums<16>(half_sums<32>(v[0], v[2]), half_sums<32>(v[1], v[3]));
      else { t = half_sums<32>(v[0], v[1]); t = half_sums<16>(t, t); }
      t += row_down<8>(t);
      t += row_down<4>(t);
      t += row_down<2>(t);
      t += row_down<1>(t);
      constexpr int LQ = 64 / NQ;
      if (pt % LQ == 0) red[pt / 64 * NQ + pt % 64 / LQ] = t;
    } else if constexpr (WAVES) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        double t = v[q];
#pragma unroll
        for (int off = SG / 2; off > 0; off >>= 1) t += __shfl_down(t, off, SG);
        if (pt % SG == 0) red[pt / SG * NQ + q] = t;
      }
    } else {
#pragma unroll
      for (int q = 0; q < NQ; ++q) red[q * WN + pt] = v[q];
    }
  }

  // between two barriers behind the last add: the tree down to 8 values, in their places
  static __device__ __forceinline__ void fold(double* red, int tid) {
    if constexpr (!WAVES) {
      for (int u = tid; u < NQ * WN / SG * 8; u += NT) {
        double* c = red + u / 8 * SG + u % 8;
        double t[SG / 8];
#pragma unroll
        for (int k = 0; k < SG / 8; ++k) t[k] = c[8 * k];
#pragma unroll
        for (int off = SG / 16; off > 0; off >>= 1)
#pragma unroll
          for (int k = 0; k < off; ++k) t[k] += t[k + off];
        c[0] = t[0];
      }
    }
  }

  // after them: the sum of parameter Q0 + q over line g of the block
  static __device__ __forceinline__ double line(const double* red, int g, int q) {
    double sum = 0.0;
    for (int s = 0; s < N / SG; ++s) {
      if constexpr (WAVES) {
        sum += red[(g * (N / SG) + s) * NQ + q];
      } else {
        const double* c = red + q * WN + g * N + s * SG;
        sum += ((c[0] + c[4]) + (c[2] + c[6])) + ((c[1] + c[5]) + (c[3] + c[7]));
      }
    }
    return sum;
  }
};

// Body of one block of a pass over `tile` (W lines), with caller-provided LDS (red: GradSum's
// values, adjoint passes only).
template <typename T, int N, int E, int W, int KIND>
__device__ __forceinline__ void pass_body(cx<T>* __restrict__ psi, const PassArgs& a, long tile, cx<T>* lx,
                                          cx<T>* ltw, [[maybe_unused]] double* red) {
  constexpr int TL = N / E;
  constexpr int NT = W * 5 * TL;
  using GS = GradSum<N, E, W, KIND>;
  constexpr int LS = PadLine<N>::size;
  constexpr bool XL = KindInfo<KIND>::XL;
  constexpr bool XADJ = KindInfo<KIND>::XADJ;
  constexpr bool ADJ = KindInfo<KIND>::ADJ;
  constexpr bool PW = KindInfo<KIND>::PW;

  const int tid = threadIdx.x;
  const int c = tid % 5;
  const int rest = tid / 5;
  // x-lines: the TL threads of a line are adjacent (contiguous loads);
  // columns: the W columns are adjacent (W*5 contiguous values per row)
  const int col = XL ? rest / TL : rest % W;
  const int t = XL ? rest % TL : rest / W;

  // Line geometry: the tile's first value (uniform, in scalar registers), the thread's byte
  // offset from it and the element stride of the line.  The offset is 32 bits wide where a
  // line's TL threads span less than 2^32 bytes (TL <= 64; every supported state has fewer
  // than 2^31 elements).
  using Off = std::conditional_t<TL <= 64, uint32_t, uint64_t>;
  const int estride = XL ? 5 : (int)a.stride;
  int line0 = 0;    // x-lines: first line of the block (line = z * ny + y)
  int o = 0, kx0 = 0;
  cx<T>* tb;
  bool active;
  // every supported length is a multiple of 16, so only wider tiles have idle lines
  constexpr bool FULL = W <= 16;
  if constexpr (XL) {
    line0 = (int)tile * W;
    active = FULL || line0 + col < a.nlines;
    tb = psi + (long)line0 * N * 5;
  } else {
    const int ncolblk = ((int)a.ncols + W - 1) / W;
    o = (int)tile / ncolblk;
    kx0 = ((int)tile % ncolblk) * W;
    active = FULL || kx0 + col < a.ncols;
    tb = psi + (long)o * a.outer_stride + kx0 * 5;
  }
  const Off voff = active ? ((Off)(XL ? col * N * 5 : col * 5) + (Off)t * (Off)estride + c) * (Off)sizeof(cx<T>) : 0;

  constexpr int TW = pass_tw<N, E, KIND>();
  TwStage<T, NT, (TW > 0 ? TW : 2)> stage;
  // table first, so that the barrier behind it passes while the state is in flight; 512
  // complex64 points measured the other way round (x-pass 14.3 against 13.9 us)
  constexpr bool TWFIRST = sizeof(T) == 8 || E == 12;
  if constexpr (TW > 0 && TWFIRST) stage.load(a.tw, tid);
  cx<T> v[1][E];
#pragma unroll
  for (int m = 0; m < E; ++m)
    v[0][m] = active ? *reinterpret_cast<const cx<T>*>(reinterpret_cast<const char*>(tb + (long)(TL * m) * estride) + voff)
                     : mk<T>(T(0), T(0));

  cx<T>* xl = lx + (col * 5 + c) * LS;
  const cx<T>* tw = ltw;
  if constexpr (TW > 0 && !TWFIRST) stage.load(a.tw, tid);
  if constexpr (TW > 0) stage.store(ltw, a.tw, tid);

  // read here, with the state loads: at its place of use, behind the transform and its
  // barriers, the clock is a round trip to memory of its own in every block
  double ct = 1.0, st = 0.0;
  if constexpr (XL && PW) trap_angle(a, ct, st);

  // propagator tables of this thread's points.  With one line per block (few blocks, all
  // of them in the same phase) they are loaded here, under the state loads; with more
  // lines per block other wavefronts cover the loads at their place of use, and the
  // registers are worth more.
  constexpr int PP = (E + 4) / 5;  // points per thread
  constexpr bool PRE = !XL && PW && W == 1;
  [[maybe_unused]] constexpr int UN = PRE ? PP : 1;
  T pcs[PRE ? PP : 1][2];
  cx<T> pkl[PRE ? PP : 1];
  cx<T> pka = mk<T>(T(0), T(0));
  if constexpr (PRE) {
    const T* cs = reinterpret_cast<const T*>(a.cs) + 2 * (size_t)(kx0 * a.n_q);
    const cx<T>* kl = reinterpret_cast<const cx<T>*>(a.kin_l);
    pka = reinterpret_cast<const cx<T>*>(a.kin_a)[kx0];
#pragma unroll
    for (int i = 0; i < PP; ++i) {
      const int p = pass_point<T, W * N, NT>(i, tid);
      const int pt = p < N ? p : 0;
      pcs[i][0] = cs[2 * pt];
      pcs[i][1] = cs[2 * pt + 1];
      pkl[i] = kl[pt];
    }
  }

  if constexpr (KIND == X_MID || KIND == X_LAST || KIND == XA_FIRST || KIND == XA_MID || KIND == X_INV) {
    __syncthreads();  // the table
    fft_line<T, N, E, +1, 1, 1, 0>(v, xl, t, tw, 0);
  }
  if constexpr (KIND == C_PROP || KIND == C_ADJ || KIND == X_FWD || KindInfo<KIND>::SHEAR || KIND == C_KIN)
    fft_line<T, N, E, -1, 1, 1, 0>(v, xl, t, tw, 0);

  if constexpr (KIND == C_KIN) {
    // the kinetic phase along the line, per component: coefficient k times
    // exp(-i d nu_k^2/2), in increment form (table entry exp(..) - 1)
    const cx<T>* kin_l = reinterpret_cast<const cx<T>*>(a.kin_l);
    const T sg = a.kin_conj ? T(-1) : T(1);
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const cx<T> ph = kin_l[t + TL * m];
      v[0][m] = inc_apply(mk<T>(ph.re, sg * ph.im), v[0][m]);
    }
    fft_line<T, N, E, +1, 1, 1, 0>(v, xl, t, tw, 0);
  }

  if constexpr (KindInfo<KIND>::SHEAR) {
    // f(.. + a w ..) along the line: coefficient k times exp(i nu_k a w) / N, w the
    // line's coordinate on the other in-plane axis; FP64 phase
    double w;
    if constexpr (XL) {
      const int line = (int)line0 + col;
      const int iy = a.dim == 3 ? line - (line / a.ny) * a.ny : line;
      w = -a.L[1] + iy * a.h[1];
    } else {
      w = -a.L[0] + (kx0 + col) * a.h[0];
    }
    const double nus = XL ? a.nu_scale_a : a.nu_scale_l;
    double cr = 1.0, ci = 0.0;
    if (a.cphase_on) sincos((2 - c) * a.cphase, &ci, &cr);
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int k = t + TL * m;
      const int p = k < N / 2 ? k : k - N;
      double sn, cs;
      sincos(p * nus * a.shear * w, &sn, &cs);
      const double zr = (cs * cr - sn * ci) / N, zi = (cs * ci + sn * cr) / N;
      const T vr = v[0][m].re, vi = v[0][m].im;
      v[0][m] = mk<T>(T(zr) * vr - T(zi) * vi, T(zr) * vi + T(zi) * vr);
    }
    fft_line<T, N, E, +1, 1, 1, 0>(v, xl, t, tw, 0);
  }

  // forward store mode: keep the pointwise-stage input for the adjoint
  if constexpr (PW && !ADJ) {
    if (a.store != nullptr && active) {
      cx<T>* st = reinterpret_cast<cx<T>*>(a.store) + (tb - psi);
      const Off so = pin(voff);
#pragma unroll
      for (int m = 0; m < E; ++m)
        *reinterpret_cast<cx<T>*>(reinterpret_cast<char*>(st + (long)(TL * m) * estride) + so) = v[0][m];
    }
  }

  if constexpr (PW) {
    // to the tile: point (col, j) component c at (col * N + j) * 5 + c
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int o5 = (col * N + t + TL * m) * 5 + c;
      lx[o5] = v[0][m];
    }
    __syncthreads();
    if constexpr (XL) {
      NLCoef K;
      K.d = a.d;
      K.c0p = a.c0p;
      K.c1 = a.c1;
      K.c2 = a.c2;
      // (y, z) indices of the block's first line (uniform); the block's W lines follow it
      // (z from the launch's first plane a.z0 on)
      const int izl = a.dim == 3 ? line0 / a.ny : 0;
      const int iy0 = line0 - izl * a.ny;
      const int iz0 = izl + a.z0;
      auto point = [&](int i) { return pass_point<T, W * N, NT>(i, tid); };
      for (int i = 0, pt = point(0); pt < W * N; pt = point(++i)) {
        const int pc = pt / N, j = pt % N;
        const int line = (int)line0 + pc;  // y + ny z (< 2^31 for every supported grid)
        int iy = iy0 + pc, iz = iz0;
        while (iy >= a.ny) {
          iy -= a.ny;
          iz += 1;
        }
        const double x = -a.L[0] + j * a.h[0];
        const double y = -a.L[1] + iy * a.h[1];
        const double z = -a.L[2] + iz * a.h[2];
        const double V = trap_potential(a, ct, st, x, y, z);
        cx<T> p[5];
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) p[cc] = lx[pt * 5 + cc];
        if constexpr (XADJ) {
          // forward input of this nonlinear substep at the point, from the store
          const cx<T>* fw = reinterpret_cast<const cx<T>*>(a.fwd) + (line < a.nlines ? line : 0) * N * 5 + j * 5;
          cx<T> q[5];
#pragma unroll
          for (int cc = 0; cc < 5; ++cc) q[cc] = fw[cc];
          // dV/dOmega = s (gx^2 - gy^2) X Y (trap at R(Omega s) x)
          const double X = ct * x + st * y, Y = -st * x + ct * y;
          const double dVdO = a.s_arg * (a.g2[0] - a.g2[1]) * X * Y;
          double acc4[4] = {0.0, 0.0, 0.0, 0.0};
          nl_point_adj<T>(q, p, V, dVdO, K, acc4);
          if constexpr (!FULL)
            if (line >= a.nlines) acc4[0] = acc4[1] = acc4[2] = acc4[3] = 0.0;
          GS::add(red, pt, acc4);
        } else {
          nl_point<T>(p, V, K);
        }
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) lx[pt * 5 + cc] = p[cc];
      }
    } else {
      const T* cs = reinterpret_cast<const T*>(a.cs);
      const cx<T>* kin_a = reinterpret_cast<const cx<T>*>(a.kin_a);
      const cx<T>* kin_l = reinterpret_cast<const cx<T>*>(a.kin_l);
      const T Om = T(a.Omega), ga = T(a.gamma), norm = T(a.norm);
      // 1/N^d as a (hi, lo) pair: exact for powers of two, compensated otherwise
      const T norm_lo = T(a.norm - (double)norm);
      const int nxx = (int)a.ncols;
#pragma unroll UN
      for (int i = 0; i < PP; ++i) {
        const int pt = pass_point<T, W * N, NT>(i, tid);
        if (pt >= W * N) break;
        const int pc = pt / N, kl = pt % N;
        const int kx = kx0 + pc < nxx ? kx0 + pc : 0;
        const int px = kx < nxx / 2 ? kx : kx - nxx;
        const T nup = T(px * a.nu_scale_a);
        // table kx-major: a column block reads its entries contiguously
        cx<T> ka, kl1;
        T Cm1, S;
        if constexpr (PRE) {
          ka = pka;
          kl1 = pkl[i];
          Cm1 = pcs[i][0];
          S = pcs[i][1];
        } else {
          const int qidx = kx * a.n_q + kl;
          ka = kin_a[kx];
          kl1 = kin_l[kl];
          Cm1 = cs[2 * qidx];
          S = cs[2 * qidx + 1];
        }
        const int pq = kl < a.n_q / 2 ? kl : kl - a.n_q;
        const T nuq = T(pq * a.nu_scale_q);
        // alpha - 1 = (C - 1) - i S Omega; beta = i S gamma a = S gamma (nu_p - i nu_q)
        const cx<T> as = mk<T>(Cm1, -S * Om);
        const cx<T> beta = mk<T>(S * ga * nup, -S * ga * nuq);
        const cx<T> ss = ka + kl1 + ka * kl1;  // kinetic phase - 1
        cx<T> p[5];
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) p[cc] = lx[pt * 5 + cc];
        scale_phase<T>(norm, norm_lo, KIND == C_ADJ ? conj(ss) : ss, p);
        if constexpr (KIND == C_ADJ) {
          // P^H = P(-d): same (C - 1), S -> -S, conjugate kinetic phase
          sym4_apply_inc<T>(conj(as), mk<T>(-beta.re, -beta.im), p);
          double acc2[2] = {0.0, 0.0};
          if (FULL || kx0 + pc < a.ncols) {
            // m_a = -d Im(L^H f_a H), L = P^H L'/N^d (p), H the stored forward input
            const cx<T>* fw = reinterpret_cast<const cx<T>*>(a.fwd) + o * (int)a.outer_stride + kx * 5 + kl * (int)a.stride;
            const double w4[4] = {1.0, 1.22474487139158904909864203735294570, 1.22474487139158904909864203735294570, 1.0};
            double upr = 0, upi = 0, umr = 0, umi = 0, uzi = 0;
            cx<T> hq[5];
#pragma unroll
            for (int cc = 0; cc < 5; ++cc) hq[cc] = fw[cc];
#pragma unroll
            for (int l = 0; l < 4; ++l) {
              const cx<T> a1 = cmulc(p[l], hq[l + 1]), a2 = cmulc(p[l + 1], hq[l]);
              upr += 2.0 * w4[l] * a1.re; upi += 2.0 * w4[l] * a1.im;
              umr += 2.0 * w4[l] * a2.re; umi += 2.0 * w4[l] * a2.im;
            }
#pragma unroll
            for (int l = 0; l < 5; ++l) uzi += (2 - l) * (double)cmulc(p[l], hq[l]).im;
            const double dd = a.d;
            const double mx = -dd * 0.5 * (upi + umi);
            const double my = dd * 0.5 * (upr - umr);
            const double mz = -dd * uzi;
            // dJ/dn = J_r(-d n)^T m, n = (gamma Re a, -gamma Im a, -Omega), a = -nu_q - i nu_p
            const double nupd = px * a.nu_scale_a, nuqd = pq * a.nu_scale_q;
            const double ox = -dd * a.gamma * (-nuqd), oy = -dd * (-a.gamma) * (-nupd), oz = -dd * (-a.Omega);
            const double th2 = ox * ox + oy * oy + oz * oz;
            double ja, jb;
            if (th2 < 1e-8) { ja = 0.5 - th2 / 24.0; jb = 1.0 / 6.0 - th2 / 120.0; }
            else {
              const double th = sqrt(th2), hs = sin(0.5 * th);
              ja = 2.0 * hs * hs / th2;
              jb = (th - sin(th)) / (th2 * th);
            }
            const double cx1 = oy * mz - oz * my, cy1 = oz * mx - ox * mz, cz1 = ox * my - oy * mx;
            const double cx2 = oy * cz1 - oz * cy1, cy2 = oz * cx1 - ox * cz1, cz2 = ox * cy1 - oy * cx1;
            const double Dx = mx + ja * cx1 + jb * cx2, Dy = my + ja * cy1 + jb * cy2, Dz = mz + ja * cz1 + jb * cz2;
            acc2[0] = -nuqd * Dx + nupd * Dy;  // dn/dgamma = (Re a, -Im a, 0) = (-nu_q, nu_p, 0)
            acc2[1] = -Dz;                     // dn/dOmega = (0, 0, -1)
          }
          GS::add(red, pt, acc2);
        } else {
          sym4_apply_inc<T>(as, beta, p);
        }
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) lx[pt * 5 + cc] = p[cc];
      }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int o5 = (col * N + t + TL * m) * 5 + c;
      v[0][m] = lx[o5];
    }
    if constexpr (ADJ) GS::fold(red, tid);
    __syncthreads();
  }
  if constexpr (ADJ) {
    for (int u = tid; u < W * GS::NQ; u += NT) {
      const int g = u / GS::NQ, q = u % GS::NQ;
      const long slot = XL ? (long)line0 + g : (long)o * a.ncols + kx0 + g;
      if (FULL || (XL ? line0 + g < a.nlines : kx0 + g < a.ncols)) a.gacc[slot * NGRAD + GS::Q0 + q] += GS::line(red, g, q);
    }
  }

  if constexpr (KIND == X_FIRST || KIND == X_MID || KIND == XA_MID || KIND == XA_LAST)
    fft_line<T, N, E, -1, 1, 1, 0>(v, xl, t, tw, 0);
  if constexpr (KIND == C_PROP || KIND == C_ADJ) fft_line<T, N, E, +1, 1, 1, 0>(v, xl, t, tw, 0);

  if (active) {
    // made opaque: else the addresses of the loads stay in registers (two per value)
    const Off so = pin(voff);
#pragma unroll
    for (int m = 0; m < E; ++m)
      *reinterpret_cast<cx<T>*>(reinterpret_cast<char*>(tb + (long)(TL * m) * estride) + so) = v[0][m];
  }
  if constexpr (XL && !ADJ && PW) {
    if (a.clock_mode == CLOCK_ARG && tile == 0 && tid == 0) {
      a.clock[0] = a.s_arg;
      a.clock[1] = ct;
      a.clock[2] = st;
    }
  }
}

// The device clock's advance runs in a block of its own, after the tiles' blocks (see
// pass_blocks): in a tile's block its load and sine ended every pass of a small grid
// ~2 us after the other blocks.
template <typename T, int N, int E, int W, int KIND>
__global__ __launch_bounds__(W * 5 * (N / E)) void k_pass(cx<T>* __restrict__ psi, PassArgs a) {
  constexpr int BUF = pass_lds<N, W, KIND>();
  constexpr int NT = W * 5 * (N / E);
  constexpr int TWB = (pass_tw<N, E, KIND>() * (int)sizeof(cx<T>) + 15) / 16;
  constexpr int RED = GradSum<N, E, W, KIND>::size;
  __shared__ cx<T> lx[BUF];
  __shared__ uint4 ltw[TWB > 0 ? TWB : 1];
  __shared__ double red[RED > 0 ? RED : 1];
  long nb = gridDim.x;
  if constexpr (KIND == C_PROP || KIND == C_KIN) {
    if (a.advance_clock) {
      nb -= 1;
      if (blockIdx.x == nb) {
        if (threadIdx.x == 0) advance_clock(a);
        return;
      }
    }
  }
  pass_body<T, N, E, W, KIND>(psi, a, xcd_tile(blockIdx.x, nb), lx, reinterpret_cast<cx<T>*>(ltw), red);
}

// ---------------------------------------------------------------------------
// Batched pass over many grids (an ensemble): block b processes work item
// items[b] = (instance, tile) with that instance's arguments.  One kernel per plan
// width E; every line length it serves runs with 320 threads per block (W = 64 E / N
// lines), the geometry of the single-grid kernel of the same plan, so an instance
// gives bitwise the same result alone or inside an ensemble.
// ---------------------------------------------------------------------------
template <int N, int E, int KIND, int ES>
constexpr int batched_lds() {
  if constexpr (batched_plan_ok(N, E, ES)) return pass_lds<N, lines_per_block(N, E), KIND>();
  else return 0;
}
template <int N, int E, int KIND, int ES>
constexpr int batched_tw() {
  if constexpr (batched_plan_ok(N, E, ES)) return pass_tw<N, E, KIND>();
  else return 0;
}
constexpr int cmax(int a, int b) { return a > b ? a : b; }

// NMAX: the longest line the kernel serves (512, or 768 for the E = 12 / 24 plans);
// its static LDS is sized for lines up to NMAX only, so instances of the common
// sizes keep the occupancy they have without 768-point lines in the ensemble.
template <typename T, int KIND, int E, int NMAX>
__global__ __launch_bounds__(320) void k_pass_batched(const int2* __restrict__ items, const PassArgs* __restrict__ args) {
  constexpr int ES = (int)sizeof(T);
  constexpr int BUF = cmax(cmax(cmax(cmax(batched_lds<64, E, KIND, ES>(), batched_lds<128, E, KIND, ES>()),
                                     cmax(batched_lds<256, E, KIND, ES>(), batched_lds<384, E, KIND, ES>())),
                                cmax(batched_lds<512, E, KIND, ES>(), batched_lds<192, E, KIND, ES>())),
                           NMAX >= 768 ? batched_lds<768, E, KIND, ES>() : 0);
  constexpr int TWM = cmax(cmax(cmax(cmax(batched_tw<64, E, KIND, ES>(), batched_tw<128, E, KIND, ES>()),
                                     cmax(batched_tw<256, E, KIND, ES>(), batched_tw<384, E, KIND, ES>())),
                                cmax(batched_tw<512, E, KIND, ES>(), batched_tw<192, E, KIND, ES>())),
                           NMAX >= 768 ? batched_tw<768, E, KIND, ES>() : 0);
  constexpr int TWB = (TWM * (int)sizeof(cx<T>) + 15) / 16;
  __shared__ cx<T> lx[BUF > 0 ? BUF : 1];
  __shared__ uint4 ltwr[TWB > 0 ? TWB : 1];
  // a block's 64 E points (320 threads), in 64-point sums of at most four parameters
  __shared__ double red[KindInfo<KIND>::ADJ ? 4 * E : 1];
  cx<T>* ltw = reinterpret_cast<cx<T>*>(ltwr);
  const int2 it = items[blockIdx.x];
  const PassArgs& a = args[it.x];
  if constexpr (KIND == C_PROP) {
    if (a.advance_clock && it.y == 0 && threadIdx.x == 319) advance_clock(a);
  }
  cx<T>* psi = reinterpret_cast<cx<T>*>(a.state);
#define SGP_BCASE(NN)                                                                                  \
  case NN:                                                                                             \
    if constexpr (NN <= NMAX && batched_plan_ok(NN, E, ES)) {                                          \
      static_assert(GradSum<NN, E, lines_per_block(NN, E), KIND>::size <= 4 * E, "the sums fit");      \
      pass_body<T, NN, E, lines_per_block(NN, E), KIND>(psi, a, it.y, lx, ltw, red);                   \
    }                                                                                                  \
    break;
  switch (a.n_line) {
    SGP_BCASE(64) SGP_BCASE(128) SGP_BCASE(192) SGP_BCASE(256) SGP_BCASE(384) SGP_BCASE(512) SGP_BCASE(768)
    default: break;
  }
#undef SGP_BCASE
}

// ---------------------------------------------------------------------------
// Propagator table, FP64: Q = n.f with n = (gamma Re a, -gamma Im a, -Omega), so
// exp(i d Q) is the spin-2 image of exp(i d n.sigma/2) = C + i S n.sigma with
// C = cos(lam d/2), S = sin(lam d/2)/lam, lam = |n| = sqrt(Omega^2 + gamma^2
// (nu_p^2 + nu_q^2)).  Stored per (p, q), rounded to T: (C - 1, S), with
// C - 1 = -2 sin^2(lam d/4), at entry kx * ny + ky (kx-major, the order the
// last-axis pass reads it in).  Kinetic tables per axis: exp(-i d nu^2/2) - 1.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_build_cs(T* __restrict__ cs, int nx, int ny, double Lx, double Ly, double Omega, double gamma,
                           double d) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)nx * ny) return;
  const int kx = (int)(i / ny), ky = (int)(i % ny);
  const int p = kx < nx / 2 ? kx : kx - nx;
  const int q = ky < ny / 2 ? ky : ky - ny;
  const double pi = 3.14159265358979323846264338327950288;
  const double nup = pi * p / Lx, nuq = pi * q / Ly;
  const double lam = sqrt(Omega * Omega + gamma * gamma * (nup * nup + nuq * nuq));
  double Cm1, S;
  if (lam == 0.0) {
    Cm1 = 0.0;
    S = 0.5 * d;
  } else {
    const double s4 = sin(0.25 * lam * d);
    Cm1 = -2.0 * s4 * s4;
    S = sin(0.5 * lam * d) / lam;
  }
  cs[2 * i] = (T)Cm1;
  cs[2 * i + 1] = (T)S;
}

template <typename T>
__global__ void k_build_kin(cx<T>* __restrict__ kin, int n, double L, double d) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int p = k < n / 2 ? k : k - n;
  const double nu = 3.14159265358979323846264338327950288 * p / L;
  const double ph = -0.5 * d * nu * nu;
  const double sh = sin(0.5 * ph);
  kin[k].re = (T)(-2.0 * sh * sh);
  kin[k].im = (T)sin(ph);
}

}  // namespace sgp
