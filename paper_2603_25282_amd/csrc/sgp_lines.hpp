// Passes with all five components of a point in one thread ("line" kernels), for grids
// with many lines.
//
// A line of N points is owned by TL = N/E <= 64 threads of ONE wavefront (64/TL lines per
// wavefront); a thread holds E points with their five components in registers.  Against
// the component-split passes of sgp_passes.hpp (one component per thread):
//   * the pointwise stage works on the registers (no LDS tile and its two exchanges, and
//     every thread has the same number of points);
//   * twiddles, addresses and the line's coordinates serve five components;
//   * a wavefront's LDS operations execute in order, so the exchanges need no barrier.
// That is ~25 % fewer vector instructions per point, which is what bounds a pass over a
// large grid.  It needs 5 times fewer, 5 times longer wavefronts, so grids with few lines
// (a single 2D grid) keep the component-split passes (line_elems).
#pragma once
#include "sgp_passes.hpp"

namespace sgp {

// kLineWaves wavefronts per block (they share the staged twiddles): four.  Two: x 54.0
// instead of 51.0 us at 128^3; eight: 58.8.

// Wavefronts per SIMD to keep room for: 80 registers of state come out at 150 to 175 in
// all, and above 168 (two wavefronts) the 192x128x64 complex128 y-pass takes 70 instead of
// 58 us, the 256^3 complex64 z-pass 361 instead of 318.  (Four, 128 registers, spill.)
constexpr int line_min_waves(int e, int esize) { return e * (esize / 4) == 8 ? 3 : 1; }

// LDS of a wavefront: its 64/TL lines' exchanges, one component at a time, or 64 points
// between memory order and point order.
template <int N, int E>
constexpr int line_lds() { return cmax(64 / (N / E) * PadLine<N>::size, 64 * 5); }

// Slice m of a wavefront's values (64 points of five components, one point per thread)
// between memory order (value i * 64 + lane) and point order (component c of point lane),
// through LDS: a thread's point is 40 or 80 bytes, and reading and writing it in place
// touches three times the cache lines per instruction (128^3 complex64: y-pass 55 instead
// of 44 us, z-pass 47 instead of 38; 128x128x64 complex128: x-pass 58 instead of 44).
template <typename T, int E, bool IN>
__device__ __forceinline__ void line_reorder(const cx<T> (&v)[5][E], int m, cx<T>* lx, int lane, cx<T> (&r)[5]) {
  lds_sync<1>();
#pragma unroll
  for (int i = 0; i < 5; ++i) lx[IN ? i * 64 + lane : lane * 5 + i] = v[i][m];
  lds_sync<1>();
#pragma unroll
  for (int i = 0; i < 5; ++i) r[i] = lx[IN ? lane * 5 + i : i * 64 + lane];
}

// The values v to memory at dst (the state or a forward store), in memory order.
template <typename T, int E>
__device__ __forceinline__ void line_store(const cx<T> (&v)[5][E], cx<T>* dst, long step, const uint32_t (&off)[5],
                                           cx<T>* lx, int lane) {
  // the offsets are made opaque here: seen through, they become 64-bit addresses of every
  // value that live through the pointwise stage (2 * 5 * E registers)
  uint32_t o[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) o[i] = pin(off[i]);
#pragma unroll
  for (int m = 0; m < E; ++m) {
    cx<T> r[5];
    line_reorder<T, E, false>(v, m, lx, lane, r);
    char* d = reinterpret_cast<char*>(dst + m * step);
#pragma unroll
    for (int i = 0; i < 5; ++i) *reinterpret_cast<cx<T>*>(d + o[i]) = r[i];
  }
}

// One wavefront's tile of a line pass: 64/TL lines; xch: the wavefront's LDS, ltw: the
// block's table.
template <typename T, int N, int E, int KIND>
__device__ __forceinline__ void line_body(cx<T>* __restrict__ psi, const PassArgs& a, int tile, cx<T>* xch,
                                          cx<T>* ltw) {
  constexpr int TL = N / E;
  constexpr int W = 64 / TL;  // lines per wavefront
  constexpr int LS = PadLine<N>::size;
  constexpr bool XL = KindInfo<KIND>::XL;
  constexpr int TW = pass_tw<N, E, KIND>();
  const int lane = threadIdx.x & 63;
  // x-lines: the threads of a line are adjacent; columns: the W columns are
  const int col = XL ? lane / TL : lane % W;
  const int t = XL ? lane % TL : lane / W;
  // the lines of a launch are a multiple of W, its wavefronts may not fill the last block
  const int ncolblk = XL ? 1 : (int)a.ncols / W;
  const bool active = tile < (XL ? (int)a.nlines / W : ncolblk * (int)a.nouter);
  const int tl = active ? tile : 0;
  const int o = XL ? 0 : tl / ncolblk;
  const int kx = XL ? 0 : (tl - o * ncolblk) * W + col;
  const int line = XL ? tl * W + col : 0;
  // Memory order of the 64 points m of the wavefront's threads (one per thread): rows of RL
  // consecutive values (columns: W points of one row; x-lines: TL points of one line),
  // `pitch` values apart, `step` values from one m to the next.
  constexpr int RL = XL ? 5 * TL : 5 * W;
  const long pitch = XL ? 5 * N : a.stride;
  const long step = XL ? 5 * TL : TL * a.stride;
  const long start = XL ? (long)tl * W * N * 5 : (long)o * a.outer_stride + (long)(tl - o * ncolblk) * W * 5;
  uint32_t off[5];  // byte offsets of the thread's five values of a slice (below 2^32: TL <= 64)
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int e = i * 64 + lane;
    off[i] = (uint32_t)(((long)(e / RL) * pitch + e % RL) * (int)sizeof(cx<T>));
  }
  cx<T>* lx0 = xch;
  TwStage<T, 64 * kLineWaves, TW> stage;
  stage.load(a.tw, threadIdx.x);
  cx<T> v[5][E];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    const char* src = reinterpret_cast<const char*>(psi + start + m * step);
#pragma unroll
    for (int i = 0; i < 5; ++i) v[i][m] = *reinterpret_cast<const cx<T>*>(src + off[i]);
  }
  stage.store(ltw, a.tw, threadIdx.x);
  const cx<T>* tw = ltw;
  double ct = 1.0, st = 0.0;
  if constexpr (XL) trap_angle(a, ct, st);
  __syncthreads();
  if (!active) return;

#pragma unroll
  for (int m = 0; m < E; ++m) {
    cx<T> r[5];
    line_reorder<T, E, true>(v, m, lx0, lane, r);
#pragma unroll
    for (int c = 0; c < 5; ++c) v[c][m] = r[c];
  }
  cx<T>* lx = lx0 + col * LS;
  if constexpr (KIND == X_MID || KIND == X_LAST) fft_line<T, N, E, +1, 5, 1, 1>(v, lx, t, tw, 0);
  if constexpr (!XL) fft_line<T, N, E, -1, 5, 1, 1>(v, lx, t, tw, 0);

  if constexpr (KIND != C_KIN) {
    // forward store mode: the pointwise-stage input in the state's layout, as the state's
    // own stores.  Point by point, 8 or 16 bytes a lane 40 or 80 apart, a stored TS2 step took
    // 104 instead of 90 us at 128 x 512 x 16 complex64, 177 instead of 154 at 64 x 128 x 128
    // complex128.
    if (a.store != nullptr)
      line_store<T, E>(v, reinterpret_cast<cx<T>*>(a.store) + start, step, off, lx0, lane);
  }

  if constexpr (XL) {
    NLCoef K;
    K.d = a.d;
    K.c0p = a.c0p;
    K.c1 = a.c1;
    K.c2 = a.c2;
    const int izl = a.dim == 3 ? line / a.ny : 0;
    const double y = -a.L[1] + (line - izl * a.ny) * a.h[1];
    const double z = -a.L[2] + (izl + a.z0) * a.h[2];
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const double x = -a.L[0] + (t + TL * m) * a.h[0];
      const double V = trap_potential(a, ct, st, x, y, z);
      cx<T> p[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) p[c] = v[c][m];
      nl_point<T>(p, V, K);
      // pinned: else the compiler sinks the maps of all E points past each other's branches
      // to the transform behind them and holds their coefficients in 100 more registers
#pragma unroll
      for (int c = 0; c < 5; ++c) v[c][m] = pin(p[c]);
    }
  } else if constexpr (KIND == C_PROP) {
    // table entries one point ahead of their use
    const cx<T>* cs = reinterpret_cast<const cx<T>*>(a.cs);
    const cx<T>* kin_l = reinterpret_cast<const cx<T>*>(a.kin_l);
    const cx<T> ka = reinterpret_cast<const cx<T>*>(a.kin_a)[kx];
    const PropCoef<T> P(a, kx);
    cx<T> e = cs[(uint32_t)(kx * a.n_q + t)], k1 = kin_l[(uint32_t)t];
#pragma unroll
    for (int m = 0; m < E; ++m) {
      cx<T> en = e, kn = k1;
      if (m + 1 < E) {
        const uint32_t kl = pin((uint32_t)(t + TL * (m + 1)));
        en = cs[(uint32_t)(kx * a.n_q) + kl];
        kn = kin_l[kl];
      }
      cx<T> p[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) p[c] = v[c][m];
      prop_point<T>(P, t + TL * m, e.re, e.im, ka, k1, p);
#pragma unroll
      for (int c = 0; c < 5; ++c) v[c][m] = pin(p[c]);
      e = en;
      k1 = kn;
    }
  } else {
    const cx<T>* kin_l = reinterpret_cast<const cx<T>*>(a.kin_l);
    const T sg = a.kin_conj ? T(-1) : T(1);
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const cx<T> k1 = kin_l[t + TL * m];
      const cx<T> ph = mk<T>(k1.re, sg * k1.im);
#pragma unroll
      for (int c = 0; c < 5; ++c) v[c][m] = inc_apply(ph, v[c][m]);
    }
  }

  if constexpr (KIND == X_FIRST || KIND == X_MID) fft_line<T, N, E, -1, 5, 1, 1>(v, lx, t, tw, 0);
  if constexpr (!XL) fft_line<T, N, E, +1, 5, 1, 1>(v, lx, t, tw, 0);

  line_store<T, E>(v, psi + start, step, off, lx0, lane);
  if constexpr (XL) {
    if (a.clock_mode == CLOCK_ARG && tile == 0 && lane == 0) {
      a.clock[0] = a.s_arg;
      a.clock[1] = ct;
      a.clock[2] = st;
    }
  }
}

template <typename T, int N, int E, int KIND>
__global__ __launch_bounds__(64 * kLineWaves, line_min_waves(E, (int)sizeof(T))) void k_line(cx<T>* __restrict__ psi,
                                                                                          PassArgs a) {
  __shared__ cx<T> xch[kLineWaves][line_lds<N, E>()];
  __shared__ uint4 ltw[(pass_tw<N, E, KIND>() * (int)sizeof(cx<T>) + 15) / 16];
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
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  line_body<T, N, E, KIND>(psi, a, (int)xcd_tile(blockIdx.x, nb) * kLineWaves + wave, xch[wave],
                           reinterpret_cast<cx<T>*>(ltw));
}

// Line pass over many grids (an ensemble's partition, see k_pass_batched): block b processes
// work item items[b] = (instance, group of kLineWaves tiles).
template <int N, int E, int KIND, int ES>
constexpr int batched_line_tw() {
  if constexpr (line_ok(N, E, ES)) return pass_tw<N, E, KIND>();
  else return 0;
}
template <typename T, int KIND, int E>
__global__ __launch_bounds__(64 * kLineWaves, line_min_waves(E, (int)sizeof(T))) void k_line_batched(
    const int2* __restrict__ items, const PassArgs* __restrict__ args) {
  constexpr int ES = (int)sizeof(T);
  constexpr int BUF = E == 4 ? cmax(cmax(line_lds<64, 4>(), line_lds<128, 4>()), line_lds<256, 4>())
                             : cmax(cmax(line_lds<192, 12>(), line_lds<384, 12>()), line_lds<768, 12>());
  constexpr int TWM = cmax(cmax(cmax(batched_line_tw<64, E, KIND, ES>(), batched_line_tw<128, E, KIND, ES>()),
                                cmax(batched_line_tw<192, E, KIND, ES>(), batched_line_tw<256, E, KIND, ES>())),
                           cmax(batched_line_tw<384, E, KIND, ES>(), batched_line_tw<768, E, KIND, ES>()));
  __shared__ cx<T> xch[kLineWaves][BUF];
  __shared__ uint4 ltwr[(TWM * (int)sizeof(cx<T>) + 15) / 16];
  cx<T>* ltw = reinterpret_cast<cx<T>*>(ltwr);
  const int2 it = items[blockIdx.x];
  const PassArgs& a = args[it.x];
  if constexpr (KIND == C_PROP) {
    if (a.advance_clock && it.y == 0 && threadIdx.x == 64 * kLineWaves - 1) advance_clock(a);
  }
  cx<T>* psi = reinterpret_cast<cx<T>*>(a.state);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = it.y * kLineWaves + wave;
#define SGP_LCASE(NN)                                                                              \
  case NN:                                                                                         \
    if constexpr (line_ok(NN, E, ES)) line_body<T, NN, E, KIND>(psi, a, tile, xch[wave], ltw);      \
    break;
  switch (a.n_line) {
    SGP_LCASE(64) SGP_LCASE(128) SGP_LCASE(192) SGP_LCASE(256) SGP_LCASE(384) SGP_LCASE(768)
    default: break;
  }
#undef SGP_LCASE
}

}  // namespace sgp
