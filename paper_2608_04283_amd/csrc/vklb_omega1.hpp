// Step kernels of solves with omega = 1, whose state is U alone.
//
// At omega = 1 the collision f* = f - omega (f - f^eq(U)) is f^eq(U) itself,
// so what a cell's populations held before it no longer matters: the
// populations of step n + 1 are f_q(x) = f^eq_q(U^n(x - v_q)), a function of
// the U field of step n (Sec. 4.1), and U^{n+1} is their sum. These kernels
// therefore read and write U instead of Q populations: 2 p s bytes per
// cell-step in place of 2 Q p s (2D Euler FP32: 32 instead of 160). The
// populations are not lost: k_upopulate rebuilds them from U^n, which the
// other buffer still holds, when a checkpoint asks for them, and k_uextract
// takes U from a checkpoint's populations.
//
// U is formed as in the kernels that store populations: as their sum (BASIS
// 0), or as U plus the streamed differences of the moving ones (BASIS 1, and
// compensated 2, whose low part of U is kept as p more planes).
//
// Layout: rows in grid order; a row holds its PL planes one after another,
// `us` values each (nx rounded up to 64), so a wavefront's plane access is
// one aligned run at a scalar base plus the lane, and the address arithmetic
// stays on the scalar unit.
#pragma once

#include "vklb_kernels.hpp"

namespace vklb {

// Lane i of the wavefront gets lane i - 1's value (wave_from_left) or lane
// i + 1's (wave_from_right); the lane at the end gets its own `edge`.
__device__ inline float wave_from_left(float v, float edge) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xF, 0xF, false));
}
__device__ inline float wave_from_right(float v, float edge) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xF, 0xF, false));
}
template <int CTRL>
__device__ inline double wave_shift64(double v, double edge) {
  const long long b = __double_as_longlong(v), e = __double_as_longlong(edge);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)e, (int)b, CTRL, 0xF, 0xF, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(e >> 32), (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline double wave_from_left(double v, double edge) { return wave_shift64<0x138>(v, edge); }
__device__ inline double wave_from_right(double v, double edge) { return wave_shift64<0x130>(v, edge); }

template <int KIND, int DIM, class T, int BASIS>
struct UKern {
  using K = Kern<KIND, DIM, T, BASIS>;
  static constexpr int P = K::P, Q = K::Q, REST = K::REST;
  static constexpr bool SUM = !K::DELTA;
  static constexpr int PL = K::COMP ? 2 * P : P;  // stored planes of a row

  // Offset of a row in a U buffer; plane v of it starts v * sd.us further on.
  __device__ static inline long long row(const SolveDesc& sd, long long r) { return r * PL * sd.us; }

  // U of the cell at element offset `off` of plane 0.
  template <class SP>
  __device__ static inline void load(SP __restrict__ src, const SolveDesc& sd, long long off, T (&U)[P]) {
#pragma unroll
    for (int v = 0; v < P; ++v) U[v] = src[off + (long long)v * sd.us];
  }

  // The equilibria moving along axis d and, for the sum form, F+ - F- of the
  // axis (its share of the rest population).
  template <int AXIS>
  __device__ static inline void axis(const T (&U)[P], const Phys& ph, double ixi, double Lam, double ch, T (&fp)[P],
                                     T (&fm)[P], T (&net)[P]) {
    Equilibrium<KIND, DIM, T>::eval_axis_net(U, ph, T(ixi), T(Lam), T(ch), AXIS, fp, fm, net);
  }
  // MHD, delta forms: the cleaning pair (B_n, psi) of an axis has a linear
  // flux, (psi, c_h^2 B_n), and D = eta (B_n, psi) with eta = beta(c_h) c_h, so
  // its increment of U needs only differences of U between the cells:
  //   dB_n = (psi_L - psi_R) / (2 xi) + e (B_L - 2 B + B_R),
  //   dpsi = c_h^2 (B_L - B_R) / (2 xi) + e (psi_L - 2 psi + psi_R),  e = c + eta / xi.
  // Formed that way it does not carry the rounding of the pair's populations,
  // which are c_h / |psi| times larger than psi's own (a 2 x 3 grid's psi: the
  // difference of populations left it at 1.1e-4 of the FP64 oracle in FP32).
  // With the sigmoid normalized per cell (alpha_local) eta differs from cell
  // to cell and the pair's populations are exchanged like the others.
  static constexpr bool PAIR = KIND == K_MHD && !SUM;
  struct Pair {
    T hb, hp, e;  // 1 / (2 xi), c_h^2 / (2 xi), c + eta / xi
    bool on;
  };
  __device__ static inline Pair pair_of(const Phys& ph, double ixi, double Lam, double ch) {
    Pair p;
    p.on = PAIR && !ph.alpha_local;
    p.hb = T(0.5 * ixi);
    p.hp = T(0.5 * ch * ch * ixi);
    const T hk = Lam > 0.0 ? qdiv(T(0.5 * ph.k), T(Lam)) : T(0);
    p.e = T(ph.c) + beta_w(T(ch), hk, ph.kinf) * T(ch) * T(ixi);
    return p;
  }
  // As axis, with the pair's values U itself in both directions (p.on).
  template <int AXIS>
  __device__ static inline void axis_sent(const T (&U)[P], const Phys& ph, const Pair& p, double ixi, double Lam,
                                          double ch, T (&fp)[P], T (&fm)[P], T (&net)[P]) {
    axis<AXIS>(U, ph, ixi, Lam, ch, fp, fm, net);
    if constexpr (PAIR) {
      if (p.on) {
        fp[5 + AXIS] = fm[5 + AXIS] = U[5 + AXIS];
        fp[8] = fm[8] = U[8];
      }
    }
  }
  // The axis' increment of the pair from the values sent by the left (or
  // lower) cell l, the cell itself and the right (upper) cell r.
  template <int AXIS>
  __device__ static inline void pair_step(const Pair& p, T Bl, T Pl, T B, T Ps, T Br, T Pr, T& dB, T& dP) {
    dB = p.hb * (Pl - Pr) + p.e * ((Bl - B) + (Br - B));
    dP = p.hp * (Bl - Br) + p.e * ((Pl - Ps) + (Pr - Ps));
  }
  // Rest population from U and the sum of the axes' F+ - F-.
  __device__ static inline T rest(T U, T net, const Phys& ph, double ixi) {
    return (T(1) - T(2 * DIM) * T(ph.c)) * U - net * T(ixi);
  }
};

// ---------------------------------------------------------------------------
// 2D step. Every wavefront marches on its own: it owns 64 columns and `band`
// rows, keeps one row's equilibria in registers, takes the x neighbours' from
// the lanes on either side with DPP wave shifts, and finishes row r - 1 when
// row r's y equilibria are known. Nothing is exchanged between wavefronts and
// no barrier stands in the march, so the wavefronts of a SIMD drift apart and
// fill each other's waits; the columns left and right of the strip are
// collided 32 rows at a time (lanes 0-31 left, 32-63 right) into the
// wavefront's own LDS. The workgroup (four wavefronts, neighbouring strips of
// a band first) meets only in the two reductions of the step's maxima.
// ---------------------------------------------------------------------------
constexpr int kUWaves = 4;  // wavefronts of a workgroup

template <int KIND, class T, int BASIS>
__device__ inline void ustep2d_tile(const SolveDesc& sd, int tile) {
  using UK = UKern<KIND, 2, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, PL = UK::PL, W = 64 * kUWaves;
  constexpr bool MHD = KIND == K_MHD;
  __shared__ double red[2 * kUWaves + 2], red_end[2 * kUWaves + 2];
  __shared__ T s_halo[kUWaves][2][32][P];  // wavefront, (left +x, right -x), row, var
  const int nx = sd.nx, ny = sd.ny, H = sd.band;
  const long long us = sd.us;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int nstrips = (nx + 63) / 64, nbands = (ny + H - 1) / H;
  const int gw = tile * kUWaves + wid;
  const bool active = gw < nstrips * nbands;  // the last workgroup may have idle wavefronts
  const int strip = active ? gw % nstrips : 0, band = active ? gw / nstrips : 0;
  const int x0 = strip * 64, y0 = band * H, y1 = min(y0 + H, ny), nr = y1 - y0;
  // Lanes past the side repeat the last column; the column right of it then
  // comes from the halo, as at lane 63 of a full strip.
  const int nvalid = min(64, nx - x0), last = nvalid - 1;
  const unsigned lc = min(lane, last);
  const StateIn in = read_state(sd);
  const int bp = predicted_parity(sd);
  const gmem<T>* __restrict__ src = gl((const T*)(bp ? sd.fb : sd.fa));
  auto load_row = [&](long long r, T(&U)[P]) {
    const gmem<T>* p = src + UK::row(sd, r) + x0;
#pragma unroll
    for (int v = 0; v < P; ++v) U[v] = p[v * us + lc];
  };
  auto load_lo = [&](long long r, T(&lo)[P]) {
    const gmem<T>* p = src + UK::row(sd, r) + x0;
#pragma unroll
    for (int v = 0; v < P; ++v) lo[v] = K::COMP ? p[(P + v) * us + lc] : T(0);
  };
  const int hside = lane >> 5;
  const int hx = map_index(hside == 0 ? x0 - 1 : min(x0 + 64, nx), nx, sd.bcx);
  auto load_halo = [&](int k, T(&hU)[P]) {  // row k of the band, if it has one
    UK::load(src, sd, UK::row(sd, y0 + min(k, nr - 1)) + hx, hU);
  };
  const int pre = map_index(y0 - 1, ny, sd.bcy), post = map_index(y1, ny, sd.bcy);
  T preU[P], nU[P], nlo[P], hU[P];
  auto load_first = [&]() {
    if (!active) return;
    load_row(pre, preU);
    load_halo(lane & 31, hU);
    load_row(y0, nU);
    load_lo(y0, nlo);
  };
  load_first();
  double pa, pb;
  const bool few = sd.nred <= kWavePartials;
  if (few) load_partials_wave<MHD>(sd, pa, pb);
  else load_partials<MHD>(sd, W, pa, pb);
  const Step S = few ? begin_step_wave<MHD>(sd, in, pa, pb) : begin_step<MHD>(sd, red, W, in, pa, pb);
  if (S.done) {
    carry_done(sd, S, tile);
    return;
  }
  const long long n = S.n;
  if (int(n & 1) != bp) {
    src = gl((const T*)((n & 1) ? sd.fb : sd.fa));
    load_first();
  }
  gmem<T>* __restrict__ dst = gl((T*)((n & 1) ? sd.fa : sd.fb));
  const double ixi = 1.0 / S.xi, Lam = S.lam, ch = S.ch;
  const typename UK::Pair pr = UK::pair_of(sd.ph, ixi, Lam, ch);
  T lamT = T(0), cfT = T(0);  // (widened after the march: exact)
  if (active) {
    T prevm[P];  // +y equilibrium of the row below the one being collided
    {
      T fm[P], net[P];
      UK::template axis_sent<1>(preU, sd.ph, pr, ixi, Lam, ch, prevm, fm, net);
    }
    // Of the row waiting for the row above it: the sum so far (sum form) or
    // U, the x and +y differences (cD) and its own -y equilibrium (c5); of
    // MHD's cleaning pair, the row below's B_y and psi (cB, cP).
    T cU[P], cD[P], c5[P], clo[P], cB = T(0), cP = T(0);
    auto finish = [&](int j, const T(&ym)[P]) {
      const int r = y0 + j;
      T Un[P], lo_new[P], d[P];
#pragma unroll
      for (int v = 0; v < P; ++v) d[v] = UK::SUM ? T(0) : cD[v] + (ym[v] - c5[v]);
      if constexpr (UK::PAIR) {
        if (pr.on) {
          T dB, dP;
          UK::template pair_step<1>(pr, cB, cP, cU[6], cU[8], ym[6], ym[8], dB, dP);
          d[6] = cD[6] + dB;
          d[8] = cD[8] + dP;
        }
      }
#pragma unroll
      for (int v = 0; v < P; ++v) {
        if (UK::SUM) Un[v] = cU[v] + ym[v];
        else Un[v] = K::advance(cU[v], d[v], clo[v], lo_new[v]);
      }
      if (lane < nvalid) {
        gmem<T>* p = dst + UK::row(sd, r) + x0;
#pragma unroll
        for (int v = 0; v < P; ++v) {
          p[v * us + lc] = Un[v];
          if (K::COMP) p[(P + v) * us + lc] = lo_new[v];
        }
        K::new_state(sd, Un, (long long)r * nx + x0 + lane, n + 1, lamT, cfT);
      }
    };
    for (int i = 0; i < nr; ++i) {
      if ((i & 31) == 0) {  // halo columns of the next 32 rows
        if (i) load_halo(i + (lane & 31), hU);
        T fp[P], fm[P], net[P];
        UK::template axis_sent<0>(hU, sd.ph, pr, ixi, Lam, ch, fp, fm, net);
#pragma unroll
        for (int v = 0; v < P; ++v) s_halo[wid][hside][lane & 31][v] = hside == 0 ? fp[v] : fm[v];
        // this wavefront alone reads them
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      T U[P], lo[P], hl[P], hr[P];
#pragma unroll
      for (int v = 0; v < P; ++v) {
        U[v] = nU[v];
        lo[v] = nlo[v];
        hl[v] = s_halo[wid][0][i & 31][v];
        hr[v] = s_halo[wid][1][i & 31][v];
      }
      if (i + 1 < nr) {
        load_row(y0 + i + 1, nU);
        load_lo(y0 + i + 1, nlo);
      } else {
        load_row(post, nU);
      }
      T fp1[P], fm1[P], net1[P];
      UK::template axis_sent<1>(U, sd.ph, pr, ixi, Lam, ch, fp1, fm1, net1);
      if (i > 0) finish(i - 1, fm1);
      T fp0[P], fm0[P], net0[P];
      UK::template axis_sent<0>(U, sd.ph, pr, ixi, Lam, ch, fp0, fm0, net0);
      T a1[P], a2[P];
#pragma unroll
      for (int v = 0; v < P; ++v) {
        a1[v] = wave_from_left(fp0[v], hl[v]);
        a2[v] = wave_from_right(fm0[v], hr[v]);
      }
      if (last != 63) {
#pragma unroll
        for (int v = 0; v < P; ++v) a2[v] = lane == last ? hr[v] : a2[v];
      }
#pragma unroll
      for (int v = 0; v < P; ++v) {
        if (UK::SUM) {
          cU[v] = ((a1[v] + a2[v]) + UK::rest(U[v], net0[v] + net1[v], sd.ph, ixi)) + prevm[v];
        } else {
          cU[v] = U[v];
          cD[v] = ((a1[v] - fp0[v]) + (a2[v] - fm0[v])) + (prevm[v] - fp1[v]);
          c5[v] = fm1[v];
          clo[v] = lo[v];
        }
      }
      if constexpr (UK::PAIR) {
        if (pr.on) {
          T dB, dP;
          UK::template pair_step<0>(pr, a1[5], a1[8], U[5], U[8], a2[5], a2[8], dB, dP);
          cD[5] = dB + (prevm[5] - fp1[5]);
          cD[6] = (a1[6] - fp0[6]) + (a2[6] - fm0[6]);
          cD[8] = dP;
          cB = prevm[6];
          cP = prevm[8];
        }
      }
#pragma unroll
      for (int v = 0; v < P; ++v) prevm[v] = fp1[v];
    }
    T fp[P], fm[P], net[P];
    UK::template axis_sent<1>(nU, sd.ph, pr, ixi, Lam, ch, fp, fm, net);
    finish(nr - 1, fm);
  }
  double lam = double(lamT), cfm = double(cfT);
  block_max2<MHD>(lam, cfm, red_end, W);
  end_step(sd, S, tile, lam, cfm);
}

template <int KIND, class T, int BASIS>
__global__ void __launch_bounds__(64 * kUWaves) k_ustep2d(const SolveDesc sd) {
  ustep2d_tile<KIND, T, BASIS>(sd, xcd_remap(blockIdx.x, gridDim.x));
}

// ---------------------------------------------------------------------------
// Characteristic boundary of a 1D U solve (Sec. 3.3), as step1d_tile applies
// it: U_b^{n+1} = U_b - P (Lambda dW)' / xi from U^n of the boundary cell and
// of its interior neighbour `nb`; the cell's populations become the
// equilibrium of it, whose sum is the new U in the sum form.
// ---------------------------------------------------------------------------
template <int KIND, class T, int BASIS>
__device__ inline void uchar_state(const SolveDesc& sd, const T* U, const T* nb, bool right, double ixi, double Lam,
                                   double ch, T* Un, T* fplus, T* rest, T* fminus) {
  using UK = UKern<KIND, 1, T, BASIS>;
  constexpr int P = UK::P;
  T du[P], corr[P];
#pragma unroll
  for (int v = 0; v < P; ++v) du[v] = right ? U[v] - nb[v] : nb[v] - U[v];
  Cell<KIND, 1, T>::char_correction(U, du, sd.ph, T(ch), right, corr);
#pragma unroll
  for (int v = 0; v < P; ++v) Un[v] = U[v] - corr[v] * T(ixi);
  T fe[3][P];
  Equilibrium<KIND, 1, T>::eval(Un, sd.ph, T(ixi), T(Lam), T(ch), fe);
#pragma unroll
  for (int v = 0; v < P; ++v) {
    if (UK::SUM) Un[v] = ((T(0) + fe[0][v]) + fe[1][v]) + fe[2][v];
    fplus[v] = fe[0][v];
    rest[v] = UK::SUM ? fe[1][v] : Un[v];
    fminus[v] = fe[2][v];
  }
}

// New U of a 1D cell from its own equilibria and the populations arriving
// from the left (a1) and the right (a2).
template <int KIND, class T, int BASIS>
__device__ inline void uadvance1d(const SolveDesc& sd, const typename UKern<KIND, 1, T, BASIS>::Pair& pr, double ixi,
                                  const T* U, const T* lo, const T* fp, const T* fm, const T* net, const T* a1,
                                  const T* a2, T* Un, T* lo_new) {
  using UK = UKern<KIND, 1, T, BASIS>;
  constexpr int P = UK::P;
  T d[P];
#pragma unroll
  for (int v = 0; v < P; ++v) d[v] = (a1[v] - fp[v]) + (a2[v] - fm[v]);
  if constexpr (UK::PAIR) {
    if (pr.on) UK::template pair_step<0>(pr, a1[5], a1[8], U[5], U[8], a2[5], a2[8], d[5], d[8]);
  }
#pragma unroll
  for (int v = 0; v < P; ++v) {
    if (UK::SUM) Un[v] = (a1[v] + UK::rest(U[v], net[v], sd.ph, ixi)) + a2[v];
    else Un[v] = UK::K::advance(U[v], d[v], lo[v], lo_new[v]);
  }
}

// ---------------------------------------------------------------------------
// 1D step: one cell per lane, the populations exchanged through LDS. The cells
// on either side of a tile are collided by the first and the last of its 256
// lanes (254 cells a tile), or (SIDE) by a fifth wavefront (256 cells a tile). The fifth
// wavefront shares a SIMD with another one, so it pays only where it saves a
// workgroup on some compute units that the others would wait for: 65,536 cells
// are 256 tiles of 256, one for each unit, but 259 of 254 (uside_of).
// ---------------------------------------------------------------------------
constexpr int utile1d(bool side) { return side ? 256 : 254; }
constexpr int ulanes1d(bool side) { return side ? 320 : 256; }

template <int KIND, class T, int BASIS, bool CHARBC, bool SIDE>
__device__ inline void ustep1d_tile(const SolveDesc& sd, int tile) {
  using UK = UKern<KIND, 1, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, B = ulanes1d(SIDE), TW = utile1d(SIDE);
  constexpr bool MHD = KIND == K_MHD;
  __shared__ double red[2 * (B / 64) + 2], red_end[2 * (B / 64) + 2];
  __shared__ T s_plus[P][TW + 2], s_minus[P][TW + 2];  // by position in the tile, its side cells included
  __shared__ T s_unb[2][P];  // characteristic boundaries: U^n of cells 1 and N - 2
  const int N = sd.nx;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool side = SIDE && wid == TW / 64;
  const int x0 = tile * TW;
  const int x = SIDE ? (side ? (lane == 0 ? x0 - 1 : x0 + TW) : x0 + tid) : x0 - 1 + tid;
  const bool own = SIDE ? !side : tid >= 1 && tid <= TW;
  const int xl = map_index(min(x, N), N, sd.bcx);
  const StateIn in = read_state(sd);
  const int bp = predicted_parity(sd);
  T U[P], lo[P];
  auto load_cell = [&](const gmem<T>* __restrict__ src) {
    UK::load(src, sd, xl, U);
#pragma unroll
    for (int v = 0; v < P; ++v) lo[v] = K::COMP ? src[xl + (long long)(P + v) * sd.us] : T(0);
  };
  load_cell(gl((const T*)(bp ? sd.fb : sd.fa)));
  double pa, pb;
  const bool few = sd.nred <= kWavePartials;
  if (few) load_partials_wave<MHD>(sd, pa, pb);
  else load_partials<MHD>(sd, B, pa, pb);
  const Step S = few ? begin_step_wave<MHD>(sd, in, pa, pb) : begin_step<MHD>(sd, red, B, in, pa, pb);
  if (S.done) {
    carry_done(sd, S, tile);
    return;
  }
  const long long n = S.n;
  if (int(n & 1) != bp) load_cell(gl((const T*)((n & 1) ? sd.fb : sd.fa)));
  gmem<T>* __restrict__ dst = gl((T*)((n & 1) ? sd.fa : sd.fb));
  const double ixi = 1.0 / S.xi, Lam = S.lam, ch = S.ch;
  const typename UK::Pair pr = UK::pair_of(sd.ph, ixi, Lam, ch);
  T fp[P], fm[P], net[P];
  UK::template axis_sent<0>(U, sd.ph, pr, ixi, Lam, ch, fp, fm, net);
  const int pos = x - x0 + 1;
  if (!side || lane < 2) {
#pragma unroll
    for (int v = 0; v < P; ++v) {
      s_plus[v][pos] = fp[v];
      s_minus[v][pos] = fm[v];
    }
  }
  const bool charbc = CHARBC && sd.bcx == 2 && N >= 2;
  if (charbc && x == 1) {
#pragma unroll
    for (int v = 0; v < P; ++v) s_unb[0][v] = U[v];
  }
  if (charbc && x == N - 2) {
#pragma unroll
    for (int v = 0; v < P; ++v) s_unb[1][v] = U[v];
  }
  __syncthreads();
  double lam = 0.0, cfm = 0.0;
  if (own && x < N) {
    T a1[P], a2[P], Un[P], lo_new[P];
#pragma unroll
    for (int v = 0; v < P; ++v) {
      a1[v] = s_plus[v][pos - 1];
      a2[v] = s_minus[v][pos + 1];
    }
    if (charbc && (x == 0 || x == N - 1)) {
      T e0[P], e1[P], e2[P];
      uchar_state<KIND, T, BASIS>(sd, U, s_unb[x == 0 ? 0 : 1], x != 0, ixi, Lam, ch, Un, e0, e1, e2);
#pragma unroll
      for (int v = 0; v < P; ++v) lo_new[v] = T(0);
    } else {
      uadvance1d<KIND, T, BASIS>(sd, pr, ixi, U, lo, fp, fm, net, a1, a2, Un, lo_new);
    }
#pragma unroll
    for (int v = 0; v < P; ++v) {
      dst[x + (long long)v * sd.us] = Un[v];
      if (K::COMP) dst[x + (long long)(P + v) * sd.us] = lo_new[v];
    }
    K::new_state(sd, Un, x, n + 1, lam, cfm);
  }
  block_max2<MHD>(lam, cfm, red_end, B);
  end_step(sd, S, tile, lam, cfm);
}

template <int KIND, class T, int BASIS, bool CHARBC, bool SIDE>
__global__ void __launch_bounds__(ulanes1d(SIDE)) k_ustep1d(const SolveDesc sd) {
  ustep1d_tile<KIND, T, BASIS, CHARBC, SIDE>(sd, blockIdx.x);
}

// Largest grid that runs in one workgroup, [MHD][FP64]: what its kernels hold
// at two cells a lane (MHD and FP64: as many registers as spill beyond), and
// where a step still takes less than a launch. us per step at the limit, one
// workgroup / a launch each: FP32 Euler 2.88 / 3.14, shallow water 2.38 / 2.93,
// MHD 4.18 / 4.69; FP64 Euler 2.98 / 3.35, MHD 5.35 / 5.74.
constexpr int kUWgMax[2][2] = {{2048, 1024}, {768, 512}};

// Max over the wavefront, in every lane, of non-negative values (negatives
// and NaN count as 0). FP32 values are reduced as FP32: widening is exact.
__device__ inline float wave_max_t(float v) { return __uint_as_float(wave_umax(__float_as_uint(v >= 0.f ? v : 0.f))); }
__device__ inline double wave_max_t(double v) { return wave_max(v); }

// ---------------------------------------------------------------------------
// Small 1D grids: `count` whole steps in one workgroup, as k_run1d_wg, with U
// in registers. A step meets at two barriers: after the wavefronts' end
// populations are in LDS, and after their maxima are (with a flag for a
// non-physical state). 64-cell chunk k = r NW + w is held by wavefront w.
// Bitwise the results of `count` k_ustep1d launches.
// ---------------------------------------------------------------------------
template <int KIND, class T, int BASIS, int R, int B, bool CHARBC>
__global__ void __launch_bounds__(B) k_urun1d(const SolveDesc sd, int count) {
  using UK = UKern<KIND, 1, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, NW = B / 64, NC = R * NW;
  constexpr bool MHD = KIND == K_MHD;
  __shared__ T s_p[NC + 1][P], s_m[NC + 1][P];
  __shared__ T s_unb[2][P];
  __shared__ T s_lam[NW], s_cf[NW];
  __shared__ int s_bad[NW];
  __shared__ double red[2 * NW + 2];
  const int N = sd.nx;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  gmem<DevState>* st = gl(sd.st);
  const StateIn in = read_state(sd);
  const double T_end = in.T;
  const long long max_steps = in.max_steps;
  Scal sc = in.S;
  bool err = in.err;
  double lam = 0.0, cfm = 0.0;
  {
    const gmem<double>* pl = gl(sd.part) + (long long)sd.par * 2 * sd.nblocks;
    for (int i = tid; i < sd.nblocks; i += B) {
      lam = fmax(lam, pl[i]);
      if (MHD) cfm = fmax(cfm, pl[sd.nblocks + i]);
    }
    block_max2_all<MHD>(lam, cfm, red, B);
  }
  T U[R][P], lo[R][P], Uo[R][P];  // Uo: U of the step before, which a checkpoint's populations are built from
  {
    const gmem<T>* __restrict__ src = gl((const T*)((sc.n & 1) ? sd.fb : sd.fa));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = min(r * B + tid, N - 1);  // lanes past the end hold a copy of the last cell
      UK::load(src, sd, c, U[r]);
#pragma unroll
      for (int v = 0; v < P; ++v) lo[r][v] = K::COMP ? src[c + (long long)(P + v) * sd.us] : T(0);
    }
  }
  const bool periodic = sd.bcx == 0, charbc = CHARBC && N >= 2;
  Step last;
  bool stepped = false;
  for (int it = 0; it < count; ++it) {
    const Step S = derive_step(sc, T_end, max_steps, err, lam, cfm, sd.ph.ch_factor, sd.xi_mode, sd.nu, sd.xi_fixed,
                               sd.dx);
    if (S.done) {
      sc.done = 1;
      break;
    }
    last = S;
    stepped = true;
    const double ixi = 1.0 / S.xi, Lam = S.lam, ch = S.ch;
    const typename UK::Pair pr = UK::pair_of(sd.ph, ixi, Lam, ch);
    T fp[R][P], fm[R][P], net[R][P];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int k = r * NW + wid, c = r * B + tid;
      if (r * B + wid * 64 >= N) continue;  // a chunk past the end
      UK::template axis_sent<0>(U[r], sd.ph, pr, ixi, Lam, ch, fp[r], fm[r], net[r]);
      if (lane == 0) {
#pragma unroll
        for (int v = 0; v < P; ++v) s_m[k][v] = fm[r][v];
      }
      if (lane == 63) {
#pragma unroll
        for (int v = 0; v < P; ++v) s_p[k + 1][v] = fp[r][v];
      }
      if (c == (periodic ? N - 1 : 0)) {  // the left ghost's
#pragma unroll
        for (int v = 0; v < P; ++v) s_p[0][v] = fp[r][v];
      }
      if (charbc && c == 1) {
#pragma unroll
        for (int v = 0; v < P; ++v) s_unb[0][v] = U[r][v];
      }
      if (charbc && c == N - 2) {
#pragma unroll
        for (int v = 0; v < P; ++v) s_unb[1][v] = U[r][v];
      }
    }
    __syncthreads();
    T lm = T(0), cm = T(0);
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int k = r * NW + wid, c = r * B + tid;
      if (r * B + wid * 64 >= N) continue;
      T a1[P], a2[P], Un[P], lo_new[P];
#pragma unroll
      for (int v = 0; v < P; ++v) {
        const T hv = lane < 32 ? s_p[k][v] : s_m[k + 1][v];
        a1[v] = wave_from_left(fp[r][v], hv);
        a2[v] = wave_from_right(fm[r][v], hv);
      }
      if (c == N - 1) {  // the right ghost's
#pragma unroll
        for (int v = 0; v < P; ++v) a2[v] = periodic ? s_m[0][v] : fm[r][v];
      }
      if (c < N) {
        if (charbc && (c == 0 || c == N - 1)) {
          T e0[P], e1[P], e2[P];
          uchar_state<KIND, T, BASIS>(sd, U[r], s_unb[c == 0 ? 0 : 1], c != 0, ixi, Lam, ch, Un, e0, e1, e2);
#pragma unroll
          for (int v = 0; v < P; ++v) lo_new[v] = T(0);
        } else {
          uadvance1d<KIND, T, BASIS>(sd, pr, ixi, U[r], lo[r], fp[r], fm[r], net[r], a1, a2, Un, lo_new);
        }
        bad |= K::new_state(sd, Un, c, S.n + 1, lm, cm);
#pragma unroll
        for (int v = 0; v < P; ++v) {
          Uo[r][v] = U[r][v];
          U[r][v] = Un[v];
          if (K::COMP) lo[r][v] = lo_new[v];
        }
      }
    }
    const T wl = wave_max_t(lm), wc = MHD ? wave_max_t(cm) : T(0);
    const int wb = __ballot(bad) != 0;
    if (lane == 0) {
      s_lam[wid] = wl;
      if (MHD) s_cf[wid] = wc;
      s_bad[wid] = wb;
    }
    __syncthreads();
    T ml = T(0), mc = T(0);
    int mb = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      ml = fmax(ml, s_lam[w]);
      if (MHD) mc = fmax(mc, s_cf[w]);
      mb |= s_bad[w];
    }
    lam = double(ml);
    cfm = double(mc);
    err = err || mb != 0;
    sc.t = S.landing ? T_end : S.t + sd.dx / S.xi;
    sc.n = S.n + 1;
  }
  gmem<T>* __restrict__ dst = gl((T*)((sc.n & 1) ? sd.fb : sd.fa));
  gmem<T>* __restrict__ old = gl((T*)((sc.n & 1) ? sd.fa : sd.fb));
  if (stepped) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = r * B + tid;
      if (c < N) {
#pragma unroll
        for (int v = 0; v < P; ++v) {
          dst[c + (long long)v * sd.us] = U[r][v];
          old[c + (long long)v * sd.us] = Uo[r][v];
          if (K::COMP) dst[c + (long long)(P + v) * sd.us] = lo[r][v];
        }
      }
    }
  }
  const int pf = sd.par ^ (count & 1);
  gmem<double>* pl = gl(sd.part) + (long long)pf * 2 * sd.nblocks;
  for (int i = tid; i < sd.nblocks; i += B) {
    pl[i] = lam;
    pl[sd.nblocks + i] = cfm;
  }
  if (tid == 0) {
    store_scal(st, pf, sc);
    if (stepped) store_last(sd, last);
  }
}

// Batched step of the solves that keep U (see k_step_batched).
template <int KIND, int DIM, class T, int BASIS>
__global__ void __launch_bounds__(DIM == 1 ? ulanes1d(false) : 64 * kUWaves)
    k_ustep_batched(const SolveDesc* __restrict__ descs, const WorkItem* __restrict__ work,
                    const int* __restrict__ nwork, int par) {
  const int i = blockIdx.x;
  if (i >= *nwork) return;
  const WorkItem w = work[i];
  SolveDesc sd = descs[w.slot];
  sd.par = par;
  if constexpr (DIM == 1) ustep1d_tile<KIND, T, BASIS, true, false>(sd, w.tile);
  else ustep2d_tile<KIND, T, BASIS>(sd, w.tile);
}

// U of step 0 from the staging, and the speeds the populations f^eq(U_0) are
// built with. In the sum form U is formed from those populations, as every
// later step forms it; they are kept when the solve has room for them
// (sd.pop), since U alone does not give them back bit for bit.
template <int KIND, int DIM, class T, int BASIS>
__global__ void __launch_bounds__(256) k_uinit(const SolveDesc sd) {
  using UK = UKern<KIND, DIM, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, Q = UK::Q;
  __shared__ double red[10];
  const Step S = begin_step(sd, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) store_last(sd, S);
  T* __restrict__ u = (T*)sd.fa;
  T* __restrict__ f = (T*)sd.pop;
  const long long cells = (long long)sd.nx * sd.ny;
  const double ixi = 1.0 / S.xi;
  for (long long c = blockIdx.x * 256ll + threadIdx.x; c < cells; c += (long long)gridDim.x * 256) {
    const long long j = DIM == 2 ? c / sd.nx : 0;
    const long long off = UK::row(sd, j) + (c - j * sd.nx);
    T U[P];
#pragma unroll
    for (int v = 0; v < P; ++v) U[v] = T(sd.stage[v * cells + c]);
    if (UK::SUM) {
      T fe[Q][P];
      Equilibrium<KIND, DIM, T>::eval(U, sd.ph, T(ixi), T(S.lam), T(S.ch), fe);
      const long long pc = pcell(sd, c, false);
#pragma unroll
      for (int v = 0; v < P; ++v) {
        T s = T(0);
#pragma unroll
        for (int q = 0; q < Q; ++q) s += fe[q][v];
        U[v] = s;
        if (f) {
#pragma unroll
          for (int q = 0; q < Q; ++q) f[K::pidx(q * P + v, pc)] = fe[q][v];
        }
      }
    }
#pragma unroll
    for (int v = 0; v < P; ++v) {
      if (K::COMP) u[off + (long long)(P + v) * sd.us] = T(sd.stage[v * cells + c] - double(U[v]));
      u[off + (long long)v * sd.us] = U[v];
    }
  }
}

// U (hi + lo when compensated) into the FP64 staging.
template <int KIND, int DIM, class T, int BASIS>
__global__ void __launch_bounds__(256) k_umoments(const SolveDesc sd) {
  using UK = UKern<KIND, DIM, T, BASIS>;
  constexpr int P = UK::P;
  const long long n = sd.st->S[sd.par].n;
  const T* __restrict__ u = (const T*)((n & 1) ? sd.fb : sd.fa);
  double* out = const_cast<double*>(sd.stage);
  const long long cells = (long long)sd.nx * sd.ny;
  for (long long c = blockIdx.x * 256ll + threadIdx.x; c < cells; c += (long long)gridDim.x * 256) {
    const long long j = DIM == 2 ? c / sd.nx : 0;
    const long long off = UK::row(sd, j) + (c - j * sd.nx);
#pragma unroll
    for (int v = 0; v < P; ++v) {
      const T hi = u[off + (long long)v * sd.us];
      out[v * cells + c] = UK::K::COMP ? double(hi) + double(u[off + (long long)(P + v) * sd.us]) : double(hi);
    }
  }
}

// Populations of the current step n into sd.pop, in the blocked layout of the
// kernels that store them: after a step, f_q(x) = f^eq_q(U^{n-1}(x - v_q)) with
// that step's speeds; before the first one, f^eq(U_0) of the cell itself. They
// are this solve's own: in the sum form they add up, bit for bit, to the U it
// holds, and they equal the populations a storing kernel would hold up to
// rounding (its equilibria are formed in another order, eval_axis). Those an
// initialization or a restored checkpoint left there are kept (pop_n; n never
// comes back to it without another of the two).
template <int KIND, int DIM, class T, int BASIS>
__global__ void __launch_bounds__(256) k_upopulate(const SolveDesc sd) {
  using UK = UKern<KIND, DIM, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, Q = UK::Q, REST = UK::REST;
  const DevState* st = sd.st;
  const long long n = st->S[sd.par].n;
  if (n == st->pop_n) return;
  const bool first = n == 0;
  const T* __restrict__ cur = (const T*)((n & 1) ? sd.fb : sd.fa);
  const T* __restrict__ old = first ? cur : (const T*)((n & 1) ? sd.fa : sd.fb);
  T* __restrict__ f = (T*)sd.pop;
  const double ixi = 1.0 / st->last[0], Lam = st->last[1], ch = st->last[2];
  const int nx = sd.nx, ny = sd.ny;
  const long long cells = (long long)nx * ny;
  for (long long c = blockIdx.x * 256ll + threadIdx.x; c < cells; c += (long long)gridDim.x * 256) {
    const int j = DIM == 2 ? int(c / nx) : 0, i = int(c - (long long)j * nx);
    const long long pc = pcell(sd, c, false);
    T U[P], V[P], fp[P], fm[P], net[P], r[P];
    if constexpr (DIM == 1) {
      if (!first && sd.bcx == 2 && nx >= 2 && (i == 0 || i == nx - 1)) {  // a characteristic boundary cell
        UK::load(old, sd, i, U);
        UK::load(old, sd, i == 0 ? 1 : nx - 2, V);
        uchar_state<KIND, T, BASIS>(sd, U, V, i != 0, ixi, Lam, ch, net, fp, r, fm);
#pragma unroll
        for (int v = 0; v < P; ++v) {
          f[K::pidx(0 * P + v, pc)] = fp[v];
          f[K::pidx(1 * P + v, pc)] = r[v];
          f[K::pidx(2 * P + v, pc)] = fm[v];
          if (K::COMP) f[K::pidx(Q * P + v, pc)] = T(0);
        }
        continue;
      }
    }
    if (UK::SUM) {  // rest population of the cell itself
      UK::load(old, sd, UK::row(sd, j) + i, V);
      UK::template axis<0>(V, sd.ph, ixi, Lam, ch, fp, fm, r);
      if (DIM == 2) {
        UK::template axis<DIM - 1>(V, sd.ph, ixi, Lam, ch, fp, fm, net);
#pragma unroll
        for (int v = 0; v < P; ++v) r[v] += net[v];
      }
#pragma unroll
      for (int v = 0; v < P; ++v) r[v] = UK::rest(V[v], r[v], sd.ph, ixi);
    } else {
      UK::load(cur, sd, UK::row(sd, j) + i, r);
    }
#pragma unroll
    for (int v = 0; v < P; ++v) f[K::pidx(REST * P + v, pc)] = r[v];
    if (K::COMP) {
#pragma unroll
      for (int v = 0; v < P; ++v)
        f[K::pidx(Q * P + v, pc)] = cur[UK::row(sd, j) + i + (long long)(P + v) * sd.us];
    }
#pragma unroll
    for (int s = -1; s <= 1; s += 2) {  // arriving from the left / below (-1) and from the right / above (+1)
      const int ii = first ? i : map_index(i + s, nx, sd.bcx);
      UK::load(old, sd, UK::row(sd, j) + ii, U);
      UK::template axis<0>(U, sd.ph, ixi, Lam, ch, fp, fm, net);
      const int q = s < 0 ? 0 : (DIM == 1 ? 2 : 1);
#pragma unroll
      for (int v = 0; v < P; ++v) f[K::pidx(q * P + v, pc)] = s < 0 ? fp[v] : fm[v];
      if (DIM == 2) {
        const int jj = first ? j : map_index(j + s, ny, sd.bcy);
        UK::load(old, sd, UK::row(sd, jj) + i, U);
        UK::template axis<DIM - 1>(U, sd.ph, ixi, Lam, ch, fp, fm, net);
#pragma unroll
        for (int v = 0; v < P; ++v) f[K::pidx((s < 0 ? 3 : 4) * P + v, pc)] = s < 0 ? fp[v] : fm[v];
      }
    }
  }
}

// U of the current step from the populations in sd.pop (a restored checkpoint).
template <int KIND, int DIM, class T, int BASIS>
__global__ void __launch_bounds__(256) k_uextract(const SolveDesc sd) {
  using UK = UKern<KIND, DIM, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, Q = UK::Q;
  const long long n = sd.st->S[sd.par].n;
  T* __restrict__ u = (T*)((n & 1) ? sd.fb : sd.fa);
  const T* __restrict__ f = (const T*)sd.pop;
  const long long cells = (long long)sd.nx * sd.ny;
  for (long long c = blockIdx.x * 256ll + threadIdx.x; c < cells; c += (long long)gridDim.x * 256) {
    const long long j = DIM == 2 ? c / sd.nx : 0;
    const long long off = UK::row(sd, j) + (c - j * sd.nx), pc = pcell(sd, c, false);
    T U[P];
    K::moments_of(f, pc, U);
#pragma unroll
    for (int v = 0; v < P; ++v) {
      u[off + (long long)v * sd.us] = U[v];
      if (K::COMP) u[off + (long long)(P + v) * sd.us] = f[K::pidx(Q * P + v, pc)];
    }
  }
}

}  // namespace vklb
