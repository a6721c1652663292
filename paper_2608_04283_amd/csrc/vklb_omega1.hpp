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

// Lane 63's value, in every lane (all lanes active).
__device__ inline float wave_last(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ inline double wave_last(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), 63);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

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
  load_partials<MHD>(sd, W, pa, pb);
  const Step S = begin_step<MHD>(sd, red, W, in, pa, pb);
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
  double lam = 0.0, cfm = 0.0;
  if (active) {
    T prevm[P];  // +y equilibrium of the row below the one being collided
    {
      T fm[P], net[P];
      UK::template axis_sent<1>(preU, sd.ph, pr, ixi, Lam, ch, prevm, fm, net);
    }
    // Of the row waiting for the row above it: the sum so far (sum form) or
    // U, the x and +y differences and its own -y equilibrium (delta forms).
    T cU[P], cX[P], cY[P], c5[P], clo[P];
    auto finish = [&](int j, const T(&ym)[P]) {
      const int r = y0 + j;
      T Un[P], lo_new[P], dY[P];
#pragma unroll
      for (int v = 0; v < P; ++v) dY[v] = UK::SUM ? T(0) : cY[v] + (ym[v] - c5[v]);
      if constexpr (UK::PAIR) {
        if (pr.on) UK::template pair_step<1>(pr, cY[6], cY[8], c5[6], c5[8], ym[6], ym[8], dY[6], dY[8]);
      }
#pragma unroll
      for (int v = 0; v < P; ++v) {
        if (UK::SUM) Un[v] = cU[v] + ym[v];
        else Un[v] = K::advance(cU[v], cX[v] + dY[v], clo[v], lo_new[v]);
      }
      if (lane < nvalid) {
        gmem<T>* p = dst + UK::row(sd, r) + x0;
#pragma unroll
        for (int v = 0; v < P; ++v) {
          p[v * us + lc] = Un[v];
          if (K::COMP) p[(P + v) * us + lc] = lo_new[v];
        }
        K::new_state(sd, Un, (long long)r * nx + x0 + lane, n + 1, lam, cfm);
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
      T U[P], lo[P], hv[P];
#pragma unroll
      for (int v = 0; v < P; ++v) {
        U[v] = nU[v];
        lo[v] = nlo[v];
        hv[v] = s_halo[wid][hside][i & 31][v];
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
        a1[v] = wave_from_left(fp0[v], hv[v]);
        a2[v] = wave_from_right(fm0[v], hv[v]);
        if (last != 63) {
          const T e = wave_last(hv[v]);
          a2[v] = lane == last ? e : a2[v];
        }
        if (UK::SUM) {
          cU[v] = ((a1[v] + a2[v]) + UK::rest(U[v], net0[v] + net1[v], sd.ph, ixi)) + prevm[v];
        } else {
          cU[v] = U[v];
          cX[v] = (a1[v] - fp0[v]) + (a2[v] - fm0[v]);
          cY[v] = prevm[v] - fp1[v];
          c5[v] = fm1[v];
          clo[v] = lo[v];
        }
      }
      if constexpr (UK::PAIR) {
        if (pr.on) {
          UK::template pair_step<0>(pr, a1[5], a1[8], U[5], U[8], a2[5], a2[8], cX[5], cX[8]);
          cY[6] = prevm[6];  // the row below's own values, until the row above is known
          cY[8] = prevm[8];
        }
      }
#pragma unroll
      for (int v = 0; v < P; ++v) prevm[v] = fp1[v];
    }
    T fp[P], fm[P], net[P];
    UK::template axis_sent<1>(nU, sd.ph, pr, ixi, Lam, ch, fp, fm, net);
    finish(nr - 1, fm);
  }
  block_max2<MHD>(lam, cfm, red_end, W);
  end_step(sd, S, tile, lam, cfm);
}

template <int KIND, class T, int BASIS>
__global__ void __launch_bounds__(64 * kUWaves) k_ustep2d(const SolveDesc sd) {
  ustep2d_tile<KIND, T, BASIS>(sd, xcd_remap(blockIdx.x, gridDim.x));
}

// One tile of a solve that keeps U, as step2d_tile for the batched launch.
template <int KIND, class T, int BASIS>
__global__ void __launch_bounds__(64 * kUWaves)
    k_ustep_batched(const SolveDesc* __restrict__ descs, const WorkItem* __restrict__ work,
                    const int* __restrict__ nwork, int par) {
  const int i = blockIdx.x;
  if (i >= *nwork) return;
  const WorkItem w = work[i];
  SolveDesc sd = descs[w.slot];
  sd.par = par;
  ustep2d_tile<KIND, T, BASIS>(sd, w.tile);
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
// kernels that store them, bit for bit what those would hold: after a step,
// f_q(x) = f^eq_q(U^{n-1}(x - v_q)) with that step's speeds; before the
// first one (first = 1), f^eq(U_0) of the cell itself.
template <int KIND, int DIM, class T, int BASIS>
__global__ void __launch_bounds__(256) k_upopulate(const SolveDesc sd, int first) {
  using UK = UKern<KIND, DIM, T, BASIS>;
  using K = typename UK::K;
  constexpr int P = UK::P, Q = UK::Q, REST = UK::REST;
  const DevState* st = sd.st;
  const long long n = st->S[sd.par].n;
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
