// The one-dimensional quadratic model dS/dt = -S^2 used to illustrate the time
// schemes (Sec. "Phase shifting for one-dimensional problems", Eqs. model-1d-2 and
// 1d_initial, Fig. 8), FP64, for a batch of independent real signals.
//
//   N(S; s)_k = M_k conj(phi_k) (1/n) sum_j w_j e^{-2 pi i k j / n},
//   w_j = -v_j^2,  v_j = sum_k (phi M S)_k e^{2 pi i k j / n} (real field, Hermitian),
//   phi_k = e^{2 pi i k s / n},  M_k = [k <= kmax].
//
// One block per signal and launch, everything between the transforms' exchanges in
// registers: a thread holds the full spectrum (both signs of k) at the positions its
// first butterflies read, the product on the points its first transform leaves it, and
// the second transform, whose radices are the first's reversed, ends at the positions
// it started from.  Two real signals share one complex transform (the two shifts of an
// average).
//
// n a power of two: transforms of nf = n points.  Any other n: Bluestein's convolution
// over nf >= 2n - 1 points, nf a power of two.  With c_j = e^{i pi j^2 / n}, jk = (j^2 + k^2
// - (j-k)^2) / 2 turns the DFT of sign + into c_k times the convolution of z c with
// conj(c), two transforms with a multiplication by the chirp's transform between them; the
// DFT of sign - is the conjugate of that of the conjugate.
//
// A call of few signals is bound by latency: a chain of dependent transforms of 128 to 2048
// points on one CU, whose time is that of one wavefront's instructions and LDS round trips.
// So a step is one loop over its evaluations with one copy of each transform in the code,
// plans of 4 to 8 points a thread with every index known at compile time, and lines of up
// to 256 points inside one wavefront.  Direct sums are shorter up to 64 points (k_direct1d to
// 32, with every factor in registers) and for few kept modes (k_sums1d; the rule is at
// sums_waves).  Against direct O(n k_max) sums from LDS by 256 threads a signal, rk4, one step a
// call, launch included, us at 8 signals and at 40,000: n = 22 13 -> 8 and 260 -> 78; 48 23 -> 11
// and 484 -> 121; 128 51 -> 11 and 1363 -> 183; 256 101 -> 10 and 4379 -> 234; 258 with 6 modes 65
// -> 13 and 1394 -> 176; 300 169 -> 35 and 7317 -> 3235; 1022 1151 -> 54 and 99,200 -> 8210; 1024
// 1186 -> 19 and 187,000 -> 1602.
// Mixed-radix stages with the plan as an argument took 24.4 us at 256 and 31.8 us at 1024
// (index arithmetic on the one chain).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft_reg.hpp"

namespace ns1d {

using C = ns::Cx<double>;

enum Scheme { EULER = 0, EULER_PS = 1, RK2 = 2, PS_EXACT = 3, PS_APPROX = 4, RK4 = 5 };

// Evaluation e of a step: the next stage state is S0 + c r, r joins the sum with weight
// b (b = 0: the sum restarts), and after the last one S0 += fin sum.
struct Eval {
  double c, b;
  int pair;  // the average over the shifts 0 and `shift` instead of one evaluation
  int on;    // one evaluation: at `shift` instead of unshifted
};

struct Args {
  const double2* in;   // [batch][h] input spectra
  double2* out;        // [batch][h] result (may alias in)
  int n, h, kmax;
  int nsteps;          // 0: out = one evaluation N(S; shift)
  int nevals;
  int shifted;         // whether any evaluation uses the shift
  Eval eval[4];
  double fin, shift;
};

// Threads and radices of the first transform of nf points (the second's are reversed).
template <int NF> struct Plan;
template <> struct Plan<128> { static constexpr int TPL = 32; using A = ns::Radices<4, 4, 2, 4>; using B = ns::Radices<4, 2, 4, 4>; };
template <> struct Plan<256> { static constexpr int TPL = 64; using A = ns::Radices<4, 4, 4, 4>; using B = ns::Radices<4, 4, 4, 4>; };
template <> struct Plan<512> { static constexpr int TPL = 128; using A = ns::Radices<4, 4, 2, 4, 4>; using B = ns::Radices<4, 4, 2, 4, 4>; };
template <> struct Plan<1024> { static constexpr int TPL = 256; using A = ns::Radices<4, 4, 4, 4, 4>; using B = ns::Radices<4, 4, 4, 4, 4>; };
template <> struct Plan<2048> { static constexpr int TPL = 256; using A = ns::Radices<8, 8, 8, 4>; using B = ns::Radices<4, 8, 8, 8>; };

template <int NF>
constexpr int threads() { return Plan<NF>::TPL < 64 ? 64 : Plan<NF>::TPL; }

__device__ __forceinline__ C polar_pi(double x) {  // e^{i pi x}
  C z;
  sincospi(x, &z.im, &z.re);
  return z;
}

template <int NF>
__global__ void __launch_bounds__(threads<NF>()) k_model1d(Args a) {
  using P = Plan<NF>;
  constexpr int TPL = P::TPL;
  constexpr bool WAVE = TPL <= 64;
  using FA = ns::RegFft<NF, TPL, -1, typename P::A>;
  using FB = ns::RegFft<NF, TPL, +1, typename P::B>;
  constexpr int EPT = FA::EPT;
  static_assert(FA::UNIFORM && FB::UNIFORM && FA::RL == FB::R0 && FB::RL == FA::R0, "the transforms chain");
  __shared__ C tw[NF];  // e^{-2 pi i m / NF}
  __shared__ C xb[ns::line_pitch(NF)];
  __shared__ C sp[NF];  // a spectrum whose mirror is read (averages)
  const int t = threadIdx.x, n = a.n;
  const bool blue = NF != n;
  // one octant of the twiddles evaluated, the others by symmetry
  for (int m = t; m <= NF / 8; m += blockDim.x) {
    const C z = polar_pi(2.0 * (double)m / (double)NF);
    const double cs = z.re, sn = z.im;
    tw[m] = ns::cx(cs, -sn);
    tw[NF / 4 - m] = ns::cx(sn, -cs);
    tw[NF / 4 + m] = ns::cx(-sn, -cs);
    tw[NF / 2 - m] = ns::cx(-cs, -sn);
    tw[NF / 2 + m] = ns::cx(-cs, sn);
    tw[3 * NF / 4 - m] = ns::cx(-sn, cs);
    tw[3 * NF / 4 + m] = ns::cx(sn, cs);
    if (m > 0) tw[NF - m] = ns::cx(cs, sn);
  }
  __syncthreads();
  if (t >= TPL) return;  // short lines use part of their only wavefront
  const ns::LineView<double, 1> lv{xb};
  const C* in = reinterpret_cast<const C*>(a.in) + (size_t)blockIdx.x * a.h;
  C* out = reinterpret_cast<C*>(a.out) + (size_t)blockIdx.x * a.h;
  // at position p: the state (the conjugate of the mirror's past n/2), phi of the shift
  // likewise, c_p; zero or unused for p >= n
  C s0[EPT], cur[EPT], sum[EPT], ph[EPT], c[EPT], chirp[EPT], x[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int p = FA::in_pos(t, i), k = 2 * p <= n ? p : n - p;
    C v = p < n ? in[k] : ns::cx(0.0, 0.0);
    ph[i] = ns::cx(1.0, 0.0);
    if (a.shifted && p < n) ph[i] = polar_pi(2.0 * (double)k * a.shift / (double)n);
    if (2 * p > n) {
      v = ns::conj(v);
      ph[i] = ns::conj(ph[i]);
    }
    s0[i] = cur[i] = v;
    sum[i] = c[i] = chirp[i] = ns::cx(0.0, 0.0);
  }
  if (blue) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = FA::in_pos(t, i), q = NF - p;
      x[i] = ns::cx(0.0, 0.0);
      if (p < n) {
        c[i] = polar_pi((double)((p * p) % (2 * n)) / (double)n);
        x[i] = ns::conj(c[i]);
      } else if (q < n) {
        x[i] = ns::conj(polar_pi((double)((q * q) % (2 * n)) / (double)n));
      }
    }
    FA::template run<WAVE>(x, t, lv, tw);
#pragma unroll
    for (int i = 0; i < EPT; ++i) chirp[i] = ns::scale(x[i], 1.0 / (double)NF);
  }
  const double inv_n = 1.0 / (double)n;
  int step = 0, e = 0;
  for (;;) {
    const Eval ev = a.eval[e];
    // z = v_0 + i v_s of the two shifts (pair) or v alone, from the full spectra
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = FA::in_pos(t, i), k = 2 * p <= n ? p : n - p;
      C z = ns::cx(0.0, 0.0);
      if (p < n && k <= a.kmax) {
        z = cur[i];
        if (p == 0) z.im = 0.0;  // the k = 0 coefficient of a real field is real
        if (ev.pair || ev.on) {
          const C q = ns::cmul(z, ph[i]);
          z = ev.pair ? ns::cx(z.re - q.im, z.im + q.re) : q;
        }
      }
      x[i] = blue ? ns::cmul(z, c[i]) : ns::conj(z);
    }
    for (int turn = 0;; ++turn) {
      FA::template run<WAVE>(x, t, lv, tw);
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        // w = -v^2 (conjugated before and after: both transforms run conjugated)
        if (blue) x[i] = ns::cmul(x[i], chirp[i]);
        else x[i] = ns::cx(-x[i].re * x[i].re, ev.pair ? x[i].im * x[i].im : 0.0);
      }
      FB::template run<WAVE>(x, t, lv, tw);
      if (!blue || turn == 1) break;
#pragma unroll
      for (int i = 0; i < EPT; ++i) {  // c = 0 past n
        const C z = ns::cmul(x[i], c[i]);
        x[i] = ns::cmul(ns::cx(-z.re * z.re, ev.pair ? z.im * z.im : 0.0), c[i]);
      }
    }
    if (blue) {
#pragma unroll
      for (int i = 0; i < EPT; ++i) x[i] = ns::cmul(x[i], c[i]);
    }
    if (ev.pair) {
      ns::exchange_barrier<WAVE>();
#pragma unroll
      for (int i = 0; i < EPT; ++i) sp[FA::in_pos(t, i)] = x[i];
      ns::exchange_barrier<WAVE>();
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = FA::in_pos(t, i), k = 2 * p <= n ? p : n - p;
      C r = ns::cx(0.0, 0.0);
      if (p < n && k <= a.kmax) {
        const C f1 = ns::conj(x[i]);
        if (ev.pair) {
          const C f2 = ns::conj(sp[p == 0 ? 0 : n - p]);
          const C u = ns::cx(0.5 * (f1.re + f2.re), 0.5 * (f1.im - f2.im));
          const C v = ns::cx(0.5 * (f1.im + f2.im), -0.5 * (f1.re - f2.re));
          r = ns::scale(ns::scale(u, inv_n) + ns::scale(ns::cmulc(v, ph[i]), inv_n), 0.5);
        } else {
          r = ns::scale(ev.on ? ns::cmulc(f1, ph[i]) : f1, inv_n);
        }
        if (p == 0) r.im = 0.0;  // the mean of a real field
      }
      sum[i] = ev.b == 0.0 ? ns::cx(0.0, 0.0) : sum[i] + ns::scale(r, ev.b);
      if (e + 1 < a.nevals) {
        cur[i] = s0[i] + ns::scale(r, ev.c);
      } else {
        cur[i] = s0[i] = a.nsteps > 0 ? s0[i] + ns::scale(sum[i], a.fin) : r;
        sum[i] = ns::cx(0.0, 0.0);
      }
    }
    if (++e == a.nevals) {
      if (++step >= a.nsteps) break;
      e = 0;
    }
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int p = FA::in_pos(t, i);
    if (2 * p <= n) out[p] = s0[i];
  }
}

// n <= 32: direct sums with every factor in registers.  Thread j of group g (g = 0:
// unshifted, 1: shifted; both groups keep the state) holds cos and sin of 2 pi j m / n for
// 1 <= m < n/2, which serve v_j = S_0 + 2 sum_m Re(S_m e^{i ..}) and, m and n - m taken
// together, F_j = w_0 + (-1)^j w_{n/2} + sum_m ((w_m + w_{n-m}) cos - i (w_m - w_{n-m}) sin);
// the other operands are LDS broadcasts.
__global__ void __launch_bounds__(64) k_direct1d(Args a) {
  constexpr int J = 32, M = J / 2;
  __shared__ C tw[J], xs[2][M + 1], rs[2][J];
  __shared__ double ws[2][J];
  const int j = threadIdx.x % J, g = threadIdx.x / J, n = a.n, half = n / 2;
  const double inv_n = 1.0 / (double)n;
  if (g == 0 && j < n) tw[j] = polar_pi(2.0 * (double)j / (double)n);
  __syncthreads();
  const C* in = reinterpret_cast<const C*>(a.in) + (size_t)blockIdx.x * a.h;
  C* out = reinterpret_cast<C*>(a.out) + (size_t)blockIdx.x * a.h;
  const bool isk = j < a.h, kept = j <= a.kmax, isj = j < n;
  C w[M];
  {
    const int jn = isj ? j : 0;
    int e = 0;  // (j m) mod n
#pragma unroll
    for (int m = 1; m < M; ++m) {
      e += jn;
      if (e >= n) e -= n;
      w[m] = tw[e];
    }
  }
  C s0 = isk ? in[j] : ns::cx(0.0, 0.0), cur = s0, sum = ns::cx(0.0, 0.0);
  const C ph = a.shifted ? polar_pi(2.0 * (double)j * a.shift / (double)n) : ns::cx(1.0, 0.0);
  int step = 0, e = 0;
  for (;;) {
    const Eval ev = a.eval[e];
    const bool shift = ev.on || (ev.pair && g == 1);
    if (isk) {
      C x = kept ? cur : ns::cx(0.0, 0.0);
      if (j == 0) x.im = 0.0;  // the k = 0 coefficient of a real field is real
      xs[g][j] = shift ? ns::cmul(x, ph) : x;
    }
    __syncthreads();
    double v = 0.0;
#pragma unroll
    for (int m = 1; m < M; ++m) {
      if (m < half) {
        const C x = xs[g][m];
        v += x.re * w[m].re - x.im * w[m].im;
      }
    }
    v = xs[g][0].re + 2.0 * v;
    if (isj) ws[g][j] = -v * v;
    __syncthreads();
    C r = ns::cx(0.0, 0.0);
    if (kept) {
      r.re = ws[g][0] + ((j & 1) ? -ws[g][half] : ws[g][half]);
#pragma unroll
      for (int m = 1; m < M; ++m) {
        if (m < half) {
          const double p = ws[g][m], q = ws[g][n - m];
          r.re += (p + q) * w[m].re;
          r.im -= (p - q) * w[m].im;
        }
      }
      if (j == 0) r.im = 0.0;  // the mean of a real field
      r = ns::scale(shift ? ns::cmulc(r, ph) : r, inv_n);
    }
    if (ev.pair) {
      rs[g][j] = r;
      __syncthreads();
      r = ns::scale(rs[0][j] + rs[1][j], 0.5);
    }
    sum = ev.b == 0.0 ? ns::cx(0.0, 0.0) : sum + ns::scale(r, ev.b);
    if (e + 1 < a.nevals) {
      cur = s0 + ns::scale(r, ev.c);
    } else {
      cur = s0 = a.nsteps > 0 ? s0 + ns::scale(sum, a.fin) : r;
      sum = ns::cx(0.0, 0.0);
    }
    if (++e == a.nevals) {
      if (++step >= a.nsteps) break;
      e = 0;
    }
  }
  if (isk && g == 0) out[j] = s0;
}

// Few kept modes: direct sums, O(n kmax) instead of O(nf log nf).  Thread t of 64 WAVES keeps
// mode k = t mod M (M the power of two above kmax; the 64 WAVES / M segments keep the same
// state).  The points j and n - j share their factors,
//   v_j, v_{n-j} = S_0 + 2 (sum_m a_m cos -+ sum_m b_m sin),  S_m = a_m + i b_m, at 2 pi j m / n,
//   F_k = sum_{j <= n/2} (p_j cos - i q_j sin),  p, q = w_j +- w_{n-j} (w_j and 0 at j = 0, n/2):
// threads along j for v, along k for F, a segment taking every (segments)-th j.  The two
// shifts of an average share the factors.
template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES) k_sums1d(Args a) {
  constexpr int T = 64 * WAVES;
  extern __shared__ C lds[];
  const int t = threadIdx.x, n = a.n, half = n / 2, kmax = a.kmax;
  C* tw = lds;                  // [n] e^{2 pi i m / n}
  C* xs = tw + n;               // [2][kmax + 1] the modes, shifted if `on`, and shifted
  C* pq = xs + 2 * (kmax + 1);  // [2][half + 1] (p_j, q_j)
  C* part = pq + 2 * (half + 1);  // [2][T] sums of the segments (more than one wavefront)
  // a quarter of the factors evaluated, the others by symmetry
  for (int m = t; m <= n / 4; m += T) {
    const C z = polar_pi(2.0 * (double)m / (double)n);
    tw[m] = z;
    tw[half - m] = ns::cx(-z.re, z.im);
    tw[half + m] = ns::cx(-z.re, -z.im);
    if (m > 0) tw[n - m] = ns::conj(z);
  }
  int M = 2;
  while (M <= kmax) M *= 2;
  const int segs = T / M, k = t & (M - 1), seg = t / M;
  const C* in = reinterpret_cast<const C*>(a.in) + (size_t)blockIdx.x * a.h;
  C* out = reinterpret_cast<C*>(a.out) + (size_t)blockIdx.x * a.h;
  const bool kept = k <= kmax;
  C s0 = kept ? in[k] : ns::cx(0.0, 0.0), cur = s0, sum = ns::cx(0.0, 0.0);
  const C ph = a.shifted && kept ? polar_pi(2.0 * (double)k * a.shift / (double)n) : ns::cx(1.0, 0.0);
  const int e0 = seg * k % n, ek = segs * k % n;
  const double inv_n = 1.0 / (double)n;
  int step = 0, e = 0;
  for (;;) {
    const Eval ev = a.eval[e];
    if (seg == 0 && kept) {
      C x = cur;
      if (k == 0) x.im = 0.0;  // the k = 0 coefficient of a real field is real
      const C y = ns::cmul(x, ph);
      xs[k] = ev.on ? y : x;
      xs[kmax + 1 + k] = y;
    }
    ns::exchange_barrier<WAVES == 1>();
    // v and -v^2 of one signal, or of the two of an average
    auto points = [&](auto fields) {
      constexpr int F = decltype(fields)::value;
      for (int j = t; j <= half; j += T) {
        double c[F] = {}, d[F] = {};
        int at = 0;  // (j m) mod n
#pragma unroll 4
        for (int m = 1; m <= kmax; ++m) {
          at += j;
          if (at >= n) at -= n;
          const C w = tw[at];
#pragma unroll
          for (int f = 0; f < F; ++f) {
            const C x = xs[f * (kmax + 1) + m];
            c[f] += x.re * w.re;
            d[f] += x.im * w.im;
          }
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const double x0 = xs[f * (kmax + 1)].re;
          const double u = x0 + 2.0 * (c[f] - d[f]), v = x0 + 2.0 * (c[f] + d[f]);
          pq[f * (half + 1) + j] =
              j == 0 || j == half ? ns::cx(-u * u, 0.0) : ns::cx(-u * u - v * v, v * v - u * u);
        }
      }
    };
    if (ev.pair) points(std::integral_constant<int, 2>());
    else points(std::integral_constant<int, 1>());
    ns::exchange_barrier<WAVES == 1>();
    C r[2] = {ns::cx(0.0, 0.0), ns::cx(0.0, 0.0)};
    auto modes = [&](auto fields) {
      constexpr int F = decltype(fields)::value;
      int at = e0;  // (j k) mod n
#pragma unroll 4
      for (int j = seg; j <= half; j += segs) {
        const C w = tw[at];
        at += ek;
        if (at >= n) at -= n;
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const C x = pq[f * (half + 1) + j];
          r[f].re += x.re * w.re;
          r[f].im -= x.im * w.im;
        }
      }
      for (int off = M; off < 64; off *= 2) {
#pragma unroll
        for (int f = 0; f < F; ++f) {
          r[f].re += __shfl_xor(r[f].re, off);
          r[f].im += __shfl_xor(r[f].im, off);
        }
      }
      if constexpr (WAVES > 1) {  // in one order for every segment: they keep the same state
        const int period = M > 64 ? M : 64;
#pragma unroll
        for (int f = 0; f < F; ++f) part[f * T + t] = r[f];
        __syncthreads();
#pragma unroll
        for (int f = 0; f < F; ++f) {
          r[f] = part[f * T + (t & (period - 1))];
          for (int q = period + (t & (period - 1)); q < T; q += period) r[f] = r[f] + part[f * T + q];
        }
      }
    };
    if (ev.pair) modes(std::integral_constant<int, 2>());
    else modes(std::integral_constant<int, 1>());
    C g = ns::cx(0.0, 0.0);
    if (kept) {
      g = ns::scale(ev.on ? ns::cmulc(r[0], ph) : r[0], inv_n);
      if (ev.pair) g = ns::scale(g + ns::scale(ns::cmulc(r[1], ph), inv_n), 0.5);
      if (k == 0) g.im = 0.0;  // the mean of a real field
    }
    sum = ev.b == 0.0 ? ns::cx(0.0, 0.0) : sum + ns::scale(g, ev.b);
    if (e + 1 < a.nevals) {
      cur = s0 + ns::scale(g, ev.c);
    } else {
      cur = s0 = a.nsteps > 0 ? s0 + ns::scale(sum, a.fin) : g;
      sum = ns::cx(0.0, 0.0);
    }
    if (++e == a.nevals) {
      if (++step >= a.nsteps) break;
      e = 0;
    }
  }
  if (seg == 0 && kept) out[k] = s0;
  for (int m = kmax + 1 + t; m < a.h; m += T) out[m] = a.nsteps > 0 ? in[m] : ns::cx(0.0, 0.0);
}

template <int WAVES>
void launch_sums(const Args& a, int batch, hipStream_t stream) {
  const size_t entries = (size_t)a.n + 2 * (a.kmax + 1) + 2 * (a.n / 2 + 1) + (WAVES > 1 ? 128 * WAVES : 0);
  hipLaunchKernelGGL(k_sums1d<WAVES>, dim3((unsigned)batch), dim3(64 * WAVES), entries * sizeof(C), stream, a);
}

// FFT length of signals of n > 64 points.
inline int fft_length(int n) {
  int nf = 128;
  while (nf < n) nf *= 2;
  if (nf == n) return nf;
  while (nf < 2 * n - 1) nf *= 2;
  return nf;
}

// Terms a thread of k_sums1d<waves> adds up in an evaluation.
inline int sums_terms(int n, int kmax, int waves) {
  const int points = n / 2 + 1, threads = 64 * waves;
  int m = 2;
  while (m <= kmax) m *= 2;
  return (points + threads - 1) / threads * kmax + (points * m + threads - 1) / threads;
}

// Wavefronts a signal of k_sums1d, or 0 where the transforms are better: by the terms a
// thread adds up against the transforms' length, from the length and the kept modes alone,
// so that a signal's result does not depend on its batch.  An average of two shifts costs
// the transforms one evaluation and the sums nearly two, so it has limits of its own.
// Measured on both sides of the lines, us a call, transforms / sums, one signal and 40,000
// signals, classical rk4 and (in brackets) ps_exact:
//   one wavefront: n = 126, 31 modes, 63 terms 15 / 14 and 468 / 262 (10 / 12, 269 / 178), 41
//     modes, 105 terms 15 / 18 and 469 / 420; n = 90, 29 modes, 52 terms 16 / 12, 470 / 201 (11 /
//     10, 270 / 143)
//   four, 512 points: n = 130, 64 modes, 97 terms 23 / 18, 1255 / 1003 (15 / 15, 704 / 703);
//     n = 200, 66 modes, 117 terms 24 / 22, 1252 / 1445
//   1024: n = 450, 74 modes, 187 terms 35 / 31, 3250 / 3137 (21 / 29), 112 modes, 225 terms 34 /
//     36, 3257 / 3750; n = 384, 63 modes, 112 terms (20 / 19, 1781 / 1100)
//   2048: n = 600, 98 modes, 347 terms 52 / 53, 7968 / 4933 (31 / 47); 59 modes, 194 terms (30 /
//     29, 4622 / 1739); n = 720, 118 modes, 417 terms 52 / 64
inline int sums_waves(int n, int kmax, bool pair) {
  const int nf = fft_length(n);
  if (n > 64 && nf == n) return 0;
  if (kmax < 64 && sums_terms(n, kmax, 1) <= (pair ? 54 : 70)) return 1;
  const int most = nf == 2048 ? (pair ? 200 : 350) : nf == 1024 ? (pair ? 115 : 190) : nf == 512 ? (pair ? 95 : 100) : 0;
  return kmax < 256 && sums_terms(n, kmax, 4) <= most ? 4 : 0;
}

// The evaluations of a scheme's step (classical Runge-Kutta forms; there is no linear
// term), or of a single evaluation at a->shift (scheme < 0).
inline void make_scheme(Args* a, int scheme, double dt) {
  const double hd = 0.5 * dt;
  for (Eval& e : a->eval) e = Eval{0.0, 0.0, 0, 0};
  a->nevals = 1;
  a->fin = dt;
  a->eval[0].b = 1.0;
  if (scheme < 0) {
    a->eval[0].on = a->shifted = 1;
    return;
  }
  a->shift = 0.5;
  a->shifted = scheme == EULER_PS || scheme == PS_EXACT || scheme == PS_APPROX;
  switch (scheme) {
    case EULER_PS:
      a->eval[0].pair = 1;
      break;
    case RK2:       // midpoint: S_h = S0 + dt/2 N(S0), S = S0 + dt N(S_h)
    case PS_EXACT:
      a->nevals = 2;
      a->eval[0] = Eval{hd, 0.0, scheme == PS_EXACT, 0};
      a->eval[1] = Eval{0.0, 1.0, scheme == PS_EXACT, 0};
      break;
    case PS_APPROX:  // Heun: S1 = S0 + dt N(S0; 0), S = S0 + dt/2 (N(S0; 0) + N(S1; 1/2))
      a->nevals = 2;
      a->eval[0] = Eval{dt, 1.0, 0, 0};
      a->eval[1] = Eval{0.0, 1.0, 0, 1};
      a->fin = hd;
      break;
    case RK4:
      a->nevals = 4;
      a->eval[0] = Eval{hd, 1.0, 0, 0};
      a->eval[1] = Eval{hd, 2.0, 0, 0};
      a->eval[2] = Eval{dt, 2.0, 0, 0};
      a->eval[3] = Eval{0.0, 1.0, 0, 0};
      a->fin = dt / 6.0;
      break;
    default:
      break;
  }
}

template <int NF>
void launch_nf(const Args& a, int batch, hipStream_t stream) {
  hipLaunchKernelGGL(k_model1d<NF>, dim3((unsigned)batch), dim3(threads<NF>()), 0, stream, a);
}

inline void launch(const Args& a, int batch, hipStream_t stream) {
  if (a.n <= 32) {
    hipLaunchKernelGGL(k_direct1d, dim3((unsigned)batch), dim3(64), 0, stream, a);
    return;
  }
  bool pair = false;
  for (int e = 0; e < a.nevals; ++e) pair = pair || a.eval[e].pair != 0;
  switch (sums_waves(a.n, a.kmax, pair)) {
    case 1: launch_sums<1>(a, batch, stream); return;
    case 4: launch_sums<4>(a, batch, stream); return;
    default: break;
  }
  switch (fft_length(a.n)) {
    case 128: launch_nf<128>(a, batch, stream); break;
    case 256: launch_nf<256>(a, batch, stream); break;
    case 512: launch_nf<512>(a, batch, stream); break;
    case 1024: launch_nf<1024>(a, batch, stream); break;
    default: launch_nf<2048>(a, batch, stream); break;
  }
}

}  // namespace ns1d
