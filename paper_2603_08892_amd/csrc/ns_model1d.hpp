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
// A call is bound by latency: a chain of dependent transforms of 16 to 2048 points on
// one CU, whose time is that of one wavefront's instructions and LDS round trips.  So a
// step is one loop over its evaluations with one copy of each transform in the code,
// plans of 4 to 8 points a thread with every index known at compile time, and lines of
// up to 256 points inside one wavefront.  Up to 64 points direct sums with every factor
// in registers are shorter than either (k_direct1d).  Against the kernel before (direct
// O(n k_max) sums from LDS), 8 signals, one call of one step, launch included: rk4 at n =
// 22 11.6 -> 9.3 us, 62 24.8 -> 18 us, 128 42.9 -> 10.7 us, 256 84.6 -> 10.2 us, 302 134.7 ->
// 34.3 us, 1018 891 -> 53 us, 1024 919 -> 18.9 us.  Mixed-radix stages with the plan as an
// argument took 24.4 us at 256 and 31.8 us at 1024 (index arithmetic on the one chain).
#pragma once

#include <hip/hip_runtime.h>

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

// n <= J (32 or 64): direct sums with every factor in registers.  Thread j of group g
// (g = 0: unshifted, 1: shifted; both groups keep the state) holds cos and sin of
// 2 pi j m / n for 1 <= m < n/2, which serve v_j = S_0 + 2 sum_m Re(S_m e^{i ..}) and, m and
// n - m taken together, F_j = w_0 + (-1)^j w_{n/2} + sum_m ((w_m + w_{n-m}) cos - i (w_m -
// w_{n-m}) sin); the other operands are LDS broadcasts.
template <int J>
__global__ void __launch_bounds__(2 * J) k_direct1d(Args a) {
  constexpr int M = J / 2;
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

// FFT length of signals of n > 64 points.
inline int fft_length(int n) {
  int nf = 128;
  while (nf < n) nf *= 2;
  if (nf == n) return nf;
  while (nf < 2 * n - 1) nf *= 2;
  return nf;
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
    hipLaunchKernelGGL(k_direct1d<32>, dim3((unsigned)batch), dim3(64), 0, stream, a);
    return;
  }
  if (a.n <= 64) {
    hipLaunchKernelGGL(k_direct1d<64>, dim3((unsigned)batch), dim3(128), 0, stream, a);
    return;
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
