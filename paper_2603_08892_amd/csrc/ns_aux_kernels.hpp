// ns_aux_kernels.hpp -- FP64 spectra reduction and the large-scale forcing draw (gfx950).
#pragma once

#include "ns_kernels.hpp"
#include "ns_aux_types.hpp"

namespace ns {

// LDS bins of one wavefront of k_spectra: E, D(, T) by shell, E by |k_x| and by |k_y|, the
// lanes' E by k_z, E at k_z = N/2, and the five totals.
__host__ __device__ constexpr int spectra_wave_bins(int n, int nsh, bool nh) {
  return (nh ? 3 : 2) * nsh + 2 * (n / 2 + 1) + 64 + 6;
}

// Shell of an integer |k|^2 < 2^24 (exact in FP32): smallest n with n(n+1) >= k^2, i.e.
// n(n-1) < k^2 <= n(n+1).
__device__ __forceinline__ int shell_small(int k2) {
  int r = (int)sqrtf((float)k2);
  r -= r * r > k2;
  r += (r + 1) * (r + 1) <= k2;
  return r * (r + 1) >= k2 ? r : r + 1;
}

// Bin layout of one partial: [0, nsh) E, [nsh, 2nsh) D, [2nsh, 3nsh) T,
// then 3 x h one-dimensional energies, then totals E, eps, H, T, nonfinite.
//
// Pass 1.  The rows (k_x, k_y) = (+-a, +-b) and (+-b, +-a) share k_x^2 + k_y^2, so every
// k_z of theirs lies in the same shell: a wavefront takes one pair a <= b and one chunk of
// 64 k_z (lanes along k_z), adds its up to eight rows lane by lane, and sorts the sums
// into shells once.  Along a row the shell index does not decrease with k_z, so a
// segmented shuffle scan leaves each shell's sum over the 64 lanes in the segment's
// last lane, which adds it to the wavefront's bin in LDS.  The k_z energy stays in the
// lane's register (a wavefront keeps one chunk), the row totals go to their k_x and k_y
// bins, and the k_z = N/2 entries of the rows are taken by eight lanes together.  Every
// sum has a fixed order (pairs in a grid-stride loop, then wavefronts, then blocks), so
// the spectra are reproducible bit for bit.
//
// Bound by the reads (every entry of the state is read, also outside the truncation, for
// the count of non-finite ones).  With a scan and a set of bin updates per row, and a
// chunk of one lane for k_z = N/2, it was bound by those LDS operations: a call with a
// transfer field took 689 us at 384^3 FP32 (1.36 GB), now 305 us, 4.5 TB/s; 512^3 2309 -> 710
// us, 256^3 FP64 261 -> 195 us; a plain copy reaches 4.9 to 6 TB/s.  Up to 96^3 a call is its
// launches and the wait, about 40 us either way.
//
// Threads of a block at most: the four rows of two FP64 fields that a lane loads together (24
// loads of 16 bytes, 96 registers) and what it works with take more than the 128 registers a
// block of 1024 threads leaves.
template <typename R, bool NH>
constexpr int spectra_threads() { return NH && sizeof(R) == 8 ? 512 : 1024; }
template <typename R, bool NH>
__global__ void __launch_bounds__((spectra_threads<R, NH>()))
k_spectra(const Cx<R>* __restrict__ u, const Cx<R>* __restrict__ nh, double nu, int n, int h,
          int nsh, long long comp, int nchunks, double* __restrict__ partials) {
  extern __shared__ double bins_all[];
  constexpr int KIND = NH ? 3 : 2;         // shell spectra with bins here
  const int nw = spectra_wave_bins(n, nsh, NH);  // bins of a wavefront
  const int lane = threadIdx.x & 63, nwb = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* bins = bins_all + wave * nw;     // E, D(, T) by shell, E by |k_x|, by |k_y|
  const int bx = KIND * nsh, by = bx + h, bz = by + h, bt = bz + 64;
  for (int t = threadIdx.x; t < nwb * nw; t += blockDim.x) bins_all[t] = 0.0;
  __syncthreads();
  const int half = n / 2;
  const int npairs = (half + 1) * (half + 2) / 2;
  const int w0 = blockIdx.x * nwb + wave, nwaves = gridDim.x * nwb;  // nwaves is a multiple of nchunks
  const int chunk = w0 % nchunks, kz = chunk * 64 + lane;
  const bool in = kz < half;
  const double wz = kz == 0 ? 1.0 : 2.0;
  double tE = 0, tD = 0, tH = 0, tT = 0, ez = 0;
  unsigned bad = 0;
  // energy 1/2 w |u|^2, transfer and helicity of one entry; zero if it is not finite
  // helicity density: with u = a + i b, Re(conj(u).(i k x u)) = 2 k.(a x b), so
  // 1/2 w Re(conj(u).omega) = w k.(a x b)
  auto entry = [&](const Cx<R>* a, const Cx<R>* b, double w, double kx, double ky, double kzd, double& e, double& t) {
    const double ar[3] = {(double)a[0].re, (double)a[1].re, (double)a[2].re};
    const double ai[3] = {(double)a[0].im, (double)a[1].im, (double)a[2].im};
    bool fin = true;
#pragma unroll
    for (int c = 0; c < 3; ++c) fin = fin && isfinite(a[c].re) && isfinite(a[c].im);
    double tt = 0.0;
    if constexpr (NH) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        fin = fin && isfinite(b[c].re) && isfinite(b[c].im);
        tt += ar[c] * (double)b[c].re + ai[c] * (double)b[c].im;
      }
    }
    if (!fin) {
      ++bad;
      return;
    }
    e += 0.5 * w * (ar[0] * ar[0] + ai[0] * ai[0] + ar[1] * ar[1] + ai[1] * ai[1] + ar[2] * ar[2] + ai[2] * ai[2]);
    t += w * tt;
    const double cxr = ar[1] * ai[2] - ar[2] * ai[1];
    const double cyr = ar[2] * ai[0] - ar[0] * ai[2];
    const double czr = ar[0] * ai[1] - ar[1] * ai[0];
    tH += w * (kx * cxr + ky * cyr + kzd * czr);
  };
  for (int p = w0 / nchunks; p < npairs; p += nwaves / nchunks) {
    int b = (int)((sqrtf(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);  // b (b + 1) / 2 <= p, corrected below
    while (b * (b + 1) / 2 > p) --b;
    while ((b + 1) * (b + 2) / 2 <= p) ++b;
    b = __builtin_amdgcn_readfirstlane(b);
    const int a = p - b * (b + 1) / 2;                  // a <= b
    const int na = (a == 0 || a == half) ? 1 : 2, nb = (b == 0 || b == half) ? 1 : 2;
    double e2[2] = {0.0, 0.0}, t = 0.0, n2[2] = {0.0, 0.0}, tn = 0.0;
    const int q = a * a + b * b;
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if (g == 1 && a == b) break;
      const int ka = g ? b : a, kb = g ? a : b, ca = g ? nb : na, cb = g ? na : nb;
      Cx<R> va[4][3], vb[4][3];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int sx = r >> 1, sy = r & 1;
        if (sx >= ca || sy >= cb) continue;
        // the index of -k (k = N/2 has the one index N/2)
        const int xi = sx ? n - ka : ka, yi = sy ? n - kb : kb;
        const long long row = ((long long)xi * n + yi) * h;
        const long long idx = row + (in ? kz : 0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          va[r][c] = u[c * comp + idx];
          if constexpr (NH) vb[r][c] = nh[c * comp + idx];
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int sx = r >> 1, sy = r & 1;
        if (sx >= ca || sy >= cb) continue;
        const double kx = (sx || ka == half) ? -(double)ka : (double)ka;
        const double ky = (sy || kb == half) ? -(double)kb : (double)kb;
        if (in) entry(va[r], vb[r], wz, kx, ky, (double)kz, e2[g], t);
      }
    }
    if (chunk == nchunks - 1) {
      // the k_z = N/2 entries: lanes 0..3 the rows of the first group, 4..7 of the second
      const int g = lane >> 2, sx = (lane >> 1) & 1, sy = lane & 1;
      const int ka = g ? b : a, kb = g ? a : b, ca = g ? nb : na, cb = g ? na : nb;
      if (lane < 8 && sx < ca && sy < cb && !(g == 1 && a == b)) {
        const int xi = sx ? n - ka : ka, yi = sy ? n - kb : kb;
        const long long idx = ((long long)xi * n + yi) * h + half;
        Cx<R> va[3], vb[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          va[c] = u[c * comp + idx];
          if constexpr (NH) vb[c] = nh[c * comp + idx];
        }
        const double kx = (sx || ka == half) ? -(double)ka : (double)ka;
        const double ky = (sy || kb == half) ? -(double)kb : (double)kb;
        entry(va, vb, 1.0, kx, ky, (double)half, n2[g], tn);
      }
    }
    double e = e2[0] + e2[1];
    ez += e;
    const int k2 = q + kz * kz;
    double d = 2.0 * nu * (double)k2 * e;
    tE += e;
    tD += d;
    tT += t;
    // row totals: group 0 has |k_x| = a, |k_y| = b, group 1 the other way round
    double r0 = e2[0] + n2[0], r1 = e2[1] + n2[1];
    // a chunk whose contributions are all zero changes no bin
    if (__ballot(r0 != 0.0 || r1 != 0.0 || t != 0.0 || tn != 0.0) == 0) continue;
    for (int off = 32; off > 0; off >>= 1) {
      r0 += __shfl_down(r0, off);
      r1 += __shfl_down(r1, off);
    }
    if (lane == 0) {
      bins[bx + a] += r0;
      bins[by + b] += r0;
      bins[bx + b] += r1;
      bins[by + a] += r1;
    }
    if (chunk == nchunks - 1) {
      double en = n2[0] + n2[1];
      for (int off = 4; off > 0; off >>= 1) {
        en += __shfl_down(en, off);
        if constexpr (NH) tn += __shfl_down(tn, off);
      }
      if (lane == 0) {
        const int k2n = q + half * half, sn = shell_small(k2n);
        const double dn = 2.0 * nu * (double)k2n * en;
        bins[sn] += en;
        bins[nsh + sn] += dn;
        if constexpr (NH) bins[2 * nsh + sn] += tn;
        bins[bt] += en;  // E_z at N/2
        tE += en;
        tD += dn;
        tT += tn;
      }
    }
    // segmented inclusive scan over the lanes (keys s non-decreasing with the lane; lanes
    // past the row end carry a key above every shell and zeros)
    const int s = in ? shell_small(k2) : 0x7fffffff;
    for (int off = 1; off < 64; off <<= 1) {
      const double eu = __shfl_up(e, off), du = __shfl_up(d, off);
      const int su = __shfl_up(s, off);
      double tu = 0.0;
      if constexpr (NH) tu = __shfl_up(t, off);
      if (lane >= off && su == s) {
        e += eu;
        d += du;
        t += tu;
      }
    }
    const int sn = __shfl_down(s, 1);
    if (in && (lane == 63 || sn != s)) {
      bins[s] += e;
      bins[nsh + s] += d;
      if constexpr (NH) bins[2 * nsh + s] += t;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    tE += __shfl_down(tE, off);
    tD += __shfl_down(tD, off);
    tH += __shfl_down(tH, off);
    tT += __shfl_down(tT, off);
    bad += __shfl_down(bad, off);
  }
  bins[bz + lane] = ez;
  if (lane == 0) {
    bins[bt + 1] = tE;
    bins[bt + 2] = tD;
    bins[bt + 3] = tH;
    bins[bt + 4] = tT;
    bins[bt + 5] = (double)bad;
  }
  __syncthreads();
  // the block's partial, in the common layout; E_z of chunk c from the wavefronts that keep it
  const int nb_out = 3 * nsh + 3 * h + 5;
  double* out = partials + (long long)blockIdx.x * nb_out;
  for (int t = threadIdx.x; t < nb_out; t += blockDim.x) {
    const int y = t - 3 * nsh, z = y - 2 * h, tot = y - 3 * h;
    double acc = 0.0;
    if (z >= 0 && tot < 0 && z < half) {
      for (int w = 0; w < nwb; ++w)
        if ((blockIdx.x * nwb + w) % nchunks == z / 64) acc += bins_all[w * nw + bz + z % 64];
    } else if (y >= 0 || t < KIND * nsh) {
      const int from = y < 0 ? t : (tot >= 0 ? bt + 1 + tot : (z >= 0 ? bt : bx + y));
      for (int w = 0; w < nwb; ++w) acc += bins_all[w * nw + from];
    }
    out[t] = acc;
  }
}

// Pass 2: fixed-order sum over the blocks' partials.  Eight bins per block of 256
// threads; the 32 lanes of a bin sum the partials b = lane, lane + 32, ... in
// order, then a fixed shuffle tree combines the lanes (deterministic).
__global__ void __launch_bounds__(256)
k_spectra_sum(const double* __restrict__ partials, int nblocks, int nb, double* __restrict__ out) {
  const int bin = blockIdx.x * 8 + (threadIdx.x >> 5);
  const int lane = threadIdx.x & 31;
  double s = 0.0;
  if (bin < nb)
    for (int b = lane; b < nblocks; b += 32) s += partials[(long long)b * nb + bin];
  for (int off = 16; off > 0; off >>= 1) s += __shfl_down(s, off, 32);
  if (lane == 0 && bin < nb) out[bin] = s;
}

// ------------------------------------------------------------------ forcing
// SplitMix64 (Steele, Lea & Flood 2014) used counter-based:
// stream(seed, step) = mix(seed + G (step + 1)), draw j = mix(stream + G (j + 1)),
// uniform = (draw >> 11) 2^-53; Box-Muller on pairs (u1, u2).
__device__ __forceinline__ uint64_t sm64_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ double sm64_uniform(uint64_t seed, long long step, long long j) {
  const uint64_t G = 0x9E3779B97F4A7C15ull;
  const uint64_t s = sm64_mix(seed + G * (uint64_t)(step + 1));
  return (double)(sm64_mix(s + G * (uint64_t)(j + 1)) >> 11) * (1.0 / 9007199254740992.0);
}

// Forced modes 4 <= |k|^2 <= 9 in draw order (k_z 0..3, then k_x, k_y from -3 to 3;
// on k_z = 0 only k_x > 0, or k_x = 0 and k_y > 0): 48 independent modes, listed at
// compile time.
struct ForcingModes {
  int k[48][3];
};
constexpr ForcingModes make_forcing_modes() {
  ForcingModes m{};
  int c = 0;
  for (int z = 0; z <= 3; ++z)
    for (int x = -3; x <= 3; ++x)
      for (int y = -3; y <= 3; ++y) {
        const int k2 = x * x + y * y + z * z;
        if (k2 < 4 || k2 > 9) continue;
        if (z == 0 && !(x > 0 || (x == 0 && y > 0))) continue;
        m.k[c][0] = x;
        m.k[c][1] = y;
        m.k[c][2] = z;
        ++c;
      }
  return m;
}
__device__ __forceinline__ void forcing_mode(int i, int* kx, int* ky, int* kz) {
  constexpr ForcingModes m = make_forcing_modes();
  static_assert(m.k[47][2] == 3 && m.k[0][2] == 0, "48 forced modes");
  *kx = m.k[i][0];
  *ky = m.k[i][1];
  *kz = m.k[i][2];
}

// One block of 192 threads: draw g for `step` (thread 3 i + c the Gaussian pair of
// mode i, component c), project it, scale it to inject energy at rate `inj` over a
// step dt from state u, write the dense table force[c][k_x+3][k_y+3][k_z] (k_z <= 3)
// and the FP64 record fs.
template <typename R>
__global__ void __launch_bounds__(192)
k_forcing(const Cx<R>* __restrict__ u, Lay lu, Cx<R>* __restrict__ force, ForceState* __restrict__ fs, int n,
          uint64_t seed, long long step, double dt, double inj) {
  __shared__ double gre[48][3], gim[48][3], pb[48], pg[48];
  __shared__ double amp;
  const int q = threadIdx.x;
  for (int t = q; t < 3 * 196; t += blockDim.x) force[t] = cx(R(0), R(0));
  if (q < 144) {
    const long long p = q;  // = 3 i + c
    const double u1 = sm64_uniform(seed, step, 2 * p);
    const double u2 = sm64_uniform(seed, step, 2 * p + 1);
    const double r = sqrt(-2.0 * log(1.0 - u1));
    double sn, cs;
    sincospi(2.0 * u2, &sn, &cs);
    gre[q / 3][q % 3] = r * cs;
    gim[q / 3][q % 3] = r * sn;
  }
  __syncthreads();
  if (q < 48) {
    const int i = q;
    int kx, ky, kz;
    forcing_mode(i, &kx, &ky, &kz);
    double vr[3], vi[3];
    for (int c = 0; c < 3; ++c) {
      vr[c] = gre[i][c];
      vi[c] = gim[i][c];
    }
    const double k2 = (double)(kx * kx + ky * ky + kz * kz);
    const double dr = (kx * vr[0] + ky * vr[1] + kz * vr[2]) / k2;
    const double di = (kx * vi[0] + ky * vi[1] + kz * vi[2]) / k2;
    vr[0] -= kx * dr; vr[1] -= ky * dr; vr[2] -= kz * dr;
    vi[0] -= kx * di; vi[1] -= ky * di; vi[2] -= kz * di;
    // B and G contributions of the stored half-spectrum entries of this mode
    const long long idx = lay_at(lu, (kx + n) % n, (ky + n) % n, kz, n);
    double b = 0, g2 = 0;
    const double w = (kz == 0) ? 1.0 : 2.0;
    for (int c = 0; c < 3; ++c) {
      const Cx<R> a = u[c * lu.cs + idx];
      b += w * ((double)a.re * vr[c] + (double)a.im * vi[c]);
      g2 += w * (vr[c] * vr[c] + vi[c] * vi[c]);
    }
    if (kz == 0) {  // the partner -k holds conj(g)
      const long long idp = lay_at(lu, (-kx + n) % n, (-ky + n) % n, 0, n);
      for (int c = 0; c < 3; ++c) {
        const Cx<R> a = u[c * lu.cs + idp];
        b += (double)a.re * vr[c] - (double)a.im * vi[c];
        g2 += vr[c] * vr[c] + vi[c] * vi[c];
      }
    }
    for (int c = 0; c < 3; ++c) {
      gre[i][c] = vr[c];
      gim[i][c] = vi[c];
      fs->g[i][c][0] = vr[c];
      fs->g[i][c][1] = vi[c];
    }
    pb[i] = b;
    pg[i] = g2;
  }
  __syncthreads();
  if (q == 0) {
    double B = 0, G = 0;
    for (int m = 0; m < 48; ++m) { B += pb[m]; G += pg[m]; }
    const double r = sqrt(B * B + 2.0 * dt * G * inj);
    amp = 2.0 * inj / (B + r);
    fs->amp = amp;
    fs->B = B;
    fs->G = G;
    fs->r = r;
    fs->injected = dt * (amp * B + 0.5 * amp * amp * dt * G);
  }
  __syncthreads();
  if (q < 144) {
    const int i = q / 3, c = q % 3;
    int kx, ky, kz;
    forcing_mode(i, &kx, &ky, &kz);
    const double re = amp * gre[i][c], im = amp * gim[i][c];
    force[c * 196 + ((kx + 3) * 7 + (ky + 3)) * 4 + kz] = cx(R(re), R(im));
    if (kz == 0) force[c * 196 + ((-kx + 3) * 7 + (-ky + 3)) * 4] = cx(R(re), R(-im));
  }
}

// ------------------------------------------------------------------ forced step adjoint
// The forcing O = a(u0) g depends on the state through B = <u0, g> (the
// amplitude solves a B + a^2 dt/2 G = inj), with da/dB = -a/r.  With
// mu_O = (dS_new/dO)^T lam = dt (E_h lam + E_dt mu1) for the Heun step (mu1 the
// adjoint of the first stage), the step adjoint gains (da/dB) <mu_O, g> g.
// k_forcing_adj_dot (one block, before lam is overwritten) forms the scalar
// (da/dB) <mu_O, g> over the 96 forced full-grid modes (Parseval weights: 2 off
// the k_z = 0 plane, 1 on it, where both k and -k are stored); k_forcing_adj_add
// adds it times g to the result.
template <typename R>
__global__ void __launch_bounds__(64)
k_forcing_adj_dot(const Cx<R>* __restrict__ lam, Lay ll, const Cx<R>* __restrict__ mu1, Lay lm,
                  const R* __restrict__ eh, const R* __restrict__ edt, ForceState* __restrict__ fs, int n,
                  double dt) {
  __shared__ double part[64];
  const int i = threadIdx.x;
  double acc = 0.0;
  if (i < 48) {
    int kx, ky, kz;
    forcing_mode(i, &kx, &ky, &kz);
    const int k2 = kx * kx + ky * ky + kz * kz;
    const double fh = (double)eh[k2], fd = (double)edt[k2];
    for (int side = 0; side < (kz == 0 ? 2 : 1); ++side) {
      const int sx = side ? -kx : kx, sy = side ? -ky : ky;
      const int xi = (sx + n) % n, yi = (sy + n) % n;
      const double w = (kz == 0) ? 1.0 : 2.0;
      for (int c = 0; c < 3; ++c) {
        const Cx<R> l = lam[c * ll.cs + lay_at(ll, xi, yi, kz, n)];
        const Cx<R> m = mu1[c * lm.cs + lay_at(lm, xi, yi, kz, n)];
        const double mre = dt * (fh * (double)l.re + fd * (double)m.re);
        const double mim = dt * (fh * (double)l.im + fd * (double)m.im);
        const double gre = fs->g[i][c][0], gim = side ? -fs->g[i][c][1] : fs->g[i][c][1];
        acc += w * (mre * gre + mim * gim);
      }
    }
  }
  part[i] = acc;
  __syncthreads();
  if (i == 0) {
    double t = 0.0;
    for (int m = 0; m < 48; ++m) t += part[m];
    fs->dot = -(fs->amp / fs->r) * t;
  }
}

template <typename R>
__global__ void __launch_bounds__(64)
k_forcing_adj_add(Cx<R>* __restrict__ lam, Lay ll, const ForceState* __restrict__ fs, int n) {
  const int i = threadIdx.x;
  if (i >= 48) return;
  int kx, ky, kz;
  forcing_mode(i, &kx, &ky, &kz);
  const double s = fs->dot;
  for (int side = 0; side < (kz == 0 ? 2 : 1); ++side) {
    const int sx = side ? -kx : kx, sy = side ? -ky : ky;
    const int xi = (sx + n) % n, yi = (sy + n) % n;
    for (int c = 0; c < 3; ++c) {
      const long long o = c * ll.cs + lay_at(ll, xi, yi, kz, n);
      const double gre = fs->g[i][c][0], gim = side ? -fs->g[i][c][1] : fs->g[i][c][1];
      const Cx<R> v = lam[o];
      lam[o] = cx(R((double)v.re + s * gre), R((double)v.im + s * gim));
    }
  }
}

// ------------------------------------------------------------------ energy budget
// Pass 1: E = 1/2 sum w |u|^2 and eps = nu sum w |k|^2 |u|^2 over the retained
// modes of a state (any layout; entries outside the retained set are ignored),
// per block in a fixed order: every wavefront takes whole (k_x, k_y) rows in a
// grid-stride loop (rows whose k_z = 0 mode is not retained hold no retained mode
// and are skipped), lanes along k_z < kzn; a shuffle tree per wavefront, then the
// wavefronts in order.
constexpr int kBudgetBlocks = 1024;
template <typename R>
__global__ void __launch_bounds__(256)
k_budget_partial(const Cx<R>* __restrict__ u, Lay lu, Geom g, double nu, double* __restrict__ partials) {
  __shared__ double we[4], wd[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nrows = g.n * g.n, nwaves = gridDim.x * 4;
  double e = 0.0, d = 0.0;
  for (int row = blockIdx.x * 4 + wave; row < nrows; row += nwaves) {
    const int xi = row / g.n, yi = row - xi * g.n;
    const int kx = kval(xi, g.n), ky = kval(yi, g.n);
    if (!retained(g, kx, ky, 0)) continue;  // the same for the whole wavefront
    const long long base = lay_at(lu, xi, yi, 0, g.n);
    for (int kz = lane; kz < g.kzn; kz += 64) {
      if (!retained(g, kx, ky, kz)) continue;
      const double w = (kz == 0 || 2 * kz == g.n) ? 1.0 : 2.0;
      double m2 = 0.0;
      for (int c = 0; c < 3; ++c) {
        const Cx<R> a = u[c * lu.cs + base + kz];
        m2 += (double)a.re * (double)a.re + (double)a.im * (double)a.im;
      }
      const double em = 0.5 * w * m2;
      e += em;
      d += 2.0 * nu * (double)((long long)kx * kx + (long long)ky * ky + (long long)kz * kz) * em;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    e += __shfl_down(e, off);
    d += __shfl_down(d, off);
  }
  if (lane == 0) {
    we[wave] = e;
    wd[wave] = d;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = ((we[0] + we[1]) + we[2]) + we[3];
    partials[2 * blockIdx.x + 1] = ((wd[0] + wd[1]) + wd[2]) + wd[3];
  }
}

// Pass 2 (one wavefront): sum the partials in a fixed order and update the
// record.  dt == 0 starts the budget at this state.  forced: add the injected
// energy of the step from the forcing record.
__global__ void __launch_bounds__(64)
k_budget_step(const double* __restrict__ partials, int nblocks, Budget* __restrict__ b,
              const ForceState* __restrict__ fs, double dt, int forced) {
  const int lane = threadIdx.x;
  double e = 0.0, d = 0.0;
  for (int k = lane; k < nblocks; k += 64) {
    e += partials[2 * k];
    d += partials[2 * k + 1];
  }
  for (int off = 32; off > 0; off >>= 1) {
    e += __shfl_down(e, off);
    d += __shfl_down(d, off);
  }
  if (lane != 0) return;
  if (dt == 0.0) {
    b->t = 0.0;
    b->E0 = e;
    b->int_eps = 0.0;
    b->int_p = 0.0;
    b->p_last = 0.0;
  } else {
    b->t += dt;
    b->int_eps += 0.5 * dt * (b->eps + d);
    const double inj = forced ? fs->injected : 0.0;
    b->int_p += inj;
    b->p_last = inj / dt;
  }
  b->E = e;
  b->eps = d;
  b->residual = e - b->E0 + b->int_eps - b->int_p;
}

}  // namespace ns
