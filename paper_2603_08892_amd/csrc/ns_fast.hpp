// ns_fast.hpp -- compile-time specialised passes (gfx950): every grid size from 16 to 512 in
// FP32 and FP64; the plans of thirteen FP32 sizes are below, the others in ns_size_plans.hpp.
//
// Same scratch layout, tile list and pass semantics as the generic kernels of
// ns_kernels.hpp, except that in the step sequences the x-inverse passes store
// the five transforms they compute and the y-inverse pass (f_ycurl) forms the
// vorticity from them; the transforms run on registers (fft_reg.hpp) with one LDS
// exchange per radix boundary instead of one LDS round trip per stage, and all
// indices are compile-time except the thread and block coordinates.
//
// Strided passes (x, y): a block is one tile of L contiguous k_z columns (16 in FP32, 8
// in FP64: 128-byte rows);
// thread (l, t) = (tid mod L, tid div L) handles column l, points of the line
// owned by t.  LDS: the exchange buffer [position][column] (row pitch L + 1 to
// spread banks) and the twiddle table.
// Contiguous pass (z): a block holds P lines, thread (p, t) = (tid div TPL, tid mod TPL);
// TPL divides 64 and a line's threads synchronise at wavefront scope.
// In the step sequences the x-forward kernel can also run the next evaluation's
// x-inverse pass on its tile (template argument FEED), so a chained evaluation is
// four launches: y-inverse, z, y-forward, x-forward (+ next x-inverse).
#pragma once

#include "fft_reg.hpp"
#include "ns_kernels.hpp"

namespace ns {

// k_z columns of a tile of the strided passes: one 128-byte row of the scratch fields
template <typename T>
constexpr int tile_cols() { return 128 / (2 * (int)sizeof(T)); }

// Addressing: a block-uniform base pointer (a state component or scratch field)
// plus a per-lane 32-bit element offset.  Every offset stays inside one component
// of at most N^2 (N/2 + 1) elements, and the specialised sizes keep the bytes of
// that below 2^32 (LinePlan checks it), so the byte offset fits 32 bits, the base
// stays in scalar registers and the index arithmetic is 32-bit.
template <typename T>
__device__ __forceinline__ Cx<T> ld_off(const Cx<T>* __restrict__ base, uint32_t off) {
  return *reinterpret_cast<const Cx<T>*>(reinterpret_cast<const char*>(base) + off * (uint32_t)sizeof(Cx<T>));
}
// STREAM: a non-temporal store, for the scratch fields and the compact stage
// buffers of the grids whose step works on far more than the 256 MB last-level
// cache (stream_stores): each pass's output is read back only by the next pass,
// mostly on other XCDs, so keeping it in cache buys nothing.  Measured per step
// (PS-RK2 random, RK4 at 512): 3-11% faster at N = 240...512, 256 gaining least;
// at N <= 216 much of a step's data is still found in that cache and the step
// was 5-17% slower.  Outputs in the
// caller's layout (rows of N/2 + 1 elements, not whole 128-byte lines) take
// plain stores: streamed partial lines made those passes 1.5 times slower.
template <typename T>
constexpr bool stream_stores(int n) { return (long long)n * n * n * (int)sizeof(Cx<T>) >= 8ll * 240 * 240 * 240; }
template <bool STREAM = false, typename T>
__device__ __forceinline__ void st_off(Cx<T>* __restrict__ base, uint32_t off, Cx<T> v) {
  char* p = reinterpret_cast<char*>(base) + off * (uint32_t)sizeof(Cx<T>);
  if constexpr (STREAM) {
    typedef T v2 __attribute__((ext_vector_type(2)));
    const v2 w = {v.re, v.im};
    __builtin_nontemporal_store(w, reinterpret_cast<v2*>(p));
  } else {
    *reinterpret_cast<Cx<T>*>(p) = v;
  }
}

// Branch-free masked load: the offset is clamped to element 0 of the (valid)
// base when `ok` is false and the value multiplied by 0 (the arrays hold finite
// values), so the load is unconditional and a thread issues all of its loads back
// to back before the first use (a select would let the compiler turn the load
// back into a branch with a wait right behind it).
template <typename T>
__device__ __forceinline__ Cx<T> ld_masked(const Cx<T>* __restrict__ base, uint32_t off, bool ok) {
  const Cx<T> v = ld_off(base, ok ? off : 0u);
  const T m = ok ? T(1) : T(0);
  return cx(v.re * m, v.im * m);
}

// Masked loads through a buffer descriptor: an offset past its end reads zero without
// touching memory, so a masked element costs a select on the offset and no arithmetic,
// and every load of a thread can be issued before the first use.
using BufDesc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ BufDesc buf_desc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
template <typename T>
__device__ __forceinline__ Cx<T> ld_buf(BufDesc b, uint32_t off, bool ok) {
  const uint32_t byte = ok ? off * (uint32_t)sizeof(Cx<T>) : 0x80000000u;  // fields are below 2 GiB (TypedPlan)
  Cx<T> v;
  if constexpr (sizeof(T) == 4) {
    const auto w = __builtin_amdgcn_raw_buffer_load_b64(b, (int)byte, 0, 0);
    __builtin_memcpy(&v, &w, sizeof(v));
  } else {
    const auto w = __builtin_amdgcn_raw_buffer_load_b128(b, (int)byte, 0, 0);
    __builtin_memcpy(&v, &w, sizeof(v));
  }
  return v;
}

// Truncation test along one k_x line (fixed k_y, k_z) in 32-bit arithmetic
// (|k_i| <= N/2 <= 256 here, so |k|^2 < 2^18): every mask is k_x^2 <= hi2 and
// |k_x| <= xmax with per-line thresholds (xmax from the pair conditions of
// double_alias_free).
struct LineTest {
  int hi2, xmax;
  __device__ __forceinline__ bool operator()(int kx) const {
    // evaluated without short-circuit branches, so masked loads stay unconditional
    return (kx * kx <= hi2) & (abs(kx) <= xmax);
  }
};
__device__ __forceinline__ LineTest line_test(const Geom& g, int ky, int kz) {
  LineTest L{0, g.n};
  if (cube_family(g)) L.hi2 = (abs(ky) <= g.kmax && kz <= g.kmax) ? g.kmax * g.kmax : -1;
  else L.hi2 = (int)g.k2max - ky * ky - kz * kz;
  if (g.mask >= 2) {
    // 3 (|k_x| + |k_y|) < 2N, 3 (|k_x| + |k_z|) < 2N and 3 (|k_y| + |k_z|) < 2N
    const int b = abs(ky), c = abs(kz), n2 = 2 * g.n;
    L.xmax = (3 * (b + c) < n2) ? (n2 - 1) / 3 - max(b, c) : -1;
  }
  return L;
}

// Shift factors of the block's k_z columns on row k_y (FP64, rounded once per
// axis like phase1), computed by one thread a column into LDS.
template <typename T>
__device__ __forceinline__ void phase_cols(Cx<T>* phc, int ky, int kz0, const Shift& sh, int n, int tid) {
  if (tid < tile_cols<T>()) phc[tid] = cmul(phase1<T>(ky, sh.s[1], n), phase1<T>(kz0 + tid, sh.s[2], n));
}

// One line plan: N points over TPL threads, inverse and forward radix lists;
// LinePlan for FP32 fields, LinePlanD for FP64 ones.  L: columns of a tile, LP: its
// pitch in LDS (one more, to spread the banks).
template <typename T_, int N_, int TPL_, typename Inv_, typename Fwd_>
struct TypedPlan {
  using T = T_;
  static constexpr int N = N_;
  static constexpr int TPL = TPL_;
  static constexpr int L = tile_cols<T>();
  static constexpr int LP = L + 1;
  // (k_z pitch of a scratch field: at most N/2 rounded up to the tile; one tile of padding a plane)
  static_assert((unsigned long long)sizeof(Cx<T>) * N * (N * ((N / 2 + L) / L * L) + L) <= (1ull << 31),
                "32-bit byte offsets and buffer descriptors need fields of at most 2 GiB");
  static constexpr int EPT = Inv_::template ept<N_, TPL_>();
  // z passes (f_zcross): whether the twiddles stay in registers, and how many slices ahead
  // a slice is loaded.  The pass is bound by its waves per SIMD and by LDS traffic: kept
  // twiddles take a quarter of the LDS reads away, a deeper prefetch hides the loads,
  // both cost registers.  Best of the six combinations, z pass in us (twiddles kept or not /
  // slices ahead): 4 registers a transform, 256^3 kept/2 113.7, kept/1 119.9, not/2 120.1; 8
  // or 9 over 32 threads, 192^3 kept/0 43.6, kept/1 47.1, not/1 45.4 and 160^3, 216^3
  // likewise (four waves instead of three); 8 or 9 over 64, 512^3 not/1 825, kept/0 843, kept/1
  // 871 and 324^3, 384^3 likewise; others kept/1 (128^3 18.1 against 18.7 kept/0, 20.1 not/2;
  // 360^3 450 against 458 to 493; 64^3, 8 threads, kept/2 8.3 against 8.5).
  static constexpr int ZREGS = EPT * (int)sizeof(T) / 4;  // 32-bit register pairs a transform
  static constexpr bool KEEP = !(TPL == 64 && ZREGS > 4);
  static constexpr int AHEAD = ZREGS <= 4 || TPL <= 8 ? 2 : (TPL == 32 && ZREGS <= 9) ? 0 : 1;
  // x-forward passes (f_xfwd): points a chunk of stage operands, for stages with one
  // operand and with two.  Small chunks, the next one loaded while one is used, keep a
  // thread at fewer registers.  Two operands: one point a chunk (one or two at EPT over
  // 12 or 16 threads a line: a quarter) brings 512-thread tiles to 128 registers and two
  // tiles to a CU, or takes the spills away (chained RK4 stages, us, against half the
  // points a chunk: 256^3 94.1 -> 78.7, 216^3 67.8 -> 51.5, 360^3 280 -> 255, 512^3 781 -> 661).  One
  // operand: all points at once unless the plan says otherwise (XPass).
  static constexpr int CHUNK_ONE = EPT;
  static constexpr int CHUNK_TWO = TPL == 32 && EPT <= 12 ? 1 : (EPT + 3) / 4;
  static_assert(EPT == Fwd_::template ept<N_, TPL_>(), "both directions hold the same registers");
  using Inv = Inv_;   // radices of the inverse transforms
  using Fwd = Fwd_;   // radices of the forward transforms (reverse order of Inv)
};
template <int N, int TPL, typename Inv, typename Fwd>
struct LinePlan : TypedPlan<float, N, TPL, Inv, Fwd> {};
template <int N, int TPL, typename Inv, typename Fwd>
struct LinePlanD : TypedPlan<double, N, TPL, Inv, Fwd> {};
// An x plan whose one-operand stages take chunks of ONE points (TypedPlan::CHUNK_ONE).
// PS-RK2 random steps, a quarter of the points against all: 216^3 590 against 625 us, 240^3
// 758 against 800, 512^3 7.80 against 8.18 ms (fewer registers: two tiles a CU, no spills);
// at 256 and 384 1-2% slower, so those keep all.
template <typename P, int ONE>
struct XPass : P {
  static constexpr int CHUNK_ONE = ONE;
};

// Plans of the five passes of one size; PZ = lines per block of the z pass; the
// adjoint z pass (five inverse and three forward slices) may take its own plan ZA
// with PZA lines per block.  YC: the step sequences run f_xinv<XI, false> and
// f_ycurl (the vorticity formed in the y-inverse pass, five scratch fields written
// by the x-inverse passes) instead of f_xinv<XI, true> and f_ypass over six fields.
// XA: the plan of the adjoint's f_xinv and f_xadj, XL: of its f_xlam.
template <typename XI, typename YP, typename ZP, int PZ_, typename XF, typename ZA = ZP, int PZA_ = PZ_,
          typename XA = XF, typename XL = XI, bool YC_ = false>
struct FastCfg {
  static constexpr int N = XI::N;
  using T = typename XI::T;
  static constexpr bool YC = YC_;
  static constexpr int PZ = PZ_;
  static constexpr int PZA = PZA_;
  static_assert(N * N % PZ_ == 0 && N * N % PZA_ == 0, "the z passes run N^2 / P blocks of P whole lines");
  // f_xfwd runs the x-inverse pass of a chained evaluation, f_xinv that of a first one
  static_assert(std::is_base_of_v<XI, XF>, "chained and single evaluations agree bit for bit");
  using XInv = XI;
  using Y = YP;
  using Z = ZP;
  using ZAdj = ZA;
  using XFwd = XF;
  using XAdj = XA;
  using XLam = XL;
};

// ------------------------------------------------------------------ x inverse
// One active tile per block, all six fields.  Along an x line k_y and k_z are
// fixed, so the x transform of omega_x = i (k_y u_z - k_z u_y) is
// i k_y X(u_z) - i k_z X(u_y), and omega_y = i k_z u_x - i k_x u_z,
// omega_z = i k_x u_y - i k_y u_x need only D_z = X(i k_x u_z) and D_y = X(i k_x u_y)
// beside the velocity transforms: five transforms for six fields, and each state
// component is read once per tile.
// CURL = true stores the vorticity itself (fields 0..5 = u_x, u_y, u_z, omega_x,
// omega_y, omega_z), as f_ypass reads it (the transposed evaluations and the sizes
// without FastCfg::YC).  CURL = false stores the five transforms as they are: u_x,
// u_y, u_z in fields 0, 1, 2, D_z in field 4 and D_y in field 5, and leaves field
// 3 alone; f_ycurl forms the vorticity from them as it loads them, so a tile
// writes five fields here and is read as five there instead of six.
template <typename C, bool CURL>
__global__ void __launch_bounds__(C::L * C::TPL)
f_xinv(const Cx<typename C::T>* __restrict__ S, Lay ls, Cx<typename C::T>* __restrict__ W, const Cx<typename C::T>* __restrict__ twg,
        Shift sh, const int2* __restrict__ tiles, Geom g) {
  using T = typename C::T;
  constexpr int N = C::N, TPL = C::TPL, EPT = C::EPT;
  using F = RegFft<N, TPL, +1, typename C::Inv>;
  __shared__ Cx<T> tw[N];
  __shared__ Cx<T> phx[N];
  __shared__ Cx<T> phc[C::L];
  __shared__ Cx<T> xb[N * C::LP];
  const int tid = threadIdx.x;
  const int l = tid % C::L, t = tid / C::L;
  const int2 tile = tiles[blockIdx.x];
  const int yi = tile.x, kz0 = tile.y, kz = kz0 + l;
  const int ky = kval(yi, N);
  for (int i = tid; i < N; i += C::L * TPL) tw[i] = twg[i];
  const bool col = kz < g.kzn;
  Cx<T> phyz = cx(T(1), T(0));
  if (sh.on) {
    phase_row(phx, N, sh.s[0], tid, C::L * TPL);
    phase_cols(phc, ky, kz0, sh, N, tid);
    __syncthreads();
    phyz = phc[l];
  }
  const LineView<T, C::LP> lv{xb + l};
  const uint32_t sbase = (uint32_t)(yi * ls.pitch + kz0) + l, sstep = (uint32_t)(N * ls.pitch + ls.pad);
  [[maybe_unused]] const T kyf = T(ky), kzf = T(kz);
  Cx<T> ux[EPT], uy[EPT], uz[EPT], v[EPT];
  {
    bool ok[EPT];
    uint32_t idx[EPT];
    const LineTest keep = line_test(g, ky, kz);
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = F::in_at(t, i);
      ok[i] = col && F::in_ok(t, i) && keep(kval(p, N));
      idx[i] = (uint32_t)p * sstep + sbase;
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      ux[i] = ld_masked(S, idx[i], ok[i]);
      uy[i] = ld_masked(S + ls.cs, idx[i], ok[i]);
      uz[i] = ld_masked(S + 2 * ls.cs, idx[i], ok[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int p = F::in_at(t, i);
    if (sh.on) {
      const Cx<T> phi = cmul(phx[p], phyz);
      ux[i] = cmul(ux[i], phi);
      uy[i] = cmul(uy[i], phi);
      uz[i] = cmul(uz[i], phi);
    }
  }
  const uint32_t obase = (uint32_t)(yi * g.kzp + kz0) + l, ostep = (uint32_t)(N * g.kzp + g.pad);
  auto store = [&](int f, const Cx<T>* v) {
    if (col) {
#pragma unroll
      for (int i = 0; i < EPT; ++i)
        if (F::out_ok(t, i))
          st_off<stream_stores<T>(N)>(W + f * g.wcomp, (uint32_t)F::out_pos(t, i) * ostep + obase, v[i]);
    }
  };
  F::run(ux, t, lv, tw);
  store(0, ux);
#pragma unroll
  for (int i = 0; i < EPT; ++i) v[i] = mul_i(scale(uz[i], T(kval(F::in_at(t, i), N))));
  F::run(v, t, lv, tw);  // D_z
  if constexpr (CURL) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) v[i] = mul_i(scale(ux[i], kzf)) - v[i];  // omega_y
  }
  store(4, v);
#pragma unroll
  for (int i = 0; i < EPT; ++i) v[i] = mul_i(scale(uy[i], T(kval(F::in_at(t, i), N))));
  F::run(v, t, lv, tw);  // D_y
  if constexpr (CURL) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) v[i] = v[i] - mul_i(scale(ux[i], kyf));  // omega_z
  }
  store(5, v);
  F::run(uy, t, lv, tw);
  store(1, uy);
  F::run(uz, t, lv, tw);
  store(2, uz);
  if constexpr (CURL) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) uy[i] = mul_i(scale(uz[i], kyf) - scale(uy[i], kzf));  // omega_x
    store(3, uy);
  }
}

// ------------------------------------------------------------------ y passes (in place)
template <typename C, int S>
__global__ void __launch_bounds__(C::L * C::TPL)
f_ypass(Cx<typename C::T>* __restrict__ W, const Cx<typename C::T>* __restrict__ twg, int ntz, Geom g) {
  using T = typename C::T;
  constexpr int N = C::N, TPL = C::TPL, EPT = C::EPT;
  using F = RegFft<N, TPL, S, std::conditional_t<(S > 0), typename C::Inv, typename C::Fwd>>;
  __shared__ Cx<T> tw[N];
  __shared__ Cx<T> xb[N * C::LP];
  const int tid = threadIdx.x;
  const int l = tid % C::L, t = tid / C::L;
  const int b = blockIdx.x;
  const int kzt = b % ntz, rest = b / ntz;
  const int x = rest % N, f = rest / N;
  const int kz0 = kzt * C::L, kz = kz0 + l;
  const int yb = ybound(g, kz0);
  for (int i = tid; i < N; i += C::L * TPL) tw[i] = twg[i];
  const bool col = kz < g.kzn;
  Cx<T>* base = W + f * g.wcomp;
  const uint32_t rbase = (uint32_t)(x * (N * g.kzp + g.pad) + kz0) + l;
  const LineView<T, C::LP> lv{xb + l};
  Cx<T> v[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int p = F::in_at(t, i);
    v[i] = ld_masked(base, (uint32_t)(p * g.kzp) + rbase, col && F::in_ok(t, i) && (S < 0 || abs(kval(p, N)) <= yb));
  }
  F::run(v, t, lv, tw);
  if (col) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = F::out_pos(t, i);
      if (F::out_ok(t, i) && (S > 0 || abs(kval(p, N)) <= yb))
        st_off<stream_stores<T>(N)>(base, (uint32_t)(p * g.kzp) + rbase, v[i]);
    }
  }
}

// ------------------------------------------------------------------ y inverse with the curl
// The y-inverse pass of the step sequences of the sizes with FastCfg::YC, after
// f_xinv<C, false> (or the fused x-forward pass), which stores u_x, u_y, u_z, D_z
// and D_y in scratch fields 0, 1, 2, 4, 5.  A point here has fixed k_y and k_z,
// so the vorticity is a pointwise combination of the stored transforms,
//   omega_x = i (k_y u_z - k_z u_y),  omega_y = i k_z u_x - D_z,  omega_z = D_y - i k_y u_x,
// formed in registers before the y transform.  Block group 0 reads u_y, u_z and
// writes u_y, u_z, omega_x (fields 1, 2, 3); group 1 reads u_x, D_z, D_y and writes
// u_x, omega_y, omega_z (fields 0, 4, 5).  Each field is read once; a block's
// loads all come before its stores and no other block touches its fields on its
// (x, k_z tile), so the pass runs in place.  Output as f_ypass<C, +1> over six
// fields.  Three line buffers a thread: at 12 points a thread or over more than
// 32 threads a line this allows one block per CU, where the six single-field
// blocks of f_ypass keep two or three resident and are faster.
template <typename C>
__global__ void __launch_bounds__(C::L * C::TPL)
f_ycurl(Cx<typename C::T>* __restrict__ W, const Cx<typename C::T>* __restrict__ twg, int ntz, Geom g) {
  using T = typename C::T;
  constexpr int N = C::N, TPL = C::TPL, EPT = C::EPT;
  using F = RegFft<N, TPL, +1, typename C::Inv>;
  __shared__ Cx<T> tw[N];
  __shared__ Cx<T> xb[N * C::LP];
  const int tid = threadIdx.x;
  const int l = tid % C::L, t = tid / C::L;
  const int b = blockIdx.x;
  const int kzt = b % ntz, rest = b / ntz;
  const int x = rest % N, grp = rest / N;
  const int kz0 = kzt * C::L, kz = kz0 + l;
  const int yb = ybound(g, kz0);
  for (int i = tid; i < N; i += C::L * TPL) tw[i] = twg[i];
  const bool col = kz < g.kzn;
  Cx<T>* const Wa = W + (grp ? 0 : 1) * g.wcomp;
  Cx<T>* const Wb = W + (grp ? 4 : 2) * g.wcomp;
  Cx<T>* const Wc = W + (grp ? 5 : 3) * g.wcomp;
  const uint32_t rbase = (uint32_t)(x * (N * g.kzp + g.pad) + kz0) + l;
  const LineView<T, C::LP> lv{xb + l};
  Cx<T> va[EPT], vb[EPT], vc[EPT];
  {
    bool ok[EPT];
    uint32_t idx[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = F::in_at(t, i);
      ok[i] = col && F::in_ok(t, i) && abs(kval(p, N)) <= yb;
      idx[i] = (uint32_t)(p * g.kzp) + rbase;
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      va[i] = ld_masked(Wa, idx[i], ok[i]);
      vb[i] = ld_masked(Wb, idx[i], ok[i]);
    }
    if (grp) {
#pragma unroll
      for (int i = 0; i < EPT; ++i) vc[i] = ld_masked(Wc, idx[i], ok[i]);
    }
  }
  const T kzf = T(kz);
  if (grp) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const T kyf = T(kval(F::in_at(t, i), N));
      vb[i] = mul_i(scale(va[i], kzf)) - vb[i];  // omega_y
      vc[i] = vc[i] - mul_i(scale(va[i], kyf));  // omega_z
    }
  } else {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const T kyf = T(kval(F::in_at(t, i), N));
      vc[i] = mul_i(scale(vb[i], kyf) - scale(va[i], kzf));  // omega_x
    }
  }
  auto store = [&](Cx<T>* base, const Cx<T>* v) {
    if (col) {
#pragma unroll
      for (int i = 0; i < EPT; ++i)
        if (F::out_ok(t, i)) st_off<stream_stores<T>(N)>(base, (uint32_t)(F::out_pos(t, i) * g.kzp) + rbase, v[i]);
    }
  };
  F::run(va, t, lv, tw);
  store(Wa, va);
  F::run(vb, t, lv, tw);
  store(Wb, vb);
  F::run(vc, t, lv, tw);
  store(Wc, vc);
}

// ------------------------------------------------------------------ z fused
// P lines per block.  Inverse slices (u_x + i u_y), (u_z + i w_x), (w_y + i w_z) built
// from the half spectra on the fly (Z(k) = a(k) + i b(k), Z(N-k) = conj a(k) + i conj b(k),
// imaginary parts of the k_z = 0 and N/2 coefficients dropped); the product
// f = u x omega stays in registers; forward slices (f_x + i f_y) and f_z; the
// spectrum of f_x + i f_y is split with its mirror through the line's LDS buffer, f_z goes
// out from the registers.  Output scratch fields 0, 1, 2 = f_x, f_y, f_z (unnormalised).
//
// Bound by LDS and by instruction issue at the large sizes (512^3: 180 LDS and 1,330 vector
// instructions a wavefront), by HBM at 256^3 (604 MB in 114 us, 5.3 TB/s, what a plain
// copy reaches).  What the pass does without: twiddles read once a thread instead of
// once a transform where they fit, masks as out-of-range buffer loads instead of a
// multiplication, no division and no block barrier in the output.  Against the pass
// before, z pass in us: 128^3 20.3 -> 18.3, 160^3 40.8 -> 34.9, 192^3 50.7 -> 44.4, 216^3 85.1 ->
// 71.4, 256^3 126.7 -> 114.3, 270^3 207 -> 166, 512^3 (C_t = 2/3) 944 -> 829; 324^3, 360^3 and
// 384^3 2-4% less.
template <typename C, int P>
__global__ void __launch_bounds__(P * C::TPL)
f_zcross(Cx<typename C::T>* __restrict__ W, const Cx<typename C::T>* __restrict__ twg, Geom g) {
  using T = typename C::T;
  constexpr int N = C::N, TPL = C::TPL, EPT = C::EPT, HN = N / 2, NT = P * TPL;
  using FI = RegFft<N, TPL, +1, typename C::Inv>;
  using FF = RegFft<N, TPL, -1, typename C::Fwd>;
  static_assert(FI::RL == FF::R0, "the forward transform must start with the last inverse radix");
  static_assert(64 % TPL == 0, "a line inside one wavefront");
  constexpr int LP = line_pitch(N);
  __shared__ Cx<T> tw[N];
  __shared__ Cx<T> xb[P * LP];
  const int tid = threadIdx.x;
  const int p = tid / TPL, t = tid % TPL;
  const uint32_t line = (uint32_t)blockIdx.x * P + p;
  const LineView<T, 1> lv{xb + p * LP};
  const uint32_t lbase = line * (uint32_t)g.kzp + (line / N) * (uint32_t)g.pad;
  const uint32_t fbytes = (uint32_t)(g.wcomp * (long long)sizeof(Cx<T>));
  T fx[EPT], fy[EPT], fz[EPT];
  Cx<T> z[2][EPT];
  Cx<T> v[EPT];
  // raw half-spectrum pairs of the slices, loaded AHEAD slices ahead so that the loads
  // overlap the transforms (the barriers inside a transform keep the compiler from
  // moving later loads above it)
  Cx<T> ra[C::AHEAD > 1 ? 2 : 1][EPT], rb[C::AHEAD > 1 ? 2 : 1][EPT];
  auto fetch = [&](int q, Cx<T>* a, Cx<T>* b) {
    const BufDesc da = buf_desc(W + (2 * q) * g.wcomp, fbytes), db = buf_desc(W + (2 * q + 1) * g.wcomp, fbytes);
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int pos = FI::in_at(t, i);
      const int k = pos <= HN ? pos : N - pos;
      a[i] = ld_buf<T>(da, lbase + k, k < g.kzn);
      b[i] = ld_buf<T>(db, lbase + k, k < g.kzn);
    }
  };
  constexpr int AHEAD = C::AHEAD;
  if (AHEAD > 0) fetch(0, ra[0], rb[0]);
  if (AHEAD > 1) fetch(1, ra[1], rb[1]);
  for (int i = tid; i < N; i += NT) tw[i] = twg[i];
  __syncthreads();  // the line transforms below synchronise only within a wavefront
  const typename FI::template Twiddles<T, C::KEEP> twi(t, tw);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    constexpr int RING = AHEAD > 1 ? 2 : 1;
    if (AHEAD == 0) fetch(q, ra[0], rb[0]);
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int pos = FI::in_at(t, i);
      const Cx<T> a = ra[q % RING][i], bb = rb[q % RING][i];
      if (pos == 0 || pos == HN) v[i] = cx(a.re, bb.re);
      else if (pos < HN) v[i] = cx(a.re - bb.im, a.im + bb.re);
      else v[i] = cx(a.re + bb.im, bb.re - a.im);
    }
    if (AHEAD > 0 && q + AHEAD < 3) fetch(q + AHEAD, ra[q % RING], rb[q % RING]);
    FI::template run<true>(v, t, lv, twi);
    if (q < 2) {
#pragma unroll
      for (int i = 0; i < EPT; ++i) z[q][i] = v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const T ux = z[0][i].re, uy = z[0][i].im, uz = z[1][i].re, wx = z[1][i].im;
    const T wy = v[i].re, wz = v[i].im;
    fx[i] = uy * wz - uz * wy;
    fy[i] = uz * wx - ux * wz;
    fz[i] = ux * wy - uy * wx;
  }
  const typename FF::template Twiddles<T, C::KEEP> twf(t, tw);
#pragma unroll
  for (int i = 0; i < EPT; ++i) v[i] = cx(fx[i], fy[i]);
  FF::template run<true>(v, t, lv, twf);
  // split f_x + i f_y: the register holds k, the mirror N - k comes from the line's
  // buffer; only registers that can hold k < kzn <= N/2 (kzn <= N/2: every truncation
  // leaves the Nyquist plane out)
  exchange_barrier<true>();
#pragma unroll
  for (int i = 0; i < EPT; ++i)
    if (FF::out_ok(t, i)) lv.at(FF::out_pos(t, i)) = v[i];
  exchange_barrier<true>();
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    if ((i % FF::RL) * (N / FF::RL) >= HN) continue;  // out_pos >= N/2 for every thread
    const int k = FF::out_pos(t, i);
    if (FF::out_ok(t, i) && k < g.kzn) {
      const Cx<T> c1 = v[i], c2 = lv.at(k == 0 ? 0 : N - k);
      st_off<stream_stores<T>(N)>(W, lbase + k, cx(T(0.5) * (c1.re + c2.re), T(0.5) * (c1.im - c2.im)));
      st_off<stream_stores<T>(N)>(W + g.wcomp, lbase + k, cx(T(0.5) * (c1.im + c2.im), T(-0.5) * (c1.re - c2.re)));
    }
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i) v[i] = cx(fz[i], T(0));
  FF::template run<true>(v, t, lv, twf);
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    if ((i % FF::RL) * (N / FF::RL) >= HN) continue;
    const int k = FF::out_pos(t, i);
    if (FF::out_ok(t, i) && k < g.kzn) st_off<stream_stores<T>(N)>(W + 2 * g.wcomp, lbase + k, v[i]);
  }
}

// ------------------------------------------------------------------ x forward + epilogue
// FEED (0: none) names the stage output that is the next evaluation's input (1:
// out0, 2: out1).  The block then also runs that evaluation's x-inverse pass on
// its own tile (shift sh2): the values just computed are still in registers, at
// the input positions of the inverse transform (its first radix is the forward
// transform's last), so the tile is not read back.  An out1 that only feeds the
// next evaluation is not stored.  FEED needs a.full == 0 (the blocks are then the
// active tiles, the same as the x-inverse pass); CURL as in f_xinv.
// OP_ANY, FEED_ANY: the stage operation and the fed output come from the arguments
// (block-uniform branches), one kernel for every stage.
template <typename C, int OP, int FEED, bool CURL>
__global__ void __launch_bounds__(C::L * C::TPL)
f_xfwd(Cx<typename C::T>* __restrict__ W, const Cx<typename C::T>* __restrict__ twg, Shift sh, Shift sh2,
       const int2* __restrict__ tiles, Geom g, EpiArgs<typename C::T> a) {
  using T = typename C::T;
  constexpr int N = C::N, TPL = C::TPL, EPT = C::EPT;
  using F = RegFft<N, TPL, -1, typename C::Fwd>;
  using FI = RegFft<N, TPL, +1, typename C::Inv>;
  static_assert(FEED == 0 || F::RL == FI::R0, "the inverse transform must start with the forward's last radix");
  __shared__ Cx<T> tw[N];
  __shared__ Cx<T> phx[N];
  __shared__ Cx<T> phc[C::L];
  __shared__ Cx<T> phx2[FEED ? N : 1];
  __shared__ Cx<T> phc2[FEED ? C::L : 1];
  __shared__ Cx<T> xb[N * C::LP];
  const int tid = threadIdx.x;
  const int l = tid % C::L, t = tid / C::L;
  int yi, kz0;
  if (a.full) {
    yi = blockIdx.x / a.ntzf;
    kz0 = (blockIdx.x % a.ntzf) * C::L;
  } else {
    const int2 tile = tiles[blockIdx.x];
    yi = tile.x;
    kz0 = tile.y;
  }
  const int kz = kz0 + l;
  const int ky = kval(yi, N);
  const bool active = line_active(g, ky, kz0);
  const LineView<T, C::LP> lv{xb + l};
  Cx<T> r[3][EPT];
  Cx<T> phyz = cx(T(1), T(0));
  // stage operands, read a chunk of points ahead of the chunk whose outputs are stored
  // (out0 may alias an operand, but only at the same point, so the next chunk's loads may
  // go before this chunk's stores); the first chunk is read before the last transform
  const int op = OP == OP_ANY ? a.op : OP;
  [[maybe_unused]] const int feed = FEED == FEED_ANY ? a.feed : FEED;
  constexpr bool may0 = OP == OP_ANY || op_reads0(OP), may1 = OP == OP_ANY || op_reads1(OP);
  const bool need0 = op_reads0(op), need1 = op_reads1(op);
  constexpr bool may_out1 = (OP == OP_ANY || op_writes1(OP)) && FEED != 2;
  const bool use1 = may_out1 && op_writes1(op) && feed != 2;
  static_assert(FEED == 0 || FEED == FEED_ANY || op_can_feed(OP, FEED), "this stage output is not an evaluation input");
  Cx<T> nx[FEED ? 3 : 1][FEED ? EPT : 1];  // the fed output on this thread's points
  if constexpr (FEED != 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int i = 0; i < EPT; ++i) nx[c][i] = cx(T(0), T(0));
  }
  constexpr int CH = may0 && may1 ? C::CHUNK_TWO : C::CHUNK_ONE;  // points a chunk
  constexpr int NBUF = CH < EPT ? 2 : 1;
  const LineTest keep = line_test(g, ky, kz);
  const bool line_kept = active && kz < g.kzn;
  // streaming stores into the compact stage buffers only (rows of whole 128-byte lines)
  const bool st0 = stream_stores<T>(N) && a.lo0.pitch == g.kzp;
  [[maybe_unused]] const bool st1 = stream_stores<T>(N) && a.lo1.pitch == g.kzp;
  Cx<T> s0v[NBUF][may0 ? 3 : 1][may0 ? CH : 1], s1v[NBUF][may1 ? 3 : 1][may1 ? CH : 1];
  auto load_ops = [&](int c0) {
    const int buf = (c0 / CH) % NBUF;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      if (c0 + j >= EPT) break;  // the last chunk may be short
      const int p = F::out_at(t, c0 + j);
      const bool ok = line_kept && F::out_ok(t, c0 + j) && keep(kval(p, N));
      if constexpr (may0) {
        const uint32_t ii0 = (uint32_t)((p * N + yi) * a.li0.pitch + p * a.li0.pad + kz);
        if (need0) {
#pragma unroll
          for (int c = 0; c < 3; ++c) s0v[buf][c][j] = ld_masked(a.in0 + c * a.li0.cs, ii0, ok);
        }
      }
      if constexpr (may1) {
        const uint32_t ii1 = (uint32_t)((p * N + yi) * a.li1.pitch + p * a.li1.pad + kz);
        if (need1) {
#pragma unroll
          for (int c = 0; c < 3; ++c) s1v[buf][c][j] = ld_masked(a.in1 + c * a.li1.cs, ii1, ok);
        }
      }
    }
  };
  if (active) {
    for (int i = tid; i < N; i += C::L * TPL) tw[i] = twg[i];
    if (sh.on) {
      phase_row(phx, N, sh.s[0], tid, C::L * TPL);
      phase_cols(phc, ky, kz0, sh, N, tid);
    }
    if constexpr (FEED != 0) {
      if (sh2.on) {
        phase_row(phx2, N, sh2.s[0], tid, C::L * TPL);
        phase_cols(phc2, ky, kz0, sh2, N, tid);
      }
    }
    const bool col = kz < g.kzn;
    const uint32_t wbase = (uint32_t)(yi * g.kzp + kz0) + l, wstep = (uint32_t)(N * g.kzp + g.pad);
    // field f + 1 is loaded while field f is transformed
#pragma unroll
    for (int i = 0; i < EPT; ++i) r[0][i] = ld_masked(W, (uint32_t)F::in_at(t, i) * wstep + wbase, col && F::in_ok(t, i));
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      if (f < 2) {
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          r[f + 1][i] = ld_masked(W + (f + 1) * g.wcomp, (uint32_t)F::in_at(t, i) * wstep + wbase, col && F::in_ok(t, i));
      } else {
        load_ops(0);
      }
      F::run(r[f], t, lv, tw);  // its barriers also publish phx and phc
    }
    if (sh.on) phyz = phc[l];
  }
  const bool epi_on = !(kz >= g.h || (!a.full && kz >= g.kzn));
  if (FEED == 0 && !epi_on) return;
  const T inv_n3 = T(1) / (T(N) * T(N) * T(N));
  if (epi_on) {
    if (!active) load_ops(0);
#pragma unroll
    for (int c0 = 0; c0 < EPT; c0 += CH) {
      if (c0 + CH < EPT) load_ops(c0 + CH);
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        const int i = c0 + j;
        if (i >= EPT) break;
        if (!F::out_ok(t, i)) continue;  // no point in this register
        const int p = F::out_pos(t, i);
        const int kx = kval(p, N);
        const uint32_t io0 = (uint32_t)((p * N + yi) * a.lo0.pitch + p * a.lo0.pad + kz);
        if (!(line_kept && keep(kx))) {
          // outside the retained set: zero in outputs that must be complete (full
          // mode, the caller's arrays); stage buffers are only read at retained modes
          if (a.full)
            for (int c = 0; c < 3; ++c) st_off(a.out0 + c * a.lo0.cs, io0, cx(T(0), T(0)));
          continue;
        }
        const uint32_t io1 = use1 ? (uint32_t)((p * N + yi) * a.lo1.pitch + p * a.lo1.pad + kz) : 0u;
        Cx<T> Fv[3] = {scale(r[0][i], inv_n3), scale(r[1][i], inv_n3), scale(r[2][i], inv_n3)};
        if (sh.on) {
          const Cx<T> phi = cmul(phx[p], phyz);
          Fv[0] = cmulc(Fv[0], phi);
          Fv[1] = cmulc(Fv[1], phi);
          Fv[2] = cmulc(Fv[2], phi);
        }
        const int k2 = kx * kx + ky * ky + kz * kz;
        if (k2 == 0) {
          Fv[0] = Fv[1] = Fv[2] = cx(T(0), T(0));
        } else {
          const T rk2 = T(1) / T(k2);
          const T kxr = T(kx), kyr = T(ky), kzr = T(kz);
          const Cx<T> kd = scale(scale(Fv[0], kxr) + scale(Fv[1], kyr) + scale(Fv[2], kzr), rk2);
          Fv[0] = Fv[0] - scale(kd, kxr);
          Fv[1] = Fv[1] - scale(kd, kyr);
          Fv[2] = Fv[2] - scale(kd, kzr);
        }
        T eh = T(1), edt = T(1);
        if (op_uses_etab(op)) { eh = a.eh[k2]; edt = a.edt[k2]; }
        const T dt = a.dt;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          Cx<T>* out0 = a.out0 + c * a.lo0.cs;
          Cx<T>* out1 = use1 ? a.out1 + c * a.lo1.cs : nullptr;
          Cx<T> Nv = Fv[c];
          Cx<T> O = cx(T(0), T(0));
          if (op_forced(op) && a.force != nullptr && k2 >= 4 && k2 <= 9)
            O = a.force[c * 196 + ((kx + 3) * 7 + (ky + 3)) * 4 + kz];
          if (op != OP_HEUN1) Nv = Nv + O;  // RK4 slopes N + O (zero for the other ops)
          Cx<T> s0 = cx(T(0), T(0)), s1 = cx(T(0), T(0));
          if constexpr (may0) s0 = s0v[(c0 / CH) % NBUF][c][j];
          if constexpr (may1) s1 = s1v[(c0 / CH) % NBUF][c][j];
          Cx<T> v0 = cx(T(0), T(0)), v1 = cx(T(0), T(0));
          if (op == OP_STORE) {
            v0 = Nv;
          } else if (op == OP_AVG) {
            v0 = scale(s1 + Nv, T(0.5));
          } else if (op == OP_HEUN1) {
            v1 = scale(s0 + scale(Nv + O, dt), edt);
            v0 = scale(s0, edt) + scale(Nv + O + O, T(0.5) * dt * eh);
          } else if (op == OP_HEUN2) {
            v0 = s1 + scale(Nv, T(0.5) * dt * eh);
          } else if (op == OP_EX1B) {
            v0 = scale(s0 + scale(s1 + Nv, T(0.5) * dt * a.w), eh);
          } else if (op == OP_EX2B) {
            v0 = scale(s0, edt) + scale(s1 + Nv, dt * a.w * eh);
          } else if (op == OP_RK4_0) {
            v1 = scale(s0 + scale(Nv, T(0.5) * dt), eh);
            v0 = scale(s0 + scale(Nv, dt / T(6)), edt);
          } else if (op == OP_RK4_1) {
            v1 = scale(s0, eh) + scale(Nv, T(0.5) * dt);
            v0 = s1 + scale(Nv, dt / T(3) * eh);
          } else if (op == OP_RK4_2) {
            v1 = scale(s0, edt) + scale(Nv, dt * eh);
            v0 = s1 + scale(Nv, dt / T(3) * eh);
          } else if (op == OP_RK4_3) {
            v0 = s1 + scale(Nv, dt / T(6));
          } else if (op == OP_ACC) {
            v0 = s1 + Nv;
          } else if (op == OP_MID1) {
            v0 = scale(s0 + scale(Nv, T(0.5) * dt), eh);
          } else if (op == OP_MID2) {
            v0 = scale(s0, edt) + scale(Nv, dt * eh);
          } else if (op == OP_EUL) {
            v0 = scale(s0 + scale(Nv, dt), edt);
          } else {  // OP_EULAV
            v0 = scale(s0 + scale(s1 + Nv, dt * a.w), edt);
          }
          if constexpr (may_out1) {
            if (use1) {
              if (st1) st_off<true>(out1, io1, v1);
              else st_off(out1, io1, v1);
            }
          }
          if (st0) st_off<true>(out0, io0, v0);
          else st_off(out0, io0, v0);
          if constexpr (FEED != 0) nx[c][i] = feed == 1 ? v0 : v1;
        }
      }
    }
  }
  if constexpr (FEED != 0) {
    // the next evaluation's x-inverse pass on this tile (as f_xinv<C, CURL>, from registers)
    const bool col = kz < g.kzn;
    Cx<T> ux[EPT], uy[EPT], uz[EPT], v[EPT];
    [[maybe_unused]] const T kyf = T(ky), kzf = T(kz);
    const Cx<T> phyz2 = sh2.on ? phc2[l] : cx(T(1), T(0));
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int p = FI::in_at(t, i);
      ux[i] = nx[0][i];
      uy[i] = nx[1][i];
      uz[i] = nx[2][i];
      if (sh2.on) {
        const Cx<T> phi = cmul(phx2[p], phyz2);
        ux[i] = cmul(ux[i], phi);
        uy[i] = cmul(uy[i], phi);
        uz[i] = cmul(uz[i], phi);
      }
    }
    const uint32_t obase = (uint32_t)(yi * g.kzp + kz0) + l, ostep = (uint32_t)(N * g.kzp + g.pad);
    auto store = [&](int f, const Cx<T>* v) {
      if (col) {
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          if (FI::out_ok(t, i))
            st_off<stream_stores<T>(N)>(W + f * g.wcomp, (uint32_t)FI::out_pos(t, i) * ostep + obase, v[i]);
      }
    };
    FI::run(ux, t, lv, tw);
    store(0, ux);
#pragma unroll
    for (int i = 0; i < EPT; ++i) v[i] = mul_i(scale(uz[i], T(kval(FI::in_at(t, i), N))));
    FI::run(v, t, lv, tw);  // D_z
    if constexpr (CURL) {
#pragma unroll
      for (int i = 0; i < EPT; ++i) v[i] = mul_i(scale(ux[i], kzf)) - v[i];  // omega_y
    }
    store(4, v);
#pragma unroll
    for (int i = 0; i < EPT; ++i) v[i] = mul_i(scale(uy[i], T(kval(FI::in_at(t, i), N))));
    FI::run(v, t, lv, tw);  // D_y
    if constexpr (CURL) {
#pragma unroll
      for (int i = 0; i < EPT; ++i) v[i] = v[i] - mul_i(scale(ux[i], kyf));  // omega_z
    }
    store(5, v);
    FI::run(uy, t, lv, tw);
    store(1, uy);
    FI::run(uz, t, lv, tw);
    store(2, uz);
    if constexpr (CURL) {
#pragma unroll
      for (int i = 0; i < EPT; ++i) uy[i] = mul_i(scale(uz[i], kyf) - scale(uy[i], kzf));  // omega_x
      store(3, uy);
    }
  }
}

// Specialised sizes (FP32).  The forward radix list is the inverse one reversed.
// YC (the vorticity formed in the y-inverse pass, f_ycurl) is on for 128, 144, 256
// and 270, where the x-inverse passes writing five fields instead of six gain more
// than the y-inverse pass loses to its three-field blocks: PS-RK2 random steps
// 3.3%, 1.3%, 2.8% and 1.5% faster.  At 64, 160, 192, 216, 324, 360, 384 and 512
// those blocks leave one or two resident a CU and the step was 0.3% to 13% slower;
// 240 was unchanged.
using LP64 = LinePlan<64, 8, Radices<8, 8>, Radices<8, 8>>;
using LP128b = LinePlan<128, 16, Radices<8, 4, 4>, Radices<4, 4, 8>>;
using LP192 = LinePlan<192, 16, Radices<12, 4, 4>, Radices<4, 4, 12>>;
using LP256b = LinePlan<256, 32, Radices<8, 8, 4>, Radices<4, 8, 8>>;
// x plans of 64 to 192, 324, 360 and 384: an x pass waits for its rows, so lines of
// more threads (16 to 60) with 4 to 10 registers a transform beat fewer threads with more,
// even where a 16-column tile is then 15 waves and the only one on its CU.  Fused x passes
// of PS-RK2 random steps, us: 64^3 8 8 over 8 threads 17.6, 4 4 4 over 16 15.6; 128^3 8 4
// 4 over 16 24.5, 4 8 4 over 32 22.8; 144^3 12 12 over 12 27.1, 6 6 4 over 24 25.9; 160^3
// 10 4 4 over 16 34.0, 5 8 4 over 32 29.4; 192^3 12 4 4 over 16 65, 6 8 4 over 32 63 (RK4
// 34.4, 31.7); 324^3 12 3 3 3 over 27 343, 6 6 9 over 54 308; 360^3 12 6 5 over 30 469, 6
// 10 6 over 60 443; 384^3 12 4 4 2 over 32 507, 8 6 8 over 48 456.  216, 240, 256 and 512
// had no better plan (256^3 4 4 4 4 over 64: 163 against 165, but 91 against 86 in RK4).
// 270 keeps 9 6 5 over 30 threads: 5 6 9 over 54 made the fused pass 154 -> 140, but
// f_xinv 74 -> 85 and the last stage 121 -> 126.  f_xinv and f_xfwd run one plan, so that
// chained and single evaluations agree bit for bit.
// The adjoint's f_xadj holds four line buffers a thread and is left with one tile a CU (144:
// two) by the plans of more threads at 144, 160 and 192, so the adjoint keeps the y plans
// there (f_xlam only at 192): f_xadj, us, on the x plans and on the y plans, without and with
// operands: 144^3 35.8, 50.6 and 19.4, 35.4; 160^3 41.1, 72.2 and 34.6, 64.4; 192^3 61.2, 130
// and 42.2, 106.  A step adjoint with its first stage kept: 144^3 399 -> 361 us, 160^3 506 -> 485,
// 192^3 835 -> 784.
using LP64x = LinePlan<64, 16, Radices<4, 4, 4>, Radices<4, 4, 4>>;
using Fast64 = FastCfg<LP64x, LP64, LP64, 16, XPass<LP64x, 2>>;
using LP128x = LinePlan<128, 32, Radices<4, 8, 4>, Radices<4, 8, 4>>;
using Fast128 = FastCfg<LP128x, LP128b, LP128b, 8, XPass<LP128x, 2>, LP128b, 8, XPass<LP128x, 2>, LP128x, true>;
// z and x passes of 192: 6 8 4 over 32 threads, 8 registers a transform (the adjoint z
// pass and the y passes keep 12 4 4 over 16)
using LP192z = LinePlan<192, 32, Radices<6, 8, 4>, Radices<4, 8, 6>>;
using Fast192 = FastCfg<LP192z, LP192, LP192z, 8, XPass<LP192z, 3>, LP192, 8, LP192, LP192>;
// z pass of 256: 4 4 4 4 over 64 threads (4 registers a transform, six waves per
// SIMD; 5% faster than 8 8 4 over 32 at 256^3, whose extra exchange costs more at
// 128^3); the adjoint z pass keeps 8 8 4 over 32
using LP256z = LinePlan<256, 64, Radices<4, 4, 4, 4>, Radices<4, 4, 4, 4>>;
using Fast256 = FastCfg<LP256b, LP256b, LP256z, 4, LP256b, LP256b, 8, LP256b, LP256b, true>;
// 216 = 12 6 3 and 324 = 12 3 3 3 with 12 points per thread (18 and 27 threads per
// line), the y passes: the grids of the k_max = 108 comparison
using LP216 = LinePlan<216, 18, Radices<12, 6, 3>, Radices<3, 6, 12>>;
using LP324 = LinePlan<324, 27, Radices<12, 3, 3, 3>, Radices<3, 3, 3, 12>>;
// z passes with the line inside one wavefront (wavefront-scope synchronisation
// instead of block barriers) and few registers a thread (more waves per SIMD),
// some butterflies predicated off: 216 = 8 3 9 over 32 threads (9 registers),
// 324 = 6 6 9 over 64 (9); the adjoint z pass of 324 keeps 12 3 3 3 over 32
using LP216z = LinePlan<216, 32, Radices<8, 3, 9>, Radices<9, 3, 8>>;
using LP324z = LinePlan<324, 64, Radices<6, 6, 9>, Radices<9, 6, 6>>;
using LP324za = LinePlan<324, 32, Radices<12, 3, 3, 3>, Radices<3, 3, 3, 12>>;
// 216 and 240 run their x passes on the z plans too (32 threads a line, 512-thread
// tiles of 8 waves, 156-161 registers a thread) rather than on 18 and 24 threads a
// line (5 and 6 waves a tile, one tile per CU): fused x pass 152 -> 132 us at 216^3,
// 154 -> 146 us at 240^3
using Fast216 = FastCfg<LP216z, LP216, LP216z, 4, XPass<LP216z, 3>>;
using LP324x = LinePlan<324, 54, Radices<6, 6, 9>, Radices<9, 6, 6>>;
using Fast324 = FastCfg<LP324x, LP324, LP324z, 4, XPass<LP324x, 3>, LP324za, 4>;
// y passes of 384: 12 4 4 2 (inverse), 32 threads per line
using LP384 = LinePlan<384, 32, Radices<12, 4, 4, 2>, Radices<2, 4, 4, 12>>;
// z pass of 384: 6 8 8 over 64 threads, 8 registers and two exchanges a transform
// (the adjoint z pass keeps 12 4 4 2 over 32)
using LP384z = LinePlan<384, 64, Radices<6, 8, 8>, Radices<8, 8, 6>>;
using LP384x = LinePlan<384, 48, Radices<8, 6, 8>, Radices<8, 6, 8>>;
using Fast384 = FastCfg<LP384x, LP384, LP384z, 4, LP384x, LP384, 4>;
// 512 (the 2/3-truncated RK4 grid of the 512^3 comparison): y and z passes 8 8 8
// with one wavefront per line, four lines per z block (at eight, one 512-thread
// block of about 130 registers a thread is all a CU holds); x passes 16 8 4 with
// 32 threads per line, so that a 16-column tile is a 512-thread block of up to 256
// registers a thread (of the chained passes only the two middle RK4 stages spill, three
// registers; fewer waves per line and more registers measured faster than 1024-thread
// tiles of 128)
using LP512 = LinePlan<512, 64, Radices<8, 8, 8>, Radices<8, 8, 8>>;
using LP512x = LinePlan<512, 32, Radices<16, 8, 4>, Radices<4, 8, 16>>;
using Fast512 = FastCfg<LP512x, LP512, LP512, 4, XPass<LP512x, 4>>;
// Grids whose radices do not all divide one points-per-thread count: 12 registers
// a thread, some butterflies of a stage predicated off (fft_reg.hpp).  144 = 12 12
// (uniform, 12 threads), 160 = 10 4 4 (16), 240 = 10 4 6 (24), 270 = 9 6 5 (30),
// 360 = 10 4 9 (40, the y pass): the truncation sweeps at k_max = 64 and 108 and the
// coarse grid of the 512^3 comparison at C_t = 0.948.
using LP144 = LinePlan<144, 12, Radices<12, 12>, Radices<12, 12>>;
using LP160 = LinePlan<160, 16, Radices<10, 4, 4>, Radices<4, 4, 10>>;
using LP240 = LinePlan<240, 24, Radices<10, 4, 6>, Radices<6, 4, 10>>;
using LP270 = LinePlan<270, 30, Radices<9, 6, 5>, Radices<5, 6, 9>>;
// y passes of 360: 348 + 157 us on 40 threads a line, 10 6 6 on 36 took 363 + 180
using LP360 = LinePlan<360, 40, Radices<10, 4, 9>, Radices<9, 4, 10>>;
// z passes with lines inside one wavefront and few registers a thread: 144 = 6 6 4,
// 160 = 4 8 5, 240 = 8 6 5, 270 = 10 3 9, 360 = 12 6 5, all over 32 threads (8 to
// 15 registers a transform); the adjoint z passes of 160 and 360, which hold eight
// slices, keep 10 4 4 over 16 and 10 6 6 over 64
using LP144z = LinePlan<144, 32, Radices<6, 6, 4>, Radices<4, 6, 6>>;
using LP240z = LinePlan<240, 32, Radices<8, 6, 5>, Radices<5, 6, 8>>;
using LP270z = LinePlan<270, 32, Radices<10, 3, 9>, Radices<9, 3, 10>>;
using LP360z = LinePlan<360, 32, Radices<12, 6, 5>, Radices<5, 6, 12>>;
using LP360za = LinePlan<360, 64, Radices<10, 6, 6>, Radices<6, 6, 10>>;
using LP144x = LinePlan<144, 24, Radices<6, 6, 4>, Radices<4, 6, 6>>;
using Fast144 = FastCfg<LP144x, LP144, LP144z, 8, XPass<LP144x, 3>, LP144z, 8, LP144, LP144x, true>;
using LP160z = LinePlan<160, 32, Radices<4, 8, 5>, Radices<5, 8, 4>>;
using LP160x = LinePlan<160, 32, Radices<5, 8, 4>, Radices<4, 8, 5>>;
using Fast160 = FastCfg<LP160x, LP160, LP160z, 8, XPass<LP160x, 3>, LP160, 8, LP160>;
using Fast240 = FastCfg<LP240z, LP240, LP240z, 4, XPass<LP240z, 3>>;
using Fast270 = FastCfg<LP270, LP270, LP270z, 4, LP270, LP270z, 4, LP270, LP270, true>;
using LP360x = LinePlan<360, 60, Radices<6, 10, 6>, Radices<6, 10, 6>>;
using Fast360 = FastCfg<LP360x, LP360, LP360z, 4, XPass<LP360x, 6>, LP360za, 4>;

}  // namespace ns
