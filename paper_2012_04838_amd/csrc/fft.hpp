// Register/LDS FFT engine for gfx950 (64-wide wavefronts).
//
// A length-N complex line is spread over TT = N/E threads; thread j holds the
// E elements at positions j + TT*m (m = 0..E-1).  The transform runs as
// Stockham autosort stages of radix R <= E (each thread performs E/R
// butterflies per stage); between stages the line is exchanged through LDS.
// The input and output ownership are the same strided pattern, so a batch of
// lines laid out with the line index contiguous in memory (columns) is read
// and written with fully coalesced 128-byte rows, and a contiguous line is
// read with consecutive lanes on consecutive elements.
//
// Sign convention: forward uses exp(-2 pi i n k / N) (the unnormalised forward
// transform of Eq. (5)); inverse uses exp(+2 pi i n k / N) without 1/N.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace psdns {

template <typename T>
struct alignas(2 * sizeof(T)) cpx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ cpx<T> operator+(cpx<T> a, cpx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cpx<T> operator-(cpx<T> a, cpx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ cpx<T> operator*(T s, cpx<T> a) { return {s * a.x, s * a.y}; }
template <typename T>
__device__ __forceinline__ cpx<T> cmul(cpx<T> a, cpx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cpx<T> conj(cpx<T> a) { return {a.x, -a.y}; }
// multiply by +i and by -i
template <typename T>
__device__ __forceinline__ cpx<T> mul_i(cpx<T> a) { return {-a.y, a.x}; }
template <typename T>
__device__ __forceinline__ cpx<T> mul_mi(cpx<T> a) { return {a.y, -a.x}; }
// multiply by i*s for a real s
template <typename T>
__device__ __forceinline__ cpx<T> mul_is(cpx<T> a, T s) { return {-s * a.y, s * a.x}; }

// cos(pi m / 32), m = 0..16: a quarter wave of the 64th roots of unity.
__host__ __device__ constexpr double quarter_cos64(int m) {
  switch (m) {
    case 0: return 1.0;
    case 1: return 0.99518472667219688624;
    case 2: return 0.98078528040323044913;
    case 3: return 0.95694033573220886494;
    case 4: return 0.92387953251128675613;
    case 5: return 0.88192126434835502971;
    case 6: return 0.83146961230254523708;
    case 7: return 0.77301045336273696081;
    case 8: return 0.70710678118654752440;
    case 9: return 0.63439328416364549822;
    case 10: return 0.55557023301960222474;
    case 11: return 0.47139673682599764856;
    case 12: return 0.38268343236508977173;
    case 13: return 0.29028467725446236764;
    case 14: return 0.19509032201612826785;
    case 15: return 0.09801714032956060199;
    default: return 0.0;
  }
}

// cos(2 pi m / 64) for any integer m, by symmetry of the quarter wave.
__host__ __device__ constexpr double cos64(int m) {
  m &= 63;
  return m <= 16 ? quarter_cos64(m)
       : m <= 32 ? -quarter_cos64(32 - m)
       : m <= 48 ? -quarter_cos64(m - 32)
                 : quarter_cos64(64 - m);
}
__host__ __device__ constexpr double sin64(int m) { return cos64(m - 16); }

// a * exp(-+ 2 pi i m / 64) with m a compile-time constant after unrolling.
// The trivial roots become swaps/negations so no multiplication by 0 or 1 survives.
template <bool INV, typename T>
__device__ __forceinline__ cpx<T> rot64(cpx<T> a, int m) {
  m &= 63;
  if (m == 0) return a;
  if (m == 32) return {-a.x, -a.y};
  if (m == 16) return INV ? mul_i(a) : mul_mi(a);
  if (m == 48) return INV ? mul_mi(a) : mul_i(a);
  const T c = static_cast<T>(cos64(m));
  const T s = INV ? static_cast<T>(sin64(m)) : static_cast<T>(-sin64(m));
  return {a.x * c - a.y * s, a.x * s + a.y * c};
}

__device__ __forceinline__ float fma_of(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return __builtin_fma(a, b, c); }

// a + w b and a - w b with w = (c, s) a unit root, in six fused multiply-adds: four for the
// sum t, then 2 a - t for the difference, which carries the rounding of t as well.  EIGHT: the
// difference in four of its own, with a smaller error (see dft for where it is taken).
template <bool INV, bool EIGHT = false, typename T>
__device__ __forceinline__ void butterfly(cpx<T>& a, cpx<T>& b, cpx<T> w) {
  if (INV) w.y = -w.y;
  const cpx<T> t = {fma_of(-w.y, b.y, fma_of(w.x, b.x, a.x)), fma_of(w.y, b.x, fma_of(w.x, b.y, a.y))};
  if constexpr (EIGHT)
    b = {fma_of(w.y, b.y, fma_of(-w.x, b.x, a.x)), fma_of(-w.y, b.x, fma_of(-w.x, b.y, a.y))};
  else
    b = {fma_of(T(2), a.x, -t.x), fma_of(T(2), a.y, -t.y)};
  a = t;
}
// a + w b and a - w b for the root w = exp(-+ 2 pi i M / 64), 0 <= M < 32: the trivial ones are
// sums and swaps, so inputs known to be zero fold away, and the odd multiples of an eighth turn
// scale one sum and one difference
template <bool INV, int M, typename T>
__device__ __forceinline__ void butterfly64(cpx<T>& a, cpx<T>& b) {
  if constexpr (M == 0 || M == 16) {
    const cpx<T> r = rot64<INV>(b, M);
    b = a - r;
    a = a + r;
  } else if constexpr (M == 8 || M == 24) {
    const T h = static_cast<T>(cos64(8));
    // forward: w b = h (b - i b) for M = 8, and -i times that for M = 24; inverse: the conjugate root
    const cpx<T> p = INV ? b + mul_i(b) : b + mul_mi(b);
    const cpx<T> q = M == 8 ? p : INV ? mul_i(p) : mul_mi(p);
    b = {fma_of(-h, q.x, a.x), fma_of(-h, q.y, a.y)};
    a = {fma_of(h, q.x, a.x), fma_of(h, q.y, a.y)};
  } else {
    butterfly<INV, true>(a, b, cpx<T>{static_cast<T>(cos64(M)), static_cast<T>(-sin64(M))});
  }
}

template <int R>
__host__ __device__ constexpr int bitrev(int i) {
  int r = 0;
  for (int b = 1; b < R; b <<= 1) {
    r = (r << 1) | (i & 1);
    i >>= 1;
  }
  return r;
}

// In-register R-point DFT (R a power of two, R <= 64): bit-reversal permutation (free in
// registers), then radix-2 decimation in time.  Levels, butterflies and factors are template
// arguments, so that every array stays in registers at any radix.
//
// A stage after the first has inputs x_r w^r.  Up to radix 16 they take R - 1 factors, one per
// input: the upper half's inside the first level's butterflies, the lower half's before them.  The
// first level's take six instructions at radix 8 and 16 except the first, all others eight (a
// radix-8 stage: 74 instructions; with a product per input and a decimation in frequency 84).  A
// radix-32 stage holds R / 2 factors, one for each level and butterfly: w^(R / len) exp(-2 pi i k / len)
// at level len, where k >= len / 4 is -i times k - len / 4, in six instructions each; R - 1 of them
// do not fit the registers (1024^3 FP32: 157 ms a step, 135 with R / 2).
// RMS error of FP32 lines of 8 to 1024 points, 4 to 32 elements per thread, against products and a
// decimation in frequency: 0.97 to 1.00 of it, never more (tests/transform_error.cpp).  R / 2 factors
// at every radix are fewer to hold, but every input then meets log2(R) / 2 of them: up to 1.02 of it
// with eight instructions, 1.13 with six.
__host__ __device__ constexpr bool tw_by_level(int R) { return R >= 32; }
__host__ __device__ constexpr int tw_factors(int R) { return tw_by_level(R) ? R / 2 : R - 1; }
// index among the R / 2 factors of factor (len, k), 0 <= k < max(1, len / 4)
__host__ __device__ constexpr int tw_slot(int len, int k) { return len == 2 ? 0 : len / 4 + k; }
// levels LEN, 2 LEN, .. of the transform, butterflies J, J + 1, .. of the level
template <int R, bool INV, int LEN, int J = 0, typename T>
__device__ __forceinline__ void dft_levels(cpx<T> (&b)[R]) {
  if constexpr (LEN <= R) {
    constexpr int H = LEN / 2;
#pragma unroll
    for (int s = 0; s < R; s += LEN) butterfly64<INV, J * (64 / LEN)>(b[s + J], b[s + J + H]);
    if constexpr (J + 1 < H)
      dft_levels<R, INV, LEN, J + 1>(b);
    else
      dft_levels<R, INV, 2 * LEN>(b);
  }
}
// the same with a factor per level and butterfly
template <int R, bool INV, int LEN, int J = 0, typename T, class Tw>
__device__ __forceinline__ void dft_levels_tw(cpx<T> (&b)[R], const Tw& tw) {
  if constexpr (LEN <= R) {
    constexpr int H = LEN / 2;
    constexpr bool q = LEN >= 4 && 2 * J >= H;  // second quarter: -i (or +i) times the first
    const cpx<T> w = tw.template get<tw_slot(LEN, q ? J - H / 2 : J)>();
#pragma unroll
    for (int s = 0; s < R; s += LEN) {
      cpx<T> v = b[s + J + H];
      if constexpr (q) v = INV ? mul_i(v) : mul_mi(v);
      butterfly<INV>(b[s + J], v, w);
      b[s + J + H] = v;
    }
    if constexpr (J + 1 < H)
      dft_levels_tw<R, INV, LEN, J + 1>(b, tw);
    else
      dft_levels_tw<R, INV, 2 * LEN>(b, tw);
  }
}
// first level of the bit-reversed inputs, a factor per input
template <int R, bool INV, int S = 0, typename T, class Tw>
__device__ __forceinline__ void dft_first_tw(cpx<T> (&b)[R], const Tw& tw) {
  if constexpr (S < R) {
    constexpr int r = bitrev<R>(S);
    if constexpr (r > 0) {
      cpx<T> w = tw.template get<r - 1>();
      if (INV) w.y = -w.y;
      b[S] = cmul(b[S], w);
    }
    butterfly<INV, (R < 8 || S == 0)>(b[S], b[S + 1], tw.template get<r + R / 2 - 1>());
    dft_first_tw<R, INV, S + 2>(b, tw);
  }
}
template <int R, bool INV, typename T>
__device__ __forceinline__ void dft(cpx<T> (&a)[R]) {
  cpx<T> b[R];
#pragma unroll
  for (int i = 0; i < R; ++i) b[i] = a[bitrev<R>(i)];
  dft_levels<R, INV, 2>(b);
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = b[i];
}
// with the stage factors tw.get<i>(), i < tw_factors(R)
template <int R, bool INV, typename T, class Tw>
__device__ __forceinline__ void dft(cpx<T> (&a)[R], const Tw& tw) {
  cpx<T> b[R];
#pragma unroll
  for (int i = 0; i < R; ++i) b[i] = a[bitrev<R>(i)];
  if constexpr (tw_by_level(R)) {
    dft_levels_tw<R, INV, 2>(b, tw);
  } else {
    dft_first_tw<R, INV>(b, tw);
    dft_levels<R, INV, 4>(b);
  }
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = b[i];
}

// The same DFT by radix-2 decimation in frequency and a bit-reversal permutation, of inputs that
// were multiplied by their twiddles before: the transforms of the statistics (see fft_dif).
template <int R, bool INV, typename T>
__device__ __forceinline__ void dft_dif(cpx<T> (&a)[R]) {
#pragma unroll
  for (int len = R; len >= 2; len >>= 1) {
    const int half = len >> 1;
#pragma unroll
    for (int s = 0; s < R; s += len) {
#pragma unroll
      for (int j = 0; j < half; ++j) {
        const cpx<T> u = a[s + j];
        const cpx<T> w = a[s + j + half];
        a[s + j] = u + w;
        a[s + j + half] = rot64<INV>(u - w, j * (64 / len));
      }
    }
  }
  cpx<T> b[R];
#pragma unroll
  for (int i = 0; i < R; ++i) b[i] = a[bitrev<R>(i)];
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = b[i];
}

// LDS views used for the inter-stage exchange; x is the running exchange index.
// Columns: element p of the line owned by lane column c sits at base[p * W].  With
// SPAN > 0 two buffers SPAN entries apart alternate between exchanges, so a buffer
// is only rewritten after the barrier of the following exchange, which every thread
// reaches after its reads: one barrier per exchange instead of two.
template <typename T, int W, int SPAN = 0>
struct LdsCol {
  static constexpr bool kDouble = SPAN > 0;
  cpx<T>* base;
  __device__ __forceinline__ void st(int p, cpx<T> v, int x) const { base[(x & 1) * SPAN + p * W] = v; }
  __device__ __forceinline__ cpx<T> ld(int p, int x) const { return base[(x & 1) * SPAN + p * W]; }
};
// Contiguous line (one line per E-element lane group): element p is stored at
// p ^ ((p >> log2 E) & min(31, N-1)).  The XOR swizzle keeps the Stockham writes
// (stride E between lanes in the first stage, runs of E lanes later) and the
// strided reads free of LDS bank conflicts for 32 and 64 banks of 4 bytes.
template <typename T, int N, int E>
struct LdsLine {
  cpx<T>* base;
  static constexpr int kShift = E == 1 ? 0 : E == 2 ? 1 : E == 4 ? 2 : E == 8 ? 3 : E == 16 ? 4 : E == 32 ? 5 : 6;
  static constexpr int kMask = N - 1 < 31 ? N - 1 : 31;
  static constexpr bool kDouble = false;
  static __device__ __forceinline__ int idx(int p) { return p ^ ((p >> kShift) & kMask); }
  __device__ __forceinline__ void st(int p, cpx<T> v, int = 0) const { base[idx(p)] = v; }
  __device__ __forceinline__ cpx<T> ld(int p, int = 0) const { return base[idx(p)]; }
};
template <int N>
struct LinePad {
  static constexpr int value = N + N / 16;
};

// Exchange synchronisation: the whole block (lines spread over several
// wavefronts) or one wavefront (every line owned by lanes of a single wave;
// LDS operations of a wave execute in order, so only compiler ordering is needed).
struct BlockSync {
  static __device__ __forceinline__ void sync() { __syncthreads(); }
};
struct WaveSync {
  static __device__ __forceinline__ void sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};

// Number of stage factors one thread applies (all stages after the first; see dft).
template <int N, int E, int NS = 1>
__host__ __device__ constexpr int tw_count() {
  if constexpr (NS >= N) {
    return 0;
  } else {
    constexpr int R = (NS * E <= N) ? E : N / NS;
    constexpr int NB = E / R;
    return (NS > 1 ? NB * tw_factors(R) : 0) + tw_count<N, E, NS * R>();
  }
}

// Root index of stage factor i (see dft), with w = w_N^(kv N / (NS R)); below N for every kv < NS.
template <int N, int NS, int R>
__device__ __forceinline__ int tw_index(int kv, int i) {
  if constexpr (tw_by_level(R)) {
    const int q = i ? 1 << (31 - __builtin_clz(i)) : 0, k = i - q;  // len / 4 and k of slot i
    const int sh = i ? 33 - __builtin_clz(i) : 1;                   // log2 len
    return (kv * (N / NS) + k * N) >> sh;
  } else {
    return (i + 1) * kv * (N / (NS * R));
  }
}
// The factor table of an N-point transform with E elements per thread: for each stage after the
// first, factor i of butterfly kv at i NS + kv.  A thread's factors are then one address and
// immediate offsets, where roots at multiples of kv took an address register each (phase-shift x
// pass, 512^3 FP32: 28 registers spilled against 5).  Entries of the stages before NS (NS = N: of all).
template <int N, int E, int NS, int AT = 1>
__host__ __device__ constexpr int tw_table() {
  if constexpr (AT >= NS) {
    return 0;
  } else {
    constexpr int R = (AT * E <= N) ? E : N / AT;
    return (AT > 1 ? AT * tw_factors(R) : 0) + tw_table<N, E, NS, AT * R>();
  }
}

// The factors of one thread kept in registers: identical for every line the
// thread transforms, so they are read from the table once.
template <int N, int E, typename T>
struct TwReg {
  static constexpr int C = tw_count<N, E>() > 0 ? tw_count<N, E>() : 1;
  cpx<T> w[C];
};

template <int N, int E, int NS, int OFF, typename T>
__device__ __forceinline__ void tw_fill_stage(TwReg<N, E, T>& t, int j, const cpx<T>* __restrict__ tw) {
  if constexpr (NS < N) {
    constexpr int TT = N / E;
    constexpr int R = (NS * E <= N) ? E : N / NS;
    constexpr int NB = E / R;
    if constexpr (NS > 1) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int kv = (j + TT * b) & (NS - 1);
#pragma unroll
        for (int i = 0; i < tw_factors(R); ++i)
          t.w[OFF + b * tw_factors(R) + i] = tw[tw_table<N, E, NS>() + i * NS + kv];
      }
      tw_fill_stage<N, E, NS * R, OFF + NB * tw_factors(R)>(t, j, tw);
    } else {
      tw_fill_stage<N, E, NS * R, OFF>(t, j, tw);
    }
  }
}

template <int N, int E, typename T>
__device__ __forceinline__ TwReg<N, E, T> tw_fill(int j, const cpx<T>* __restrict__ tw) {
  TwReg<N, E, T> t;
  tw_fill_stage<N, E, 1, 0>(t, j, tw);
  return t;
}

// stage factor i of butterfly b, kv = b mod NS: from the table (pointer) or from registers
template <int N, int E, int NS, int OFF, int R, typename T>
__device__ __forceinline__ cpx<T> tw_get(const cpx<T>* __restrict__ tw, int b, int i, int kv) {
  return tw[tw_table<N, E, NS>() + i * NS + kv];
}
template <int N, int E, int NS, int OFF, int R, typename T>
__device__ __forceinline__ cpx<T> tw_get(const TwReg<N, E, T>& t, int b, int i, int kv) {
  return t.w[OFF + b * tw_factors(R) + i];
}

// The factors of stage butterfly b, each fetched where dft uses it.
template <int N, int E, int NS, int OFF, int R, typename T, class Tw>
struct StageTw {
  const Tw& tw;
  int b, kv;
  template <int I>
  __device__ __forceinline__ cpx<T> get() const {
    return tw_get<N, E, NS, OFF, R, T>(tw, b, I, kv);
  }
};
// The same fetched ahead: all factors of the thread's butterflies of stage NS, loaded with the
// stage's inputs before the barrier that follows them.
template <int N, int E, int NS, typename T>
struct AheadTw {
  static constexpr int TT = N / E, R = (NS * E <= N) ? E : N / NS, NB = E / R, F = tw_factors(R);
  cpx<T> w[NB * F];
  template <int OFF, class Tw>
  __device__ __forceinline__ void fetch(const Tw& tw, int j) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < F; ++i) w[b * F + i] = tw_get<N, E, NS, OFF, R, T>(tw, b, i, (j + TT * b) & (NS - 1));
  }
  struct Butterfly {
    const cpx<T>* w;
    template <int I>
    __device__ __forceinline__ cpx<T> get() const {
      return w[I];
    }
  };
  __device__ __forceinline__ Butterfly of(int b) const { return {w + b * F}; }
};
struct NoTw {};
// At four elements per thread and fewer, where the length of a thread's chain counts (32^3 FP64: a
// step 2% shorter); at eight the registers are worth more (512^3 FP32: 0.6% longer with it).
template <int E>
constexpr bool tw_ahead() {
  return E <= 4;
}

// Number of LDS exchanges of an N-point transform with E elements per thread.
template <int N, int E, int NS = 1>
__host__ __device__ constexpr int exchanges() {
  if constexpr (NS >= N) {
    return 0;
  } else {
    constexpr int R = (NS * E <= N) ? E : N / NS;
    return (NS * R == N ? 0 : 1) + exchanges<N, E, NS * R>();
  }
}

// One Stockham stage (and, recursively, the ones after it).
// NS = product of the radices already applied; OFF = twiddles used so far;
// XI = exchanges done so far.
template <int N, int E, bool INV, int NS, int OFF, class Sync, int XI = 0, typename T, class Lds, class Tw, class Ahead>
__device__ __forceinline__ void fft_stage(cpx<T> (&v)[E], const Lds& lds, int j, const Tw& tw, const Ahead& ahead) {
  if constexpr (NS < N) {
    constexpr int TT = N / E;
    constexpr int R = (NS * E <= N) ? E : N / NS;
    constexpr int NB = E / R;
    constexpr bool LAST = (NS * R == N);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int vb = j + TT * b;
      const int kv = vb & (NS - 1);
      cpx<T> a[R];
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = v[b + r * NB];
      if constexpr (NS > 1 && tw_ahead<E>()) {
        dft<R, INV>(a, ahead.of(b));
      } else if constexpr (NS > 1) {
        dft<R, INV>(a, StageTw<N, E, NS, OFF, R, T, Tw>{tw, b, kv});
      } else {
        dft<R, INV>(a);
      }
      if constexpr (LAST) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[b + r * NB] = a[r];
      } else {
        const int base = (vb / NS) * NS * R + kv;
#pragma unroll
        for (int r = 0; r < R; ++r) lds.st(base + r * NS, a[r], XI);
      }
    }
    if constexpr (!LAST) {
      constexpr int OFF1 = NS > 1 ? OFF + NB * tw_factors(R) : OFF;
      std::conditional_t<tw_ahead<E>(), AheadTw<N, E, NS * R, T>, NoTw> next;
      Sync::sync();
      if constexpr (tw_ahead<E>()) next.template fetch<OFF1>(tw, j);
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = lds.ld(j + TT * m, XI);
      // with two buffers the trailing barrier is needed only where the next transform
      // would reuse this buffer first: after the last exchange of an odd count
      constexpr int NX = exchanges<N, E>();
      if constexpr (!Lds::kDouble || (XI + 1 == NX && NX % 2 == 1)) Sync::sync();
      fft_stage<N, E, INV, NS * R, OFF1, Sync, XI + 1>(v, lds, j, tw, next);
    }
  }
}

// Full N-point transform of the strided register line.  With BlockSync every
// thread of the block must call it; with WaveSync every lane of the wave.
// tw is either a pointer to the factor table (in LDS, stage_twiddles) or the thread's TwReg.
template <int N, int E, bool INV, class Sync = BlockSync, typename T, class Lds, class Tw>
__device__ __forceinline__ void fft(cpx<T> (&v)[E], const Lds& lds, int j, const Tw& tw) {
  fft_stage<N, E, INV, 1, 0, Sync>(v, lds, j, tw, NoTw{});
}

// The N-point transform of the statistics: the same stages and exchanges with separate input
// twiddles and dft_dif.  It keeps the rounding of the grid values that the moments and the velocity
// maximum of a record are taken from, which an FP32 plan reports as FP64 numbers: the same field
// has the same maximum there from one release to the next (sums may differ in the order of their
// FP64 terms).  The maximum of a step record comes from fft and agrees with it to FP32 rounding.
template <int N, int E, bool INV, class Sync = BlockSync, int NS = 1, typename T, class Lds>
__device__ __forceinline__ void fft_dif(cpx<T> (&v)[E], const Lds& lds, int j, const cpx<T>* __restrict__ tw) {
  if constexpr (NS < N) {
    constexpr int TT = N / E;
    constexpr int R = (NS * E <= N) ? E : N / NS;
    constexpr int NB = E / R;
    constexpr bool LAST = (NS * R == N);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int vb = j + TT * b;
      const int kv = vb & (NS - 1);
      cpx<T> a[R];
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = v[b + r * NB];
      if constexpr (NS > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) {
          cpx<T> w = tw[r * kv * (N / (NS * R))];
          if (INV) w.y = -w.y;
          a[r] = cmul(a[r], w);
        }
      }
      dft_dif<R, INV>(a);
      if constexpr (LAST) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[b + r * NB] = a[r];
      } else {
        const int base = (vb / NS) * NS * R + kv;
#pragma unroll
        for (int r = 0; r < R; ++r) lds.st(base + r * NS, a[r], 0);
      }
    }
    if constexpr (!LAST) {
      Sync::sync();
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = lds.ld(j + TT * m, 0);
      Sync::sync();
      fft_dif<N, E, INV, Sync, NS * R>(v, lds, j, tw);
    }
  }
}

// Copy the N roots into LDS (block-wide; ends with a block barrier).
template <int N, typename T>
__device__ __forceinline__ void stage_roots(cpx<T>* dst, const cpx<T>* __restrict__ src) {
  for (int i = threadIdx.x; i < N; i += blockDim.x) dst[i] = src[i];
  __syncthreads();
}

// root index of entry i of the factor table, i counted from the stage NS on
template <int N, int E, int NS = 1>
__device__ __forceinline__ int tw_entry(int i) {
  constexpr int R = (NS * E <= N) ? E : N / NS;
  constexpr int n = NS > 1 ? NS * tw_factors(R) : 0;
  if constexpr (NS > 1 && NS * R >= N) {
    return tw_index<N, NS, R>(i & (NS - 1), i / NS);
  } else if constexpr (NS * R >= N) {
    return 0;
  } else {
    if (NS > 1 && i < n) return tw_index<N, NS, R>(i & (NS - 1), i / NS);
    return tw_entry<N, E, NS * R>(i - n);
  }
}
// Lay the factor table of an N-point transform out in LDS, fewer than N entries (block-wide; ends
// with a block barrier).
template <int N, int E, typename T>
__device__ __forceinline__ void stage_twiddles(cpx<T>* dst, const cpx<T>* __restrict__ src) {
  static_assert(tw_table<N, E, N>() < N, "the factor table must fit the block's N entries");
  for (int i = threadIdx.x; i < tw_table<N, E, N>(); i += blockDim.x) dst[i] = src[tw_entry<N, E>(i)];
  __syncthreads();
}

}  // namespace psdns
