// Host program over the transforms of csrc/fft.hpp (its stages, factors and factor table, one
// butterfly at a time): RMS error of random FP32 lines against the same transform in FP64, and
// that of the direct form, a product per input and a decimation in frequency.  Prints for every
// line length N and elements per thread E: N E inverse error direct.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "fft.hpp"

using namespace psdns;

template <typename T>
using Line = std::vector<cpx<T>>;

template <int R, typename T>
static void direct_twiddles(cpx<T> (&a)[R], const Line<T>& root, int at, bool inv) {
  for (int r = 1; r < R; ++r) {
    cpx<T> w = root[r * at];
    if (inv) w.y = -w.y;
    a[r] = cmul(a[r], w);
  }
}

// stages from NS on of the line x; table: fft.hpp's factors, or null for the direct form
template <int N, int E, bool INV, int NS, typename T>
static void stages(Line<T>& x, const Line<T>& root, const cpx<T>* table) {
  if constexpr (NS < N) {
    constexpr int R = (NS * E <= N) ? E : N / NS;
    Line<T> out(N);
    for (int vb = 0; vb < N / R; ++vb) {
      const int kv = vb & (NS - 1);
      cpx<T> a[R];
      for (int r = 0; r < R; ++r) a[r] = x[vb + r * (N / R)];
      if (!table) {
        if (NS > 1) direct_twiddles<R>(a, root, kv * (N / (NS * R)), INV);
        dft_dif<R, INV>(a);
      } else if constexpr (NS > 1) {
        dft<R, INV>(a, StageTw<N, E, NS, 0, R, T, const cpx<T>*>{table, 0, kv});
      } else {
        dft<R, INV>(a);
      }
      for (int r = 0; r < R; ++r) out[(vb / NS) * NS * R + kv + r * NS] = a[r];
    }
    x = out;
    stages<N, E, INV, NS * R>(x, root, table);
  }
}

template <typename T>
static Line<T> roots(int n) {
  Line<T> r(n);
  for (int m = 0; m < n; ++m) r[m] = {(T)std::cos(2 * M_PI * m / n), (T)-std::sin(2 * M_PI * m / n)};
  return r;
}

template <int N, int E, bool INV>
static void run() {
  if constexpr (E <= N) {
    const Line<float> root = roots<float>(N);
    const Line<double> exact_root = roots<double>(N);
    std::vector<cpx<float>> table(N);
    stage_twiddles<N, E>(table.data(), root.data());
    std::mt19937 gen(N * 64 + E);
    std::normal_distribution<float> normal;
    double err = 0, dir = 0, norm = 0;
    for (int line = 0; line < 400000 / N; ++line) {
      Line<float> a(N);
      for (auto& v : a) v = {normal(gen), normal(gen)};
      Line<float> b = a;
      Line<double> ref(N);
      for (int i = 0; i < N; ++i) ref[i] = {a[i].x, a[i].y};
      stages<N, E, INV, 1>(a, root, table.data());
      stages<N, E, INV, 1>(b, root, (const cpx<float>*)nullptr);
      stages<N, E, INV, 1>(ref, exact_root, (const cpx<double>*)nullptr);
      for (int i = 0; i < N; ++i) {
        err += std::pow(a[i].x - ref[i].x, 2) + std::pow(a[i].y - ref[i].y, 2);
        dir += std::pow(b[i].x - ref[i].x, 2) + std::pow(b[i].y - ref[i].y, 2);
        norm += ref[i].x * ref[i].x + ref[i].y * ref[i].y;
      }
    }
    std::printf("%d %d %d %.6e %.6e\n", N, E, (int)INV, std::sqrt(err / norm), std::sqrt(dir / norm));
  }
}

template <int N>
static void all() {
  run<N, 4, false>();
  run<N, 8, false>();
  run<N, 16, false>();
  run<N, 8, true>();
}

int main() {
  all<8>();
  all<16>();
  all<32>();
  all<64>();
  all<128>();
  all<256>();
  all<512>();
  all<1024>();
  run<1024, 32, false>();  // the one length at 32 elements
  run<1024, 32, true>();
}
