// Runs the cheapest plans (fft_core.h, pass order 3) on the CPU, every pass in
// place as the kernels do, for one random transform of every length up to
// FFT_COST_MAX and both directions, beside the plans of order 2 with the simple
// radices.  Prints "N passes error" with the largest difference relative to the
// largest value, or "N -1" where N has no plan.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "fft_core.h"

using namespace cbp;
typedef std::vector<cplx<double>> vec;

template <int R, int DIR>
void pass(vec& buf, int N, int Ns, const cplx<double>* tw) {
  const int NR = N / R;
  const float rns = 1.0f / (float)Ns;
  std::vector<int> base(NR);
  vec v((size_t)N);
  for (int j = 0; j < NR; ++j) {
    const int k = j - fdiv_floor(j, rns) * Ns;
    base[j] = Ns > 1 ? stockham_read<R, DIR, true>(buf.data(), NR, tw, j, k, &v[(size_t)j * R])
                     : stockham_read<R, DIR, false>(buf.data(), NR, tw, j, k, &v[(size_t)j * R]);
  }
  for (int j = 0; j < NR; ++j)
    for (int r = 0; r < R; ++r) buf[base[j] + r * Ns] = v[(size_t)j * R + r];
}

template <int DIR>
void transform(vec& buf, const fft_plan& p) {
  int Ns = 1;
  for (int s = 0; s < p.npass; ++s) {
    const int R = plan_radix(p, s), P = tw_pitch(R);
    vec tw((size_t)Ns * P, cplx<double>{NAN, NAN});   // a read of the padding spoils the transform
    for (int k = 0; k < Ns; ++k)
      for (int r = 1; r < R; ++r) {
        const double ang = -2.0 * M_PI * (double)(r * k) / (double)(Ns * R);
        tw[(size_t)k * P + r - 1] = {std::cos(ang), std::sin(ang)};
      }
    switch (R) {
      case 2: pass<2, DIR>(buf, p.N, Ns, tw.data()); break;
      case 3: pass<3, DIR>(buf, p.N, Ns, tw.data()); break;
      case 4: pass<4, DIR>(buf, p.N, Ns, tw.data()); break;
      case 5: pass<5, DIR>(buf, p.N, Ns, tw.data()); break;
      case 6: pass<6, DIR>(buf, p.N, Ns, tw.data()); break;
      case 7: pass<7, DIR>(buf, p.N, Ns, tw.data()); break;
      case 8: pass<8, DIR>(buf, p.N, Ns, tw.data()); break;
      case 9: pass<9, DIR>(buf, p.N, Ns, tw.data()); break;
      case 10: pass<10, DIR>(buf, p.N, Ns, tw.data()); break;
      case 12: pass<12, DIR>(buf, p.N, Ns, tw.data()); break;
      case 14: pass<14, DIR>(buf, p.N, Ns, tw.data()); break;
      case 15: pass<15, DIR>(buf, p.N, Ns, tw.data()); break;
      default: std::printf("bad radix\n"); std::exit(2);
    }
    Ns *= R;
  }
}

int main() {
  unsigned s = 12345u;
  auto rnd = [&]() { s = s * 1664525u + 1013904223u; return (double)(s >> 8) / (double)(1 << 24) - 0.5; };
  for (int N = 1; N <= FFT_COST_MAX; ++N) {
    fft_plan p, q;
    const bool a = make_fft_plan(N, &p, 3), b = make_fft_plan(N, &q, 2);
    if (a != b) return 3;
    if (!a) {
      std::printf("%d -1\n", N);
      continue;
    }
    vec x(N), y;
    for (auto& e : x) e = {rnd(), rnd()};
    y = x;
    double err = 0.0, top = 0.0;
    auto compare = [&]() {
      for (int i = 0; i < N; ++i) {
        err = std::fmax(err, std::fmax(std::fabs(x[i].re - y[i].re), std::fabs(x[i].im - y[i].im)));
        top = std::fmax(top, std::fmax(std::fabs(y[i].re), std::fabs(y[i].im)));
      }
    };
    transform<-1>(x, p);
    transform<-1>(y, q);
    compare();
    x = y;
    transform<+1>(x, p);
    transform<+1>(y, q);
    compare();
    std::printf("%d %d %g\n", N, p.npass, err / top);
  }
  return 0;
}
