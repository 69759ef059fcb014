// table_host.hip -- TEST ONLY: the sampled noise curve's interval search
// (table_setup, table_psd of gwf_model.hpp) run on the host.
#include "../../paper_2207_06910_amd/csrc/gwf_model.hpp"

using namespace gwf;

// S[i] of the curve at f[i], by the guessed interval (guess != 0) or by
// bisection; NaN outside the range.  Returns the curve's guess kind.
extern "C" int table_psd_host(int64_t n, const double* tf, const double* tS, int kind, double piM, int64_t m,
                              const double* f, int guess, double* S) {
  SiteDesc sd{};
  sd.psd_kind = kind;
  sd.tab_f = tf;
  sd.tab_S = tS;
  sd.tab_n = n;
  SiteC sc{};
  sc.tab_f = tf;
  sc.tab_S = tS;
  sc.tab_n = n;
  sc.tab_kind = kind;
  table_setup(sd, piM, sc);
  const int found = sc.tab_guess;
  if (!guess) sc.tab_guess = 0;
  for (int64_t i = 0; i < m; ++i) {
    Point q{};
    q.f = f[i];
    q.L = (std::log(piM) + std::log(f[i])) / 3.0;
    double s;
    S[i] = table_psd(sc, q, s) ? s : __builtin_nan("");
  }
  return found;
}
