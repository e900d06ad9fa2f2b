// Host build of the flight step (AVM_HOST_DEBUG): an electron at rest in a
// zero field, in gases whose rates do not vanish at zero energy.  Its energy
// stays zero (an elastic collision takes a share of it, an excitation's window
// is shut), so each flight's outcome follows from its second uniform, the
// majorant and the rates alone, which this program works out by itself.
// Prints, per gas, tables and precision: flights, real collisions, and
// flights whose outcome differs.
#define AVM_HOST_DEBUG 1
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <limits>
#include <vector>

// (the host's library has no sincospif)
__host__ inline void sincospif(float x, float* s, float* c) {
  *s = std::sin(3.14159265358979323846f * x);
  *c = std::cos(3.14159265358979323846f * x);
}

#include "avm_device.hpp"

using namespace avm;

struct Chan {
  int kind;
  double rate, e_lo;
};

// One table entry per node, channel tables with a slot past their end that
// would end the electron if it were read.
template <class R>
struct Gas {
  static constexpr int kBins = 8, kBands = 2;
  std::vector<double> cum, cum0, total, bg, bi, be, sct;
  std::vector<float> cum_f, cum0_f, total_f, bg_f, bi_f, be_f;
  std::vector<ChanDev> ch;
  std::vector<ChanP<float>> ch_f;
  std::vector<R> fit_be, fit_cum0;
  GasDev G{};

  Gas(const std::vector<Chan>& cs, double gamma) {
    const int nc = (int)cs.size();
    for (int k = 0; k <= kBins; ++k) {
      double acc = 0.0;
      for (const Chan& c : cs) cum.push_back(acc += c.rate);
      cum0.push_back(cs[0].rate);
      total.push_back(acc);
    }
    for (int b = 0; b < kBands; ++b) {
      bg.push_back(gamma);
      bi.push_back(1.0 / gamma);
      be.push_back(b == kBands - 1 ? std::numeric_limits<double>::infinity() : 50.0);
    }
    for (int i = 0; i <= nc; ++i) {
      ChanDev d{};
      d.kind = i < nc ? cs[i].kind : (int)CH_ATTACHMENT;
      d.e_lo = i < nc ? cs[i].e_lo : -1.0;
      d.e_hi = std::numeric_limits<double>::infinity();
      d.mu2p1 = 1.0;
      if (d.kind == CH_ELASTIC) {
        d.mu = 1e-5; d.el_loss = 2e-5; d.mu2p1 = 1.0 + 1e-10; d.two_mu = 2e-5;
      } else {
        d.loss = i < nc ? cs[i].e_lo : 0.0;
      }
      ch.push_back(d);
      ChanP<float> q{};
      q.kind = d.kind; q.e_lo = d.e_lo; q.e_hi = d.e_hi;
      q.loss = (float)d.loss; q.mu = (float)d.mu; q.el_loss = (float)d.el_loss;
      q.mu2p1 = (float)d.mu2p1; q.two_mu = (float)d.two_mu;
      ch_f.push_back(q);
    }
    sct.resize(2 * kAzN);
    for (int j = 0; j < kAzN; ++j) sincospi_pos((double)j / (kAzN / 2), &sct[2 * j], &sct[2 * j + 1]);
    const auto copy = [](const std::vector<double>& a, std::vector<float>& b) { b.assign(a.begin(), a.end()); };
    copy(cum, cum_f); copy(cum0, cum0_f); copy(total, total_f); copy(bg, bg_f); copy(bi, bi_f); copy(be, be_f);
    G.cum = cum.data(); G.cum0 = cum0.data(); G.total = total.data();
    G.band_gamma = bg.data(); G.band_inv = bi.data(); G.band_edge = be.data(); G.ch = ch.data();
    G.cum_f = cum_f.data(); G.cum0_f = cum0_f.data(); G.total_f = total_f.data();
    G.band_gamma_f = bg_f.data(); G.band_inv_f = bi_f.data(); G.band_edge_f = be_f.data(); G.ch_f = ch_f.data();
    G.sct = sct.data();
    G.scale = kBins / 100.0; G.scale_f = (float)G.scale;
    G.gamma = gamma; G.inv_gamma = 1.0 / gamma;
    G.gamma_f = (float)gamma; G.inv_gamma_f = (float)(1.0 / gamma);
    G.band_scale = kBands / 100.0; G.band_scale_f = (float)G.band_scale;
    G.n_bins = kBins; G.n_ch = nc; G.n_bands = kBands; G.band_bins = kBins / kBands;
    G.x_top = kBins; G.x_top_f = kBins;
    // the staged form: band edges -infinity below the first and NaN for the
    // last; channel 0's rate, or -1 where it does not act at every energy
    const TabView<R> v = global_view<R>(G);
    for (int k = 0; k <= kBins; ++k) fit_cum0.push_back(v.el0 ? v.cum0[k] : R(-1));
    fit_be = {-std::numeric_limits<R>::infinity(), R(50), std::numeric_limits<R>::quiet_NaN()};
  }
  TabFit<R> fit() const {
    const TabView<R> v = global_view<R>(G);
    return TabFit<R>{v.tot, fit_cum0.data(), v.x_lo, v.el0, v.bgam, v.binv, fit_be.data() + 1, v.ch, v.sct};
  }
};

// -1 null, -2 - c masked, c real
static int outcome(const std::vector<Chan>& cs, double r_sel) {
  double acc = 0.0;
  for (int c = 0; c < (int)cs.size(); ++c)
    if (r_sel < (acc += cs[c].rate)) return cs[c].e_lo > 0.0 ? -2 - c : c;
  return -1;
}

template <class R, bool kBanded, class TV>
static void fly(const char* name, const char* tabs, const std::vector<Chan>& cs, const Gas<R>& g, const TV& T,
                double gamma) {
  FieldDev F{};
  F.z_lo = 0.0; F.z_hi = 1.0; F.z_mid = 0.5; F.z_half = F.z_half_f = 0.49;
  RunParams P{};
  P.key0 = 7; P.k_max = 1u << 30; P.t_max = std::numeric_limits<double>::infinity();
  P.k_a = 0.00176; P.two_ka = 2 * P.k_a; P.inv_2ka = 1 / P.two_ka;
  P.k_a_f = (float)P.k_a; P.two_ka_f = (float)P.two_ka; P.inv_2ka_f = (float)P.inv_2ka;
  P.look = 1.0;
  Elec<R> e{};
  e.z = 0.5; e.eid = 1ull << 63;
  Child<R> child{};
  uint32_t clear = 0, trace = 0, real = 0, masked = 0;
  long bad = 0;
  const long n = 4000;
  for (long i = 0; i < n; ++i) {
    const uint32_t k = e.k;
    const Block w = draw(P, e.aval, e.eid, k, 0);
    const int c = outcome(cs, u53(w.w2, w.w3) * gamma);
    real += c >= 0;
    masked += c < -1;
    if (c != -1) trace = trace_step(trace, k, c >= 0 ? (uint32_t)c : TRACE_MASKED + (uint32_t)(-2 - c));
    const int32_t r = flight_step<R, kBanded, FIELD_SLAB>(e, g.G, T, F, P, child, clear, RandInline<R>{});
    if (r != STEP_CONTINUE || e.k != k + 1 || e.n_real != real || e.n_masked != masked || e.trace != trace ||
        e.vx != 0 || e.vy != 0 || e.vz != 0) {
      ++bad;
      if (r != STEP_CONTINUE) break;
      e.n_real = real; e.n_masked = masked; e.trace = trace; e.k = k + 1;
    }
  }
  std::printf("%s-%s-%s-%s %ld %u %ld\n", name, tabs, kBanded ? "banded" : "global", sizeof(R) == 4 ? "f32" : "f64", n, real, bad);
}

template <class R>
static void gas(const char* name, const std::vector<Chan>& cs, double gamma) {
  const Gas<R> g(cs, gamma);
  fly<R, true>(name, "global", cs, g, global_view<R>(g.G), gamma);
  fly<R, false>(name, "global", cs, g, global_view<R>(g.G), gamma);
  fly<R, true>(name, "staged", cs, g, g.fit(), gamma);
  fly<R, false>(name, "staged", cs, g, g.fit(), gamma);
}

int main() {
  const Chan el{CH_ELASTIC, 8.0, 0.0}, ex{CH_EXCITATION, 4.0, 11.5}, ion{CH_IONISATION, 2.0, 15.8};
  const std::vector<Chan> one{el}, two{el, ex}, three{el, ex, ion}, late{ex, el, ion};
  gas<double>("one", one, 16.0); gas<float>("one", one, 16.0);
  gas<double>("two", two, 16.0); gas<float>("two", two, 16.0);
  gas<double>("three", three, 16.0); gas<float>("three", three, 16.0);
  gas<double>("late", late, 16.0); gas<float>("late", late, 16.0);
}
