// Host build of the flight step's filters (AVM_HOST_DEBUG): random flights,
// each answer of a short form against the general one.  Prints the number of
// cases and of disagreements per check.
#define AVM_HOST_DEBUG 1
#include <cmath>
#include <cstdio>
#include <limits>
#include <random>
#include <vector>

#include "avm_device.hpp"

using namespace avm;
static std::mt19937_64 rng(12345);
static double uni(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }

// slab_clear() true must mean slab_inside() true and no exit
template <class R>
static void slab(const char* name) {
  long n = 0, clear = 0, bad = 0;
  for (int i = 0; i < 2000000; ++i) {
    FieldDev F{};
    F.z_lo = i % 3 == 0 ? 0.0 : uni(-5.0, 5.0);
    F.z_hi = F.z_lo + std::pow(10.0, uni(-4.0, 1.0));
    const double half = 0.5 * (F.z_hi - F.z_lo), coord = std::fabs(F.z_lo) + std::fabs(F.z_hi);
    F.z_mid = F.z_lo + half;
    F.z_half = half - (1e-9 * half + 1e-11 * coord);
    F.z_half_f = half - (1e-5 * half + 1e-11 * coord);
    // flights of up to a few gaps, many of them turning close to a plane
    Elec<R> e{};
    const double T = std::pow(10.0, uni(-5.0, 1.0));
    e.z = F.z_lo + (F.z_hi - F.z_lo) * (i % 2 ? uni(-0.01, 1.01) : i % 4 ? std::pow(10.0, uni(-12.0, 0.0)) : 1.0 - std::pow(10.0, uni(-12.0, 0.0)));
    e.vz = (R)(uni(-3.0, 3.0) * half * std::pow(10.0, uni(-4.0, 0.5)) / T);
    const R az = (R)(uni(-2.0, 2.0) * (i % 5 ? std::fabs((double)e.vz) / T : half / (T * T)));
    const R s = (R)T;
    double rx, ry, rz, s_exit = 0.0;
    propagate_r<R>(e, R(0), R(0), az, s, rx, ry, rz);
    ++n;
    if (!slab_clear<R>(F, e.z, rz, e.vz * s)) continue;
    ++clear;
    const double vz = e.vz, a = az;
    bad += !slab_inside(e.z, vz, a, F.z_lo, F.z_hi, (double)s) || slab_exit(e.z, vz, a, F.z_lo, F.z_hi, (double)s, s_exit) ||
           region_status<R, FIELD_SLAB>(F, e);
  }
  std::printf("%s %ld %ld %ld\n", name, n, clear, bad);
}

// the staged tables' band search against the general one
template <class R>
static void bands(const char* name) {
  long n = 0, bad = 0;
  for (int nb : {1, 2, 3, 7, 200, 511, 512})
    for (double e_max : {1.0, 400.0, 977.3}) {
      const int width = 1 + (int)(rng() % 100), bins = nb * width - (int)(rng() % width);
      std::vector<R> gen(nb), fit(nb + 1), g(nb), v(nb);
      GasDev G{};
      G.n_bands = nb;
      G.band_scale = (double)bins / (e_max * (double)width);
      G.band_scale_f = (float)G.band_scale;
      fit[0] = -std::numeric_limits<R>::infinity();
      for (int b = 0; b < nb; ++b) {
        const double edge = ((double)((b + 1) * width) * e_max) / (double)bins;
        R r = (R)edge;
        if ((double)r > edge) r = std::nextafter(r, R(0));
        gen[b] = b == nb - 1 ? std::numeric_limits<R>::infinity() : r;
        fit[b + 1] = b == nb - 1 ? std::numeric_limits<R>::quiet_NaN() : r;
        g[b] = R(b + 1);
        v[b] = R(1) / R(b + 1);
      }
      TabView<R> T{};
      T.bedge = gen.data(); T.bgam = g.data(); T.binv = v.data();
      TabFit<R> F{};
      F.bedge = fit.data() + 1; F.bgam = g.data(); F.binv = v.data();
      std::vector<R> es{R(0), std::numeric_limits<R>::denorm_min(), std::numeric_limits<R>::max(),
                        std::numeric_limits<R>::infinity()};
      for (int b = 0; b < nb - 1; ++b)
        for (R e : {gen[b], std::nextafter(gen[b], R(0)), std::nextafter(gen[b], std::numeric_limits<R>::max())}) es.push_back(e);
      for (int i = 0; i < 2000; ++i) es.push_back((R)uni(0.0, 1.5 * e_max));
      for (R e : es) {
        R ga, ia, ea, gb, ib, eb;
        // (the general search converts the product to an integer: keep it in range here)
        const R lim = e * Sel<R>::band_scale(G) < R(1e9) ? e : (R)(1e8 / G.band_scale);
        const int want = band_of<R>(G, T, lim);
        const int a = band_of_tabs<R>(G, T, lim, ga, ia, ea), b = band_of_tabs<R>(G, F, e, gb, ib, eb);
        ++n;
        bad += band_of<R>(G, F, e) != want || a != want || b != want || ga != gb || ia != ib || (want < nb - 1 && ea != eb);
      }
      const R nan = std::numeric_limits<R>::quiet_NaN();
      bad += band_of<R>(G, F, nan) != nb - 1;
    }
  std::printf("%s %ld %ld %ld\n", name, n, n, bad);
}

int main() {
  slab<double>("slab_f64");
  slab<float>("slab_f32");
  bands<double>("bands_f64");
  bands<float>("bands_f32");
}
