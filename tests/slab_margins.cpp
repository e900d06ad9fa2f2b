// Host build of the slab filter with the margins the library gives a field:
// flights that end or turn within a few margins of a plane.  Prints the flights,
// those the filter passes, and those of them that may leave.
#define AVM_HOST_DEBUG 1
#include <cmath>
#include <cstdio>
#include <random>

#include "avm_device.hpp"

using namespace avm;
static std::mt19937_64 rng(99);
static double uni(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }

template <class R>
static void run(const char* name) {
  long n = 0, clear = 0, bad = 0;
  for (int i = 0; i < 2000000; ++i) {
    FieldDev F{};
    F.z_lo = i % 3 == 0 ? 0.0 : uni(-5.0, 5.0);
    F.z_hi = F.z_lo + std::pow(10.0, uni(-4.0, 1.0));
    set_slab_filter(F);
    const double gap = F.z_hi - F.z_lo, T = std::pow(10.0, uni(-5.0, 1.0));
    // a distance from a plane, from well inside the rounding to a tenth of the gap
    const double d = gap * std::pow(10.0, uni(sizeof(R) == 8 ? -14.0 : -9.0, -1.0));
    const bool top = i & 1;
    const double at = top ? F.z_hi - d : F.z_lo + d, out = top ? 1.0 : -1.0;
    // the flight ends (even) or turns (odd) there, from up to half a gap away
    const double far = gap * uni(0.0, 0.5), z0 = at - out * far;
    Elec<R> e{};
    e.z = z0;
    R az;
    if (i >> 1 & 1) {
      // vertex at time f T: far = v^2 / (2 |a|), v = |a| f T
      const double f = uni(0.05, 0.95), a = 2.0 * far / (f * T * f * T);
      e.vz = (R)(out * a * f * T);
      az = (R)(-out * a);
    } else {
      const double h = far * uni(-1.0, 1.0);
      az = (R)(out * 2.0 * h / (T * T));
      e.vz = (R)(out * (far - h) / T);
    }
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

int main() {
  run<double>("f64");
  run<float>("f32");
}
