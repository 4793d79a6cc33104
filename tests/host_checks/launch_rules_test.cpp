// Host check of the launch rules (csrc/launch_rules.hpp, the header the
// library compiles) against times measured on gfx950: at each measured point
// the rule's choice takes no more than 3% over the fastest of the choices, or
// over the form that a rule replaced where that is named.
// Built with g++ under ASan/UBSan.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../../paper_2510_01190_amd/csrc/launch_rules.hpp"

namespace {

int failures = 0;

void check(bool ok, const char* what, double a, double b, double c) {
  if (!ok) {
    std::printf("FAIL %s (%g, %g, %g)\n", what, a, b, c);
    ++failures;
  }
}

// Ensemble fit: kOne8 and kFour2 relative to kFour4, the form every grid took
// before; no grid may be left with one more than 4% slower than it.
struct FitTime {
  int in, out;
  double mi;  // 2^20 points
  int m;
  double one8, four2;
};

void check_fit() {
  const FitTime times[] = {
      {4, 4, 0.0625, 15, 0.45, 0.84}, {4, 4, 0.238, 20, 0.85, 0.98}, {4, 4, 0.238, 50, 0.86, 0.92},
      {4, 4, 0.324, 32, 0.88, 0.93},  {4, 4, 0.41, 25, 0.93, 0.95},  {4, 4, 0.41, 28, 1.08, 0.94},
      {4, 4, 0.477, 22, 0.89, 0.88},  {4, 4, 0.477, 24, 1.07, 0.96}, {4, 4, 0.591, 18, 0.86, 0.94},
      {4, 4, 0.591, 20, 1.10, 0.98},  {4, 4, 0.725, 18, 1.03, 0.97}, {4, 4, 0.906, 18, 1.14, 1.01},
      {4, 4, 0.954, 22, 1.09, 1.00},  {4, 4, 0.989, 18, 1.08, 1.00}, {4, 4, 0.989, 20, 1.06, 0.99},
      {4, 4, 0.989, 50, 1.12, 1.00},  {4, 4, 1.144, 20, 1.12, 1.03}, {4, 4, 1.24, 22, 1.14, 1.05},
      {4, 4, 2.0, 10, 0.96, 0.97},    {4, 4, 2.0, 18, 1.11, 1.01},   {4, 4, 2.0, 23, 1.12, 1.00},
      {4, 4, 2.67, 15, 0.93, 0.87},   {4, 4, 3.81, 12, 1.03, 1.00},  {4, 4, 3.81, 18, 0.98, 0.91},
      {2, 4, 0.0625, 30, 0.46, 1.15}, {2, 4, 0.238, 50, 0.85, 1.30}, {2, 4, 0.41, 20, 1.06, 1.20},
      {2, 4, 0.477, 30, 0.92, 1.04},  {2, 4, 0.477, 40, 1.15, 1.23}, {2, 4, 0.591, 50, 1.09, 0.98},
      {2, 4, 0.725, 25, 0.99, 1.01},  {2, 4, 0.725, 35, 1.06, 0.96}, {2, 4, 0.906, 24, 0.93, 0.94},
      {2, 4, 0.906, 35, 1.11, 0.92},  {2, 4, 0.989, 24, 0.96, 1.04}, {2, 4, 0.989, 30, 1.08, 1.05},
      {2, 4, 1.144, 28, 1.05, 0.99},  {2, 4, 1.383, 16, 0.89, 1.07}, {2, 4, 1.383, 25, 1.07, 1.04},
      {2, 4, 2.0, 18, 1.03, 0.98},    {2, 4, 2.67, 18, 1.07, 1.05},  {2, 4, 3.81, 18, 0.94, 0.93},
      {2, 4, 5.72, 26, 0.95, 0.93},  {2, 2, 0.143, 20, 0.81, 1.29}, {2, 2, 0.381, 20, 1.13, 1.19},
      {2, 2, 0.496, 16, 1.10, 1.17}, {2, 2, 0.725, 20, 1.09, 1.04}, {2, 2, 0.858, 24, 0.98, 0.89},
      {2, 2, 2.0, 13, 1.11, 1.04},   {2, 2, 2.67, 10, 1.10, 1.01},  {4, 2, 2.67, 10, 1.08, 1.02},
  };
  for (const FitTime& t : times) {
    const pdiv::FitForm f = pdiv::fit_form(t.in, t.out, int64_t(t.mi * (1 << 20)), t.m);
    const double took = f == pdiv::FitForm::kOne8    ? t.one8
                        : f == pdiv::FitForm::kFour2 ? t.four2
                                                     : 1.0;
    check(took <= 1.04 && took <= 1.12 * std::min(t.one8, std::min(t.four2, 1.0)), "fit", t.in,
          t.mi, t.m);
  }
}

}  // namespace

int main() {
  check_fit();
  if (failures == 0) std::printf("ALL PASS\n");
  return failures != 0;
}
