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

// 3D divergence Gaussians: the times of default and of streamed stores with 4,
// 6 and 12 slices, relative to 12 slices with streamed stores, the shape that
// every volume took before; no volume may be left more than 4% slower.
struct Div3Time {
  int bytes, nz, ny, nx;
  double plain[3], streamed[3];
};

void check_div3() {
  const Div3Time times[] = {
      {4, 100, 100, 32, {0.74, 0.76, 1.06}, {0.70, 0.71, 1.00}},
      {2, 150, 200, 32, {1.04, 0.95, 1.07}, {0.97, 0.89, 1.01}},
      {4, 175, 327, 32, {1.12, 1.04, 1.03}, {1.08, 1.00, 0.99}},
      {2, 175, 327, 32, {1.19, 1.10, 1.06}, {1.11, 1.03, 0.99}},
      {2, 250, 400, 32, {1.17, 1.08, 1.04}, {1.13, 1.03, 1.00}},
      {2, 100, 200, 72, {1.04, 1.02, 1.05}, {0.98, 0.97, 0.99}},
      {4, 59, 396, 72, {1.04, 0.98, 0.99}, {1.03, 1.00, 1.00}},
      {2, 59, 396, 72, {1.17, 1.10, 1.06}, {1.12, 1.04, 1.00}},
      {4, 151, 192, 71, {0.94, 0.89, 0.94}, {0.92, 0.95, 1.00}},
      {2, 151, 192, 71, {1.17, 1.09, 1.04}, {1.12, 1.04, 0.99}},
      {2, 100, 120, 64, {0.72, 0.77, 1.08}, {0.65, 0.71, 1.00}},
      {2, 120, 120, 100, {0.99, 0.92, 1.04}, {0.94, 0.87, 1.00}},
      {4, 89, 182, 193, {1.349, 1.320, 1.426}, {0.915, 0.910, 1.000}},
      {2, 89, 182, 193, {1.061, 0.971, 1.004}, {1.034, 0.945, 1.004}},
      {4, 110, 190, 160, {1.034, 1.066, 1.140}, {0.871, 0.896, 0.988}},
      {2, 128, 160, 160, {1.006, 0.994, 1.037}, {0.958, 0.945, 0.997}},
      {2, 150, 200, 130, {1.158, 1.043, 1.017}, {1.127, 1.008, 0.995}},
      {4, 150, 300, 129, {0.827, 0.839, 0.894}, {0.921, 0.932, 0.992}},
      {2, 150, 300, 129, {1.510, 1.469, 1.516}, {1.121, 0.994, 0.998}},
      {4, 150, 50, 496, {1.11, 1.09, 1.15}, {0.96, 0.96, 0.99}},
      {4, 299, 139, 112, {1.10, 1.10, 1.06}, {1.02, 1.01, 1.00}},
      {4, 188, 445, 32, {1.31, 1.29, 1.30}, {1.13, 1.03, 1.00}},
      {2, 279, 508, 35, {1.48, 1.42, 1.40}, {1.20, 1.09, 0.99}},
      {4, 279, 508, 35, {0.89, 0.90, 0.90}, {0.95, 1.01, 0.99}},
      {4, 200, 250, 190, {0.952, 0.943, 0.922}, {1.079, 1.064, 1.003}},
      {2, 180, 200, 220, {0.898, 0.926, 0.969}, {0.953, 0.978, 1.005}},
      {2, 256, 512, 64, {1.083, 1.053, 1.073}, {0.996, 0.951, 0.995}},
      {2, 256, 256, 256, {1.029, 1.000, 1.023}, {0.988, 0.958, 0.998}},
      {4, 256, 400, 251, {0.856, 0.874, 0.885}, {0.961, 0.985, 0.998}},
      {2, 400, 512, 384, {1.021, 1.015, 1.024}, {1.000, 0.974, 0.995}},
  };
  for (const Div3Time& t : times) {
    const pdiv::Div3Shape s = pdiv::div3_shape(t.bytes, t.nz, t.ny, t.nx);
    const int z = s.z_chunk == 4 ? 0 : s.z_chunk == 6 ? 1 : 2;
    check(s.z_chunk == 4 || s.z_chunk == 6 || s.z_chunk == 12, "div3 slices", t.nz, t.ny, t.nx);
    check((s.stream ? t.streamed : t.plain)[z] <= 1.04, "div3", t.bytes, t.nz, t.nx);
  }
}

// Isocontours: count, scan and write with a wave a row (both passes), with a
// block a row (both passes), and counting alone with each; the choice may not
// lose more than 4% to a wave a row, the form that every field took before.
struct ContourTime {
  int rows, nx;
  double wave, block, count_wave, count_block;
};

void check_contour() {
  const ContourTime times[] = {
      {63, 513, 8.8, 8.8, 4.9, 4.9},         {4095, 513, 14.1, 22.6, 8.2, 9.4},
      {299, 600, 11.0, 10.1, 5.6, 5.4},      {1999, 600, 13.3, 15.7, 6.9, 7.2},
      {16383, 1024, 55.2, 76.3, 29.0, 33.3}, {999, 1440, 14.1, 12.4, 6.1, 6.1},
      {1999, 1440, 16.5, 16.7, 7.5, 7.8},    {35999, 1440, 156.0, 180.0, 73.0, 83.5},
      {1999, 1800, 20.2, 18.2, 8.3, 8.5},    {4095, 2049, 30.8, 29.3, 13.7, 13.8},
      {4095, 2300, 35.8, 39.9, 15.0, 15.4},  {999, 3000, 21.3, 17.3, 7.7, 7.2},
      {8191, 3000, 66.4, 74.5, 27.1, 28.9},  {1999, 4096, 35.3, 29.4, 13.2, 13.2},
      {4095, 4096, 51.1, 50.0, 20.0, 21.5},  {16383, 4096, 190.8, 189.9, 71.3, 73.2},
      {299, 8192, 43.8, 21.2, 12.7, 8.0},    {8191, 6000, 134.4, 126.9, 47.9, 46.6},
  };
  for (const ContourTime& t : times) {
    const double count = pdiv::contour_counts_by_blocks(t.rows, t.nx) ? t.count_block
                                                                      : t.count_wave;
    const double write = pdiv::contour_writes_by_blocks(t.rows, t.nx) ? t.block - t.count_block
                                                                      : t.wave - t.count_wave;
    check(count <= 1.06 * t.count_wave, "contour count", t.rows, t.nx, count);
    check(count + write <= 1.04 * t.wave, "contour", t.rows, t.nx, count + write);
  }
}

}  // namespace

int main() {
  check_contour();
  check_fit();
  check_div3();
  if (failures == 0) std::printf("ALL PASS\n");
  return failures != 0;
}
