// Rules that choose a kernel's form or launch shape by sizes and types: plain
// C++, so that a host test holds each rule against the times it was drawn
// from.  Times are of gfx950, three sets of buffers in turn, kernels alone.
#pragma once

#include <cstdint>
#include <initializer_list>

namespace pdiv {

// The ensemble fit's form: points a thread and members in flight.
//   kOne8   a point, eight members: four times as many waves hide the loads
//           of small grids and short ensembles;
//   kFour2  four points (16-byte loads of float32), two members;
//   kFour4  four points, four members: a wave hides more by itself, at half
//           the waves, and members past a multiple of four are walked one at a
//           time.
// The forms of four take over where the members outgrow the caches: two
// components of n points and m members from about 88 MiB.  kOne8 / kFour2 /
// kFour4, us: float32 250k points x50 19.8 / 21.3 / 23.2, 340k x32 16.0 / 16.9 /
// 18.2, 500k x22 16.8 / 16.3 / 18.6, x28 23.8 / 19.8 / 20.6, 1000x1000 x12 22.7 /
// 22.8 / 22.6, x22 38.1 / 34.3 / 34.2, 1448x1448 x10 39.1 / 38.4 / 40.2, x18 65.6 /
// 60.5 / 60.2; 16-bit 760k x25 17.6 / 19.6 / 18.8, x35 25.7 / 23.8 / 24.3, 1200x1000
// x18 23.6 / 24.6 / 24.1, x28 34.3 / 31.7 / 32.4.  Between kFour2 and kFour4 the grid
// decides: float32 1.2 M points x20 40.4 / 39.3, 2.8 M x15 69.1 / 78.1; 16-bit 1.45 M
// x24 35.7 / 33.6, 2000x2000 x18 68.0 / 72.2.
enum class FitForm { kOne8, kFour2, kFour4 };

constexpr FitForm fit_form(int in_bytes, int out_bytes, int64_t n, int64_t m) {
  constexpr int64_t kMi = int64_t(1) << 20;
  const int64_t stream = 2 * in_bytes * m * n;
  if (in_bytes == 4) {
    // (16-bit results, of which a wave of single points stores 128 bytes a
    // plane: 2.8 M points x10 47.5 us, 44 in fours)
    const int least = out_bytes == 2 && n >= 7 * kMi / 5 ? 10 : 12;
    if (n < 3 * kMi / 10 || m < least || stream < 88 * kMi) return FitForm::kOne8;
    return n >= kMi && n < 9 * kMi / 4 ? FitForm::kFour4 : FitForm::kFour2;
  }
  // 16-bit to 16-bit: short streams and the stores decide earlier (400k points
  // x20 9.0 us in fours, 10.2 by single points; 2.8 M x13 33, 38)
  if (out_bytes == 2 && ((n >= 3 * kMi / 8 && n < 4 * kMi / 5 && m >= 12) ||
                         (n >= 19 * kMi / 10 && m >= 10)))
    return FitForm::kFour4;
  // 16-bit to float32 on less than half a million points (500k x20 10.7 / 12.7 /
  // 10.1, x40 18.3 / 19.4 / 15.8)
  if (n < kMi / 2)
    return n >= 3 * kMi / 8 && ((m % 4 == 0 && m >= 20) || m >= 40) ? FitForm::kFour4
                                                                    : FitForm::kOne8;
  if (m < 17 || stream < 88 * kMi) return FitForm::kOne8;
  return n >= 19 * kMi / 20 && n < 3 * kMi ? FitForm::kFour4 : FitForm::kFour2;
}

// 3D divergence Gaussians: z slices a wave walks, and whether the results are
// streamed past the caches (non-temporal stores).
//
// Up to 2 M points: short walks until they make waves enough, longer ones past
// that, the chunk's ends re-reading W; 16-bit volumes and short rows are streamed
// from 0.3 M (below, a launch's tail waits for such stores: 28x78x61 16-bit 3.1 us
// with default ones, 3.4; 91x29x29 float32 2.9, 3.2) (float32, 4 / 6 / 12 slices, us: 100x120x64
// 5.8 / 6.1 / 8.3, 151x192x71 14.3 / 13.5 / 14.3; 16-bit, streamed: 120x120x100 8.9 /
// 8.3 / 9.5, 151x192x71 14.1 / 13.1 / 12.5; rows of 32 points, half a wave each,
// as 16-bit ones: 175x327x32 13.6 / 12.6 / 12.5).
//
// Larger volumes: rows of whole 64-byte sectors (nx a multiple of 16) are
// streamed: their stores need no other wave's, and the inputs stay in the
// caches.  Other rows' ends are completed there by the neighbouring wave's
// stores, so they take default stores; except that a volume whose inputs just
// fit the 256 MB cache beside two others keeps them there when the results go
// past it (inputs up to 88 MiB; of float32 from 2.3 Mi points: 114x442x47 13.2 / 15.3
// us, all of it in the cache; 117x54x453 21.1 / 16.6).  Default / streamed, us,
// inputs from a set of three: float32 89x182x193 27.4 / 18.6 (of many sets 29.1 /
// 31.1), 150x300x129 45.6 / 50.8, 200x250x190 72.1 / 81.7, 256x400x251 179 / 201, but 256x256x256 114 / 111,
// 150x50x496 29.2 / 25.2, 400x512x384 515 / 500; 16-bit 150x300x129 37.1 / 24.5 (36.7 /
// 38.4), 180x200x220 42.0 / 44.6, 256x400x251 121 / 134, 400x512x384 330 / 315.
// Slices: 4, 6 for streamed 16-bit volumes (150x300x129 4 / 6 / 12: 27.6 / 24.5 / 24.6),
// 12 on rows that leave lanes idle (188x445x32 float32 18.1 / 16.5 / 16.0, 279x508x35
// 16-bit 28.4 / 25.8 / 23.5; 224x359x74 16-bit 28.8 with 6, 26.8 with 12).
struct Div3Shape {
  int z_chunk;
  bool stream;
};

constexpr Div3Shape div3_shape(int in_bytes, int64_t nz, int64_t ny, int64_t nx) {
  constexpr int64_t kMi = int64_t(1) << 20;
  const int64_t points = nz * ny * nx;
  if (points <= 2 * kMi) {
    const int64_t waves = (nx + 63) / 64 * ((ny + 3) / 4 * 4) * ((nz + 3) / 4);  // of 4 slices
    if (in_bytes == 4 && nx > 32) return {waves < 9000 ? 4 : 6, false};
    return {waves < 6000 ? 4 : waves < 11000 ? 6 : 12, points >= 3 * kMi / 10};
  }
  const bool stream = nx % 16 == 0 || (6 * in_bytes * points <= 88 * kMi &&
                                       (in_bytes == 2 || points >= 7 * kMi / 3));
  const int64_t lanes = (nx + 63) / 64 * 64;
  const bool idle = nx <= 48 || (in_bytes == 2 && 100 * nx <= 78 * lanes);
  return {!stream ? 4 : idle ? 12 : in_bytes == 2 ? 6 : 4, stream};
}

// Isocontours: four waves per cell row instead of one, where a wave per row
// would be few waves with long walks.  A wave takes batches of 512 cells.
//
// Counting, for rows of more than one batch: up to 1200 of them, 1400 of three
// batches, 3600 of more, whose longer walks hide less (one / four waves, us: 300x8192
// 12.7 / 8.0, 1000x4096 9.9 / 8.2, 1533x3180 11.4 / 9.8, 2000x4096 13.6 / 13.1,
// 2500x3000 13.6 / 12.4, 3500x2300 14.5 / 14.0, 4096x4096 20.0 / 21.5; two batches
// 1600x1024 0.97 of the time with one, three 1800x1440 0.98).
constexpr bool contour_counts_by_blocks(int64_t rows, int64_t nx) {
  const int64_t batches = (nx - 1 + 511) / 512;
  return batches > 1 && rows <= (batches == 2 ? 1200 : batches == 3 ? 1400 : 3600);
}
// Writing, whose waves wait for each other at every round of four batches: a
// row whose last round is not full leaves waves idle, so the fewer of its
// places a row fills the fewer rows pay (by the fourth power of the share;
// count, scan and write, one / four waves: 1 batch 4096x513 14.1 / 22.6; 2
// batches 300x1024 11.4 / 10.1, 2000x1024 13.7 / 15.7; 3 batches 1000x1440 14.1 /
// 12.4, 4096x1440 25.2 / 27.2; 4 batches 4096x2049 30.8 / 29.3; 5 batches 1000x2300
// 18.9 / 16.5, 4096x2300 35.8 / 39.9; 8 batches 4096x4096 51.1 / 50.0, 8192x4096
// 90.6 / 93.7, 12 batches 8192x6000 134 / 127).
constexpr bool contour_writes_by_blocks(int64_t rows, int64_t nx) {
  const double batches = double((nx - 1 + 511) / 512);
  const double share = batches / (4.0 * double((nx - 1 + 2047) / 2048));
  return nx - 1 > 512 && double(rows) <= 10000.0 * share * share * share * share;
}

// Batches.  The layout of line-aligned fused ones: the paired tile from so many
// million cells (in all fields) by storage and isovalue slots (of the mean count
// where the fields' differ: it is the stores that gain); below, its seam step
// and staged rows cost more than whole-line stores save.  Split / paired
// at their best heights, us: float32 9.0 M cells x4 73 / 65, 8.1 M x6 78 / 75, 5.2 M
// x13 119 / 99, 3.5 M x15 77 / 71, 2.9 M x15 65 / 68; 16-bit 13.7 M x2 48 / 66, 14 M x4 1.2
// times the paired time, 10 M 0.78; 10 M x6 1.25 times, 7 M 0.87; 3.5 M x14 78 / 73.
constexpr bool batch_paired(int64_t cells, int in_bytes, int kc) {
  constexpr int64_t k100 = 100000;
  const int64_t least = in_bytes == 2 ? (kc >= 16   ? 33
                                         : kc >= 12 ? 30
                                         : kc >= 8  ? 64
                                         : kc >= 6  ? 90
                                         : kc >= 3  ? 120
                                                    : 160)
                                      : (kc >= 16   ? 30
                                         : kc >= 12 ? 33
                                         : kc >= 8  ? 55
                                         : kc >= 6  ? 70
                                         : kc >= 3  ? 92
                                                    : 115);
  return kc >= 2 && cells >= least * k100;
}

// SIMDs of a whole MI355X (256 CUs of four); on a part of one the rules below
// only lose speed.
constexpr int64_t kSimds = 1024;

// The band height, by the number of tiles a height leaves: 8, 4, 2 or 1 rows
// from 6000, 3000 and 1500 tiles (paired: 32 or 16 from 16000 and 4000), unless
// the rows that the fullest SIMD walks promise a twentieth off: as lcp_band_rows
// for one field, n (b + 0.7) for n rounds of the batch's tiles(b), a SIMD's only
// wave counted twice and the second, below 8 slots, 1.15 times.  Split tiles of
// many isovalues are mostly stores and gain nothing past 8 rows, those of
// 16-bit storage past 3 (15.7 M cells x11 into dense maps 260 us, 340 with 8).  Over
// 2879 batches of 8 to 64 fields of 64 to 2048 a side, times are 1.8% above the best
// shape's on average; by tile numbers alone 6.0%, and 70 were slower than a
// resident grid of 16-row tiles (3.3 M cells x14 on lines 85 us, 72 there, 70 now).
template <typename Tiles>
constexpr int batch_band_rows(const Tiles& tiles, bool fused, int in_bytes, bool paired, int kc) {
  const int tallest = !fused || paired || kc < 12 ? 16 : in_bytes == 2 ? 3 : 8;
  if (tallest >= 8 && tiles(8) >= 9000) return !paired ? 8 : tiles(32) >= 16000 ? 32 : 16;
  auto cost = [&](int b) {
    const int64_t n = (tiles(b) + kSimds - 1) / kSimds;
    return n * (10 * b + 7) * (n == 1 ? 40 : n == 2 && kc < 8 ? 23 : 20);
  };
  int64_t least = INT64_MAX;
  int best = 1;
  for (int b : {1, 2, 3, 4, 6, 8, 12, 16}) {
    if (b > tallest) break;
    const int64_t c = cost(b);
    if (c < least) least = c, best = b;
  }
  const int by_tiles = paired && tiles(16) >= 4000 ? 16
                       : tiles(8) >= 6000          ? 8
                       : tiles(4) >= 3000          ? 4
                       : tiles(2) >= 1500          ? 2
                                                   : 1;
  return by_tiles <= tallest && 20 * cost(by_tiles) <= 21 * least ? by_tiles : best;
}

// Whether b-row bands are a nearly full round of two waves per SIMD.
constexpr bool fills_two_waves(int64_t strips, int64_t rows, int b) {
  const int64_t waves = strips * ((rows + b - 1) / b);
  return waves > 17 * kSimds / 10 && waves <= 2 * kSimds;
}

// Layout choice, from float32 maps of 300^2 to 8192^2 cells at the best band
// height of each tile, three sets of buffers in turn (split against paired,
// us).  The paired tile's whole-line stores pay once the maps outgrow the
// caches; its seam step and, fused, its staged rows cost more than they
// save below that.
//   fused, rows on lines: at 1, 2, 4 isovalues 721x1440 6.8 / 9.5, 8.1 / 10.8,
//     11.0 / 13.1, 1448^2 16.2 / 19.4 at 4, 2047x3001 28.0 / 25.5, 34.4 /
//     30.9, 49.6 / 43.3: paired from 2^22 cells; at 8 and more 721x1440 15.5 /
//     17.3 (16: 27.1 / 27.1), 1448^2 32.5 / 26.8 and 55.7 / 42.8: paired from
//     1.25 M cells.
//   fused, other rows (default store policy): 2047x3001 at 1, 4, 8, 16
//     isovalues 27.8 / 28.7, 48.9 / 49.1, 78.2 / 76.3, 135.5 / 131.7;
//     3000x3500 49.4 / 52.3, 82.7 / 85.4, 125.9 / 131.4, 233 / 227; 4096^2
//     77.8 / 74.4, 130.9 / 122, 202 / 190, 357 / 334: paired from 12 M cells,
//     or 7 M where its 32-row bands are just two waves per SIMD (947x7889 at 2, 8
//     isovalues 42.1 / 41.0, 93.0 / 89.1), at 12 and more slots from 6 M.  16-bit
//     storage: at 12 and more slots from 1.5 M (1021x1531 x12 35.8 / 30.6, 2129x1804
//     x12 100 / 69), at 3 and 4 from 40 M (2123x6863 at 4 92.5 / 99.4, 8192x8192 412 /
//     382), at 1 and 2 never (2123x6863 46.8 / 59.5, 60.1 / 71.8, 8000x8191 182 / 224,
//     244 / 270).
//   two-step, rows on lines: 721x1440 4.4 / 5.1 at 1 isovalue, 9.5 / 8.4 at 4,
//     24.3 / 23.0 at 16; 4096^2 43.9 / 44.3, 99.5 / 83.1, 339 / 268: paired
//     except at 1 isovalue and on the smallest maps (300^2: equal).
//   two-step, other rows: split only.
constexpr bool use_paired_tile(bool fused, bool lines, int in_bytes, int kc, int64_t ny,
                               int64_t nx) {
  constexpr int64_t kM = 1000000;
  const int64_t cells = (ny - 1) * (nx - 1);
  if (!fused) return lines && kc >= 2 && cells >= kM / 4;
  if (lines) return cells >= (kc >= 8 ? kM * 5 / 4 : int64_t(1) << 22);
  if (in_bytes == 2 && kc <= 4) return kc >= 3 && cells >= 40 * kM;
  if (kc >= 12) return cells >= (in_bytes == 2 ? 3 * kM / 2 : 6 * kM);
  return cells >= 12 * kM ||
         (cells >= 7 * kM && kc >= 2 && fills_two_waves((nx - 1 + 127) / 128, ny - 1, 32));
}

// Cell rows per wave band.  A band re-evaluates one corner row and re-reads
// two input rows, so tall bands do less work; but a wave walks its band row
// by row, so a grid of few tall bands leaves SIMDs idle while a few waves
// walk (500x500, 1 isovalue, fused: 15.9 us with 32-row bands, 9.3 / 6.0 /
// 4.3 / 3.6 / 3.4 us with 16 / 8 / 4 / 2 / 1).
//
// Grids of less than eight 8-row bands per SIMD: the time goes with the rows
// that the fullest of the 1024 SIMDs walks, a band's own redundant work at
// half a row, n (b + 1/2) for n = ceil(waves / 1024).  1448x1448, 4 isovalues
// into dense maps, 2 ... 10 rows: 18.1 17.3 18.1 16.7 15.7 17.0 18.0 15.5 16.2 us
// (n = 9 6 5 4 3 3 3 2 2), 12 / 14 / 16: 17.8 / 19.8 / 21.5.  A SIMD's only wave
// hides no latency (721x1440, 8 isovalues, 9 rows: 17.0 us, 15.2 with 3), and
// with few isovalues two hide less than three (1000x1000, 2 isovalues, 4 rows:
// 8.3 us, 7.8 with 2).  Against the tallest band that gives a number of waves
// (6000, 3000 and 1500 for 8, 4 and 2 rows), over 208 sizes, counts and
// layouts from 300x300 to 2047x3001 the times fall by 2.3% on average: 721x1440
// 16.2 to 14.8 us at 8 isovalues and 29.6 to 25.8 at 16, 1448^2 17.1 to 15.6 at 4
// and, on lines, 44.9 to 40.5 at 16, 2047x3001 on lines 47.7 to 44.4 at 4.  Taller
// bands than 8 rows gain nothing where the stores are most of the work, the
// two-step path and many isovalues on rows that start inside a line
// (1500x4000, 16 isovalues into dense maps, 16 rows: 142.7 us, 137.5 with 8).
//
// Larger grids, whose SIMDs even out: the split tile gains nothing from more
// than 8 rows at any size (8192^2, 16 isovalues, two-step: 1.30 ms with 8 rows,
// 1.41 / 1.44 / 1.50 with 16 / 32 / 64); the paired one takes up to 64 (8192^2 fused,
// 16 isovalues: 1.106 ms, 1.125 / 1.174 / 1.176 with 32 / 16 / 8; 5792^2: 656,
// 601, 593, 608 us with 64 / 32 / 16 / 8; 4096^2 into dense maps 343, 334, 337,
// 348 us).
//
// The paired tile where tall bands are just two waves per SIMD, all resident at
// once: 32 rows into other rows (947x7889 at 8 isovalues 89.1 us, 94.5 with 16; with
// 3500 and more waves, too: 2123x6863 at 1 67.6, 70.3), float32 on lines up to 3
// isovalues (1668x4457 at 1 32.5, 34.4 with 10); 64 rows there up to 4 (4096x4097 at 1,
// 4 68.4, 110 us, 71.6, 115 with 32) from the 4000 waves of 32 rows that would else
// take those; with fewer 16 rows are as fast (1704 random sizes: 64 against 16 rows
// 1.00, 1.02, 1.04, 1.04 of the time at 1 to 4; 2189x6583 at 4 106 us, 96).
constexpr int lcp_band_rows(int64_t strips, int64_t rows, bool paired, bool fused, bool lines,
                            int in_bytes, int kc) {
  auto waves = [&](int b) { return strips * ((rows + b - 1) / b); };
  if (paired && fused) {
    if (lines && in_bytes == 4 && kc <= 4 && waves(32) >= 4000 &&
        fills_two_waves(strips, rows, 64))
      return 64;
    if ((lines ? in_bytes == 4 && kc <= 3 : in_bytes == 4 || kc <= 12) &&
        fills_two_waves(strips, rows, 32))
      return 32;
  }
  if (waves(8) >= 8000) {
    if (paired && waves(64) >= 8000) return 64;
    if (paired && waves(32) >= (fused && !lines && kc < 12 ? 3500 : 4000)) return 32;
    if (paired && waves(16) >= 6000) return 16;
    return 8;
  }
  const int tallest = fused && (paired || kc < 12) ? 16 : 8;
  int64_t least = INT64_MAX;
  int best = 1;
  for (int b = 1; b <= tallest; ++b) {
    const int64_t n = (waves(b) + kSimds - 1) / kSimds;
    const int64_t cost = n * (2 * b + 1) * (n == 1 ? 40 : n == 2 && kc < 8 ? 23 : 20);
    if (cost < least) least = cost, best = b;
  }
  return best;
}

// 3D LCP: vertex rows per band.  A band's first row is evaluated for both bands and
// its V window loaded again, but a wave walks its rows one after another, so
// small volumes want short bands (100x130x150, fused, 4 isovalues, us with 1 /
// 2 / 4 / 8 / 16 / 32 rows: 33 / 28 / 30 / 38 / 46 / 87; two-step 25 / 20 / 22 /
// 28 / 35 / 67; 48^3 7 / 9 / 14 / 23 / 43 / 81; 180x200x220 123 / 107 / 98 / 100
// / 113 / 140; 256x512x384 578 / 558 / 564 / 586 with 4 ... 32; 512^3 1573 / 1487
// / 1500 / 1563).  The line-aligned tile at 8 isovalues, most work per row, takes
// 32 rows on large volumes (512^3, 16 isovalues in two launches 2734 us with 16,
// 2687 with 32; 256x512x384, 8: 522, 534).
constexpr int band_rows3(int64_t columns, int64_t rows, bool lines, int kc) {
  auto waves = [&](int b) { return columns * ((rows + b - 1) / b); };
  if (lines && kc == 8 && waves(32) >= 12000) return 32;
  if (waves(16) >= 12000) return 16;
  if (waves(8) >= 8000) return 8;
  return waves(4) >= 3000 ? 4 : waves(2) >= 1500 ? 2 : 1;
}

// Fused 3D LCP: strips of 63 cells, whose end lanes load the neighbours that
// they miss, instead of 61 with two halo lanes, where they save a strip: always
// of float32, where U's extra loads are the smaller part; of 16-bit storage at
// 3, 4 and 7 isovalues up to 4 strips of 61, at 8 up to 6 (there the registers of
// the extra loads cost a wave per SIMD).  61 / 63 cells against the kernels of 63
// and 64 cells that loaded every lane's neighbours, 1 / 4 / 8 / 16 isovalues into
// dense maps: float32 256x512x64 (2 / 1 strips) 1.15 / 0.98, 1.18 / 0.98, 1.42 /
// 1.05, 1.48 / 1.01; 200x300x251 (5 / 4) 1.04 / 1.00, 1.08 / 1.02, 1.02 / 0.92, 1.12 /
// 0.92; 300x400x500 (9 / 8) 1.01 / 0.99, 1.03 / 0.99, 0.97 / 0.94, 0.98 / 0.92;
// bfloat16 200x300x126 (3 / 2) 0.91 / 0.77, 0.90 / 0.83, 1.15 / 0.95, 1.24 / 0.94, but
// 300x400x500 0.94 / 0.99 at 4, 0.96 / 0.98 at 8.
constexpr bool lcp3d_wide_strips(int64_t nx, int in_bytes, int n_iso) {
  const int64_t narrow = (nx - 1 + 60) / 61, wide = (nx - 1 + 62) / 63;
  if (wide >= narrow) return false;
  if (in_bytes == 4) return true;
  return n_iso == 3 || n_iso == 4 || n_iso == 7 ? narrow <= 4 : n_iso != 8 || narrow <= 6;
}

// Whether a volume takes them: where they also leave the fullest of the 1024 SIMDs
// less to walk, n (b + 1) for n = ceil(waves / 1024) bands of b rows.  A strip less
// is often no round less on small volumes, and a wave of 63 cells walks slower
// (61 / 63 cells: 27x58x249, 1 isovalue, float16 5.6 / 7.1 us; 88x24x435, 7, float32
// 24.8 / 27.8).  Over 11400 random volumes of up to 6 M points the count picks the
// slower by more than 3% in 3 of the cases that it changes; 3077 without it.
constexpr bool lcp3d_takes_wide(int64_t nz, int64_t ny, int64_t nx, int in_bytes, int n_iso) {
  if (!lcp3d_wide_strips(nx, in_bytes, n_iso)) return false;
  const int64_t layers = n_iso <= 4 ? 4 : 3;  // cell layers a wave
  const int64_t groups = (nz - 1 + layers - 1) / layers;
  auto cost = [&](int64_t cells) {
    const int64_t columns = groups * ((nx - 1 + cells - 1) / cells);
    const int b = band_rows3(columns, ny - 1, false, n_iso);
    const int64_t waves = columns * ((ny - 1 + b - 1) / b);
    return (waves + kSimds - 1) / kSimds * (b + 1);
  };
  return cost(63) < cost(61);
}

}  // namespace pdiv
